// Decode-sized layer forward (at most 64 tokens) for gfx950:
//   Y = sum_i Wq(i)^T q(T(i) X(i))      (layer forward-pass equation)
// with the weights already transformed and quantized:
//   * gemm_skinny_kernel and its variants: the MXFP4 GEMM alone for few tokens, or few output channels (wush_linear, and
//     wush_layer_decode behind the activation quantizer);
//   * layer_decode_kernel: activation transform + quantization + GEMM in ONE launch, the slower form on this part: only where
//     a test or measurement asks wush_layer_decode for it (kDbgDecodeFused).
// At these sizes the layer is bound by streaming the weights once (K/2 + K/32
// bytes per output channel); the activations are a few hundred KiB.
//
// GEMM part.  A workgroup owns one block of 32 output channels at a time; its four
// waves split K into four contiguous ranges (a wave's W fragments are then one
// contiguous run of the fragment-order layout), accumulate 32 x 32 (x 2 for
// 33..64 tokens) partial tiles on the scaled 32x32x64 MFMA, and reduce the four
// partials through LDS in a fixed order.  The W fragment is the first MFMA
// operand, so a lane's accumulator quad is four consecutive output channels of one
// token.  Latency is hidden by the workgroups a CU holds and by a short ring of K tiles
// per wave (gemm_skinny_kernel); the fused form takes 4 K tiles (2 for 33..64 tokens) at a time.
//
// Fused form.  Phase 1: the (token tile, 4 blocks) units of the activation
// quantizer are dealt out one per wave over the grid and write Xq/Xs (fragment
// order) to the workspace.  A grid-wide barrier separates it from phase 2, the
// GEMM above.  Each workgroup issues the loads of its first W tile before phase 1,
// so the weight stream is already in flight while the activations are quantized.
//
// The barrier uses no read-modify-write atomics: device-scope atomics on one
// address complete at roughly one per 100 ns on this part (measured: a counter
// barrier cost 0.1-0.17 us per workgroup), far more than the rest of the kernel.
// Instead every workgroup publishes "arrived" with one store of this launch's
// generation number to its own slot; one wave of workgroup 0 polls the slot array
// with coalesced device-scope loads until all slots carry that number and then
// stores it into the generation word, which is what the other workgroups poll (and
// what the next launch reads to form its own number).  Variants measured and
// dropped: one release slot per workgroup, and every workgroup polling the slot
// array itself -- both slower.  Device-scope release/acquire fences bracket the
// stores and loads.  From the last arrival to the last workgroup leaving the
// barrier takes 3-5 us: each hop is a trip to the memory side of the fabric.
// The barrier needs all workgroups resident: the grid is capped at one workgroup
// per CU, and every wait is bounded -- on expiry the workgroup records an error
// and exits without touching Y.
#include "skinny_reduce.hpp"
#include "transform_quant_core.hpp"
#include "wush_kernels.hpp"

namespace wush {

namespace {

using skinny::kWaves;
using skinny::reduce_store_block;
using skinny::wave_k_range;
constexpr uint32_t kSpinLimit = 1u << 21;   // polls of about 0.5 us each
constexpr int kMaxGrid = 1024;              // barrier slots in the workspace

// Barrier words in the workspace (uint32 index): generation of the last completed
// launch, error flag (each on its own 128-byte line), arrival slots (dense).
constexpr int kGenWord = 0, kErrWord = 32, kArriveWord = 64;
constexpr int kStateWords = kArriveWord + kMaxGrid;

struct FragTile {   // one (row block, K tile) of a fragment-order operand
  v4i f[4];
  int s;
};

__device__ __forceinline__ void load_frag_tile(FragTile& t, const uint8_t* __restrict__ q,
                                               const uint8_t* __restrict__ s, int64_t rb_kt, int lane) {
  const v4i* p = reinterpret_cast<const v4i*>(q + rb_kt * 4096) + lane;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) t.f[kk] = p[kk * 64];
  t.s = reinterpret_cast<const int*>(s + rb_kt * 256)[lane];
}

// K tiles a wave keeps in flight at once (its loads are issued together, then
// consumed): 4 for up to 32 tokens, 2 beyond (the X registers grow with the token blocks).
template <int RB>
struct Depth { static constexpr int U = RB == 1 ? 4 : 2; };

template <int U>
__device__ __forceinline__ void load_w_chunk(FragTile (&w)[U], const uint8_t* __restrict__ Wq,
                                             const uint8_t* __restrict__ Ws, int64_t j_kt, int n, int lane) {
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < n) load_frag_tile(w[u], Wq, Ws, j_kt + u, lane);
}

// Partial tile of column block j over K tiles [kt0, kt1), U tiles at a time.  `w`
// already holds the W tiles of the first chunk (loaded by the caller, possibly
// long ago).
template <int RB>
__device__ __forceinline__ void accumulate_block(v16f (&acc)[RB], FragTile (&w)[Depth<RB>::U],
                                                 const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs,
                                                 const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ Ws,
                                                 int KT, int j, int kt0, int kt1, int lane) {
  constexpr int U = Depth<RB>::U;
  for (int kt = kt0; kt < kt1; kt += U) {
    const int n = min(U, kt1 - kt);
    if (kt != kt0) load_w_chunk<U>(w, Wq, Ws, (int64_t)j * KT + kt, n, lane);
    FragTile x[RB][U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < n) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) load_frag_tile(x[rb][u], Xq, Xs, (int64_t)rb * KT + kt + u, lane);
      }
#define WUSH_SKINNY_ISSUE(KK)                                                                                        \
  {                                                                                                                  \
    const v8i A_ = {w[u].f[KK][0], w[u].f[KK][1], w[u].f[KK][2], w[u].f[KK][3], 0, 0, 0, 0};                         \
    _Pragma("unroll") for (int rb = 0; rb < RB; ++rb) {                                                              \
      const v8i B_ = {x[rb][u].f[KK][0], x[rb][u].f[KK][1], x[rb][u].f[KK][2], x[rb][u].f[KK][3], 0, 0, 0, 0};       \
      acc[rb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A_, B_, acc[rb], 4, 4, KK, w[u].s, KK, x[rb][u].s);  \
    }                                                                                                                \
  }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < n) {
        WUSH_SKINNY_ISSUE(0)
        WUSH_SKINNY_ISSUE(1)
        WUSH_SKINNY_ISSUE(2)
        WUSH_SKINNY_ISSUE(3)
      }
#undef WUSH_SKINNY_ISSUE
  }
}

// The GEMM: workgroup (j, y) takes output channels 32 j ... + 31 of row blocks RB y ... + RB - 1 of the tokens.  A wavefront has R K tiles in flight
// at any time, each slot refilled as soon as it has been multiplied (skinny::ring); in chunks, all of whose loads were awaited before the first product
// (four tiles, two for more row blocks), nothing covered the gap between a chunk's last product and the next one's data, with a compute unit's
// one workgroup least of all.  Replayed graphs, four sets of operands, us, chunks | ring: 64 x 14336 -> 4096 10.1 | 8.3, 100 x 14336 -> 4096 12.2 | 10.7,
// 32 x 8192 -> 8192 9.1 | 7.5, 256 x 4096 -> 4096 8.8 | 7.7, 1024 x 4096 -> 1024 9.4 | 8.2, 448 x 28672 -> 512 13.8 | 12.9; several workgroups per
// unit 32 x 8192 -> 57344 50.0 | 48.2, 24 x 4096 -> 28672 13.5 | 12.4, 32 x 512 -> 57344 8.9 | 6.0, 48 x 4096 -> 12288 9.5 | 8.1, 100 x 28672 -> 9000
// 70.8 | 71.0.  Tiles in flight: one row block four, two up to K = 2048, where a wavefront's range is no longer than that (geomeans of four against two
// there: 1.01 to 1.02 with one workgroup per unit, 1.03 to 1.25 with several); two row blocks two, one up to K = 1024, or 4096 where there are several
// workgroups per unit (two against one: K = 1024 to 4096 0.95 with one workgroup per unit, 1.02 with several); four row blocks two, held to 256
// registers (against one: 0.95 with one workgroup per unit, 0.95 to 1.02 with several; left to itself the compiler takes 268, and with one workgroup
// per unit instead of two it is 1.1 to 1.4).  More registers for deeper rings cost resident workgroups, and one alone is bound by
// what a compute unit gets out of the L2 and beyond, some 80 GB/s.
template <int RB, int R, bool OUT_F32>
__device__ __forceinline__ void gemm_skinny_ring(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  __shared__ v4f red[kWaves][RB][4][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KT = K >> 8, NB = (N + 31) >> 5, j = blockIdx.x + gridDim.x * blockIdx.z;
  if (j >= NB) return;                        // the grid's padding
  const int64_t row_block = (int64_t)RB * blockIdx.y;
  Xq += row_block * KT * 4096;
  Xs += row_block * KT * 256;
  Wq += (int64_t)j * KT * 4096;
  Ws += (int64_t)j * KT * 256;
  Y = static_cast<uint8_t*>(Y) + 32 * row_block * ldy * (OUT_F32 ? 4 : 2);
  M -= 32 * (int)row_block;
  int kt, kt1;
  wave_k_range(KT, wave, kt, kt1);
  v16f acc[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) acc[rb] = (v16f){0};
  FragTile w[R], x[R][RB];
  auto load = [&](int u, int t) {
    load_frag_tile(w[u], Wq, Ws, t, lane);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) load_frag_tile(x[u][rb], Xq, Xs, (int64_t)rb * KT + t, lane);
  };
  auto multiply = [&](int u) {
#define WUSH_RING_ISSUE(KK)                                                                                          \
  {                                                                                                                  \
    const v8i A_ = {w[u].f[KK][0], w[u].f[KK][1], w[u].f[KK][2], w[u].f[KK][3], 0, 0, 0, 0};                         \
    _Pragma("unroll") for (int rb = 0; rb < RB; ++rb) {                                                              \
      const v8i B_ = {x[u][rb].f[KK][0], x[u][rb].f[KK][1], x[u][rb].f[KK][2], x[u][rb].f[KK][3], 0, 0, 0, 0};       \
      acc[rb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A_, B_, acc[rb], 4, 4, KK, w[u].s, KK, x[u][rb].s);  \
    }                                                                                                                \
  }
    WUSH_RING_ISSUE(0)
    WUSH_RING_ISSUE(1)
    WUSH_RING_ISSUE(2)
    WUSH_RING_ISSUE(3)
#undef WUSH_RING_ISSUE
  };
  skinny::ring<R>(kt, kt1, load, multiply);
  reduce_store_block<RB, OUT_F32>(acc, red, j, M, N, Y, ldy, lane, wave);
}

template <int RB, bool OUT_F32>
__global__ __launch_bounds__(kWaves * 64, RB == 4 ? 2 : 1) void gemm_skinny_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  gemm_skinny_ring<RB, RB == 1 ? 4 : 2, OUT_F32>(Xq, Xs, Wq, Ws, M, N, K, Y, ldy);
}
template <int RB, bool OUT_F32>   // short K, by the lines above
__global__ __launch_bounds__(kWaves * 64, 1) void gemm_skinny_short_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  gemm_skinny_ring<RB, RB == 1 ? 2 : 1, OUT_F32>(Xq, Xs, Wq, Ws, M, N, K, Y, ldy);
}

// At most 16 tokens, on v_mfma_scale_f32_16x16x128_f8f6f4: half of the activations' fragments and of every product would be a row block's padding.
// Lane quarter q of instruction p takes group kk = 2 p + q / 2 of K half kh = q % 2, for both operands: the fragments as they lie, and with
// the scale dword shifted by q / 2 bytes its scale is byte 2 p in every lane.  HALVES = 16-channel halves of a block of 32 output channels
// a workgroup takes: both, or one where the blocks are so few that halves still find idle compute units.  A ring of R K tiles per wavefront as above:
// two, one up to K = 2048 (geomeans, two against one: up to K = 512 1.01, 1024 1.03 with several workgroups per unit, 2048 0.98 to 1.00; four
// against two: 4096 and more 0.99, halves beyond 8192 0.95, less than that 1.02 to 1.09).  Replayed graphs, four sets of operands, us,
// 32 x 32 fragments in chunks | this: 16 x 8192 -> 57344 48.9 | 44.4 (250 MB of weights: 5.6 TB/s), 16 x 4096 -> 28672 13.4 | 11.6, 16 x 28672 ->
// 8192 26.5 | 22.4, 1 x 14336 -> 4096 9.6 | 7.0, 1 x 4096 -> 6144 5.3 | 4.3, 9 x 28672 -> 1024 12.6 | 7.8, 16 x 256 -> 57344 7.3 | 3.2.
struct HalfTile {   // 16 rows of one (row block, K tile)
  v4i f[2];
  int s;
};
template <int HALVES, int R, bool OUT_F32>
__global__ __launch_bounds__(kWaves * 64) void gemm_skinny16_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  __shared__ v4f red[kWaves][HALVES][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, q = lane >> 4;
  const int KT = K >> 8, NB = HALVES == 2 ? (N + 31) >> 5 : (N + 15) >> 4;
  const int chunk = ((q >> 1) * 64 + (q & 1) * 32 + l16) * 16, scale = ((q & 1) * 32 + l16) * 4;
  int kt0, kt1;
  wave_k_range(KT, wave, kt0, kt1);
  auto load_half = [&](HalfTile& t, const uint8_t* qp, const uint8_t* sp, int64_t rb_kt, int a) {
    const uint8_t* p = qp + rb_kt * 4096 + chunk + 256 * a;
    t.f[0] = *reinterpret_cast<const v4i*>(p);
    t.f[1] = *reinterpret_cast<const v4i*>(p + 2048);
    t.s = *reinterpret_cast<const int*>(sp + rb_kt * 256 + scale + 64 * a);
  };
  const int j = blockIdx.x + gridDim.x * blockIdx.z;
  if (j >= NB) return;                        // the grid's padding
  const int64_t block = HALVES == 2 ? j : j >> 1;
  const int first = HALVES == 2 ? 0 : j & 1;
  v4f acc[HALVES];
#pragma unroll
  for (int a = 0; a < HALVES; ++a) acc[a] = (v4f){0, 0, 0, 0};
  HalfTile w[R][HALVES], x[R];
  auto load = [&](int u, int kt) {
#pragma unroll
    for (int a = 0; a < HALVES; ++a) load_half(w[u][a], Wq, Ws, block * KT + kt, first + a);
    load_half(x[u], Xq, Xs, kt, 0);
  };
  auto multiply = [&](int u) {
    const int sx = x[u].s >> (8 * (q >> 1));
#pragma unroll
    for (int a = 0; a < HALVES; ++a) {
      const int sw = w[u][a].s >> (8 * (q >> 1));
#define WUSH_HALF_ISSUE(P)                                                                                                    \
  {                                                                                                                         \
    const v8i A_ = {w[u][a].f[P][0], w[u][a].f[P][1], w[u][a].f[P][2], w[u][a].f[P][3], 0, 0, 0, 0};                        \
    const v8i B_ = {x[u].f[P][0], x[u].f[P][1], x[u].f[P][2], x[u].f[P][3], 0, 0, 0, 0};                                    \
    acc[a] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A_, B_, acc[a], 4, 4, 2 * P, sw, 2 * P, sx);                  \
  }
      WUSH_HALF_ISSUE(0)
      WUSH_HALF_ISSUE(1)
#undef WUSH_HALF_ISSUE
    }
  };
  skinny::ring<R>(kt0, kt1, load, multiply);
  // the waves' sums in their order; accumulator v of lane (l16, q) is token l16, output channel 4 q + v of the half
#pragma unroll
  for (int a = 0; a < HALVES; ++a) red[wave][a][lane] = acc[a];
  __syncthreads();
  if (wave < HALVES) {
    const v4f sum = ((red[0][wave][lane] + red[1][wave][lane]) + red[2][wave][lane]) + red[3][wave][lane];
    const int col = HALVES == 2 ? 32 * j + 16 * wave + 4 * q : 16 * j + 4 * q;
    const float v[4] = {sum[0], sum[1], sum[2], sum[3]};
    if (l16 < M && col < N) skinny::store_quad<OUT_F32>(Y, ldy, l16, col, N, col + 4 <= N, v);
  }
}

template <int RB, bool OUT_F32>
__global__ __launch_bounds__(kWaves * 64) void layer_decode_kernel(
    const uint16_t* __restrict__ X, int64_t ldx, const uint16_t* __restrict__ T, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, uint8_t* __restrict__ Xq, uint8_t* __restrict__ Xs, uint32_t* __restrict__ state,
    int M, int N, int K, void* __restrict__ Y, int64_t ldy, int rule, uint32_t expected_blocks,
    uint32_t spin_limit) {
  __shared__ v4f red[kWaves][RB][4][64];
  __shared__ int barrier_ok;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int KT = K >> 8, C = K >> 5, NB = (N + 31) >> 5;
  int kt0, kt1;
  wave_k_range(KT, wave, kt0, kt1);

  // This launch's generation: one more than the last completed launch's, which
  // workgroup 0 only advances after every workgroup has arrived (and so has read it).
  const uint32_t target = state[kGenWord] + 1;

  // Start the weight stream: first W chunk of this workgroup's first column block.
  // Waves with a phase-1 unit issue it after that unit's loads, which the barrier waits for.
  constexpr int U = Depth<RB>::U;
  int j = blockIdx.x;
  FragTile w_first[U];
  const int n_first = min(U, kt1 - kt0);
  const bool has_unit = (int)(blockIdx.x + wave * gridDim.x) < RB * (C >> 2);
  if (!has_unit && j < NB && kt0 < kt1) load_w_chunk<U>(w_first, Wq, Ws, (int64_t)j * KT + kt0, n_first, lane);

  // ---- phase 1: quantize the activations, one (token tile, 4 blocks) unit per wave
  {
    const int tok = lane & 31, h = lane >> 5;
    const int units = RB * (C >> 2);
    for (int u = blockIdx.x + wave * gridDim.x; u < units; u += kWaves * gridDim.x) {
      const int t = u % RB, bfirst = 4 * (u / RB);
      v8bf ta[tq::kNB][2];
      tq::XFrag cur[tq::kNB];
      tq::load_transforms(ta, T, bfirst, C, tok, h);
      tq::load_tile(cur, X, ldx, min(32 * t + tok, M - 1), bfirst, C, h);
      if (u == (int)(blockIdx.x + wave * gridDim.x) && j < NB && kt0 < kt1)
        load_w_chunk<U>(w_first, Wq, Ws, (int64_t)j * KT + kt0, n_first, lane);
      v4u out[2];
      uint32_t sbytes;
      tq::transform_quantize<false>(ta, cur, rule, out, sbytes, nullptr, tq::kNB);
      if (32 * t + tok < M) tq::store_tile_tiled<false>(out, sbytes, Xq, Xs, t, KT, bfirst, tok, h);
    }
  }

  // ---- grid-wide barrier.  Device-scope fences cost about 0.1 us each and
  // serialize within an XCD (they walk its L2), so there is one release per
  // workgroup that wrote activations and one acquire per workgroup, both issued by
  // wave 0 with the workgroup barrier extending them to the other waves.
  __syncthreads();
  if (wave == 0) {
    bool ok = true;
    if ((int)blockIdx.x < RB * (C >> 2)) __threadfence();   // release this workgroup's Xq/Xs stores
    if (lane == 0)
      __hip_atomic_store(&state[kArriveWord + blockIdx.x], target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (blockIdx.x == 0) {
      // collector: poll all arrival slots, 64 per load instruction
      uint32_t spins = 0;
      for (;;) {
        bool all = true;
        for (uint32_t i = lane; i < expected_blocks; i += 64)
          all &= __hip_atomic_load(&state[kArriveWord + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == target;
        if (__builtin_amdgcn_ballot_w64(all) == ~0ull) break;
        if (++spins >= spin_limit) { ok = false; break; }
        __builtin_amdgcn_s_sleep(4);
      }
      // every workgroup has arrived, hence has read the old generation: publish the new one
      if (ok) {
        __threadfence();
        if (lane == 0) __hip_atomic_store(&state[kGenWord], target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    } else {
      uint32_t spins = 0;
      while (__hip_atomic_load(&state[kGenWord], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != target) {
        if (++spins >= spin_limit) { ok = false; break; }
        __builtin_amdgcn_s_sleep(8);
      }
    }
    if (ok) __threadfence();   // acquire: see every workgroup's Xq/Xs
    if (lane == 0) {
      if (!ok) __hip_atomic_store(&state[kErrWord], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      barrier_ok = ok;
    }
  }
  __syncthreads();
  if (!barrier_ok) return;   // workgroup-uniform

  // ---- phase 2: GEMM over this workgroup's column blocks
  for (; j < NB; j += gridDim.x) {
    v16f acc[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[rb] = (v16f){0};
    if (kt0 < kt1) {
      if (j != (int)blockIdx.x) load_w_chunk<U>(w_first, Wq, Ws, (int64_t)j * KT + kt0, n_first, lane);
      accumulate_block<RB>(acc, w_first, Xq, Xs, Wq, Ws, KT, j, kt0, kt1, lane);
    }
    reduce_store_block<RB, OUT_F32>(acc, red, j, M, N, Y, ldy, lane, wave);
  }
}

__global__ void decode_state_reset_kernel(uint32_t* state) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kStateWords; i += gridDim.x * blockDim.x) state[i] = 0;
}

// Workgroups that are certainly resident together: one per CU, given that the
// occupancy the runtime reports for the kernel is at least that.
template <typename Kern>
hipError_t resident_limit(Kern kern, int* limit) {
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kWaves * 64, 0);
  if (e != hipSuccess) return e;
  if (per_cu < 1 || cus < 1) return hipErrorInvalidValue;
  // One workgroup per CU: measured faster than two for every shape (half the
  // arrivals and fences at the barrier; the GEMM phase keeps 4 x U tiles in flight per CU).
  *limit = cus;
  if (*limit > kMaxGrid - 1) *limit = kMaxGrid - 1;   // one slot is left for the timeout test hook
  return hipSuccess;
}

}  // namespace

// Row blocks of 32 tokens a workgroup takes.  A workgroup reads all of its tokens' activations for every 32 output
// channels, so beyond 32 tokens it is bound by that traffic into its compute unit: while the layer has too few blocks of
// output channels for all of them, the tokens are dealt out as well, as finely as one workgroup per compute unit allows
// (us, all tokens in one workgroup | two groups | one group per 32 tokens: 100 x 14336 -> 4096 14.9 | 10.2 | 12.7;
// 64 x 14336 -> 4096 10.1 | - | 7.9; 128 x 4096 -> 4096 6.8 | 5.1 | 5.4; 100 x 8192 -> 1024 8.2 | 5.5 | 4.2; with more
// groups than compute units the weights' second trip costs more than it saves: 128 x 28672 -> 8192 40.6 | 46.1 | 70.9).
// Eight waves per workgroup instead of four (deeper split of K) gave nothing.
int skinny_row_blocks(int64_t M, int64_t N) {
  const int64_t blocks = (N + 31) / 32, tokens = (M + 31) / 32, cus = device_cu_count();
  if (M <= 32 || blocks * tokens <= cus) return 1;
  if (M <= 64 || blocks * ((tokens + 1) / 2) <= cus) return 2;
  return 4;
}

// Workgroups side by side where they take four row blocks each: a multiple of 8, the last few finding no block.  Workgroups go round the 8
// XCDs, so the row groups of a block of output channels, one grid row after the other, then run on one XCD and read its weights into one
// L2 (us, tiles | as many workgroups as blocks | this: 512 x 1024 -> 1984 4.65 | 4.22 | 4.18, 384 x 1536 -> 1984 5.37 | 4.60 | 4.58; before the ring, with
// less in flight, 4.89 | 5.86 | 4.76 and 5.59 | 6.27 | 5.48).
int64_t skinny_grid_width(int64_t N) { return ((N + 31) / 32 + 7) & ~(int64_t)7; }

hipError_t launch_mxfp4_gemm_skinny(const void* Xq, const void* Xs, const void* Wq, const void* Ws, int64_t M,
                                    int64_t N, int64_t K, int out_f32, void* Y, int64_t ldy, hipStream_t stream) {
  const int NB = (int)((N + 31) / 32);
  if (M <= 16) {
    const int cus = device_cu_count();
    const bool halves = 2 * NB <= cus;
    const int64_t blocks = halves ? (N + 15) / 16 : NB;
    const bool shallow = K <= 2048;   // a wavefront's range is one or two tiles
    auto kernel = halves ? (out_f32 ? (shallow ? gemm_skinny16_kernel<1, 1, true> : gemm_skinny16_kernel<1, 2, true>)
                                    : (shallow ? gemm_skinny16_kernel<1, 1, false> : gemm_skinny16_kernel<1, 2, false>))
                         : (out_f32 ? (shallow ? gemm_skinny16_kernel<2, 1, true> : gemm_skinny16_kernel<2, 2, true>)
                                    : (shallow ? gemm_skinny16_kernel<2, 1, false> : gemm_skinny16_kernel<2, 2, false>));
    kernel<<<skinny::wide_grid(blocks, 1), dim3(kWaves * 64), 0, stream>>>(
        (const uint8_t*)Xq, (const uint8_t*)Xs, (const uint8_t*)Wq, (const uint8_t*)Ws, (int)M, (int)N, (int)K, Y, ldy);
    return hipGetLastError();
  }
  const int rb = skinny_row_blocks(M, N), groups = (int)((M + 32 * rb - 1) / (32 * rb));
  const int64_t wide = rb == 4 && groups > 1 ? skinny_grid_width(N) : NB;
#define WUSH_SKINNY(KERNEL, RB) (out_f32 ? KERNEL<RB, true> : KERNEL<RB, false>)
  auto kernel = rb == 1 ? (K <= 2048 ? WUSH_SKINNY(gemm_skinny_short_kernel, 1) : WUSH_SKINNY(gemm_skinny_kernel, 1))
              : rb == 2 ? (K <= 1024 || (K <= 4096 && (int64_t)groups * NB > device_cu_count()) ? WUSH_SKINNY(gemm_skinny_short_kernel, 2) : WUSH_SKINNY(gemm_skinny_kernel, 2))
                        : WUSH_SKINNY(gemm_skinny_kernel, 4);
#undef WUSH_SKINNY
  kernel<<<skinny::wide_grid(wide, groups), dim3(kWaves * 64), 0, stream>>>((const uint8_t*)Xq, (const uint8_t*)Xs, (const uint8_t*)Wq,
                                                                            (const uint8_t*)Ws, (int)M, (int)N, (int)K, Y, ldy);
  return hipGetLastError();
}

// workspace: Xq for 64 tokens (2 row blocks) | Xs | barrier words
size_t layer_decode_codes_bytes(int64_t K) { return (size_t)(K >> 8) * 2 * 4096; }
size_t layer_decode_scales_bytes(int64_t K) { return (size_t)(K >> 8) * 2 * 256; }
size_t layer_decode_scales_offset(int64_t K) { return layer_decode_codes_bytes(K); }
size_t layer_decode_state_offset(int64_t K) { return layer_decode_codes_bytes(K) + layer_decode_scales_bytes(K); }
size_t layer_decode_workspace_bytes(int64_t K) { return layer_decode_state_offset(K) + (size_t)kStateWords * 4; }
size_t layer_decode_error_offset(int64_t K) { return layer_decode_state_offset(K) + (size_t)kErrWord * 4; }

hipError_t launch_layer_decode_init(void* workspace, int64_t K, hipStream_t stream) {
  uint32_t* state = reinterpret_cast<uint32_t*>(static_cast<uint8_t*>(workspace) + layer_decode_state_offset(K));
  decode_state_reset_kernel<<<32, 256, 0, stream>>>(state);
  return hipGetLastError();
}

hipError_t launch_layer_decode(const void* X, int64_t M, int64_t K, int64_t ldx, const void* T, const void* Wq,
                               const void* Ws, int64_t N, int rule, int out_f32, void* Y, int64_t ldy,
                               void* workspace, int test_timeout, hipStream_t stream) {
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  uint8_t* Xq = ws;
  uint8_t* Xs = ws + layer_decode_codes_bytes(K);
  uint32_t* state = reinterpret_cast<uint32_t*>(ws + layer_decode_state_offset(K));
  const int NB = (int)((N + 31) / 32);
  dim3 block(kWaves * 64);
#define WUSH_DECODE_LAUNCH(RB, F32)                                                                          \
  {                                                                                                          \
    static int limit = 0; /* queried once per instantiation */                                               \
    if (limit == 0) {                                                                                        \
      int l = 0;                                                                                             \
      hipError_t e = resident_limit(layer_decode_kernel<RB, F32>, &l);                                       \
      if (e != hipSuccess) return e;                                                                         \
      limit = l;                                                                                             \
    }                                                                                                        \
    const unsigned g = (unsigned)(NB < limit ? NB : limit);                                                  \
    /* test hook: expect one workgroup more than launched and give up after a few polls */                   \
    const uint32_t expected = test_timeout ? g + 1 : g;                                                      \
    const uint32_t spin = test_timeout ? 16u : kSpinLimit;                                                   \
    layer_decode_kernel<RB, F32><<<dim3(g), block, 0, stream>>>(                                             \
        (const uint16_t*)X, ldx, (const uint16_t*)T, (const uint8_t*)Wq, (const uint8_t*)Ws, Xq, Xs, state,  \
        (int)M, (int)N, (int)K, Y, ldy, rule, expected, spin);                                          \
  }
  if (M <= 32) {
    if (out_f32) WUSH_DECODE_LAUNCH(1, true) else WUSH_DECODE_LAUNCH(1, false)
  } else {
    if (out_f32) WUSH_DECODE_LAUNCH(2, true) else WUSH_DECODE_LAUNCH(2, false)
  }
#undef WUSH_DECODE_LAUNCH
  return hipGetLastError();
}

}  // namespace wush
