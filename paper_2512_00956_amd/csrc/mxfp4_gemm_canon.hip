// MXFP4 GEMM on operands in the canonical (row-major) layout, any M, N and K % 32 == 0:
// Y = deq(Xq,Xs) . deq(Wq,Ws)^T on v_mfma_scale_f32_32x32x64_f8f6f4.
//
// A workgroup of four wavefronts (WM x WN) computes a tile of 32 WM RB x 32 WN CB outputs; K advances 256 elements (128
// bytes of a row) per step.  With one wavefront per SIMD nothing but the software pipeline hides latency:
//   * Both operand tiles go global -> LDS directly (no registers in flight) into a ring of ST steps, ST - 1 ahead.  An
//     instruction moves 8 rows x 128 bytes -- whole cache lines: with 64 bytes of 16 rows a line was fetched for each of
//     its halves, the 64 KiB of a 256 x 256 tile's step being more than the L1 holds (2.3 times the L2 requests, 145 against
//     116 us on 4096 x 14336 -> 4096).  The LDS side of such a load is lane-linear, so the swizzle that makes the fragment
//     reads conflict free (chunk p of row q holds source chunk p ^ (q >> 1) & 7) is applied to each lane's source address.
//   * One barrier per step: it publishes step kt and frees the slot read in step kt - 1, which is refilled, one load per
//     MFMA, during the first of the step's four issues.
//   * Issue kk (0..3) of lane half kh contracts group 4 kh + kk of the step's eight; which 64 elements an MFMA takes is
//     free as long as both operands agree.  Its fragments are read during the issue before.
//   * Scale rows are K / 32 bytes at any alignment.  Read where an MFMA needs them, they were as many cache-line lookups
//     as the operands; instead each thread fetches the 16 bytes of one row's next two steps at a time and leaves them
//     in LDS, where a lane picks its dword per step (its bytes are the four issues').  What is left of a row at its end comes
//     as its last 16 bytes, shifted into place on the way to LDS (byte by byte it cost 777 x 1376 -> 3001 1.8 us of 11.6).
// The direct loads are issued from inline asm (and the barrier's fences name LDS only) for the reason given in
// mxfp4_gemm_frag.hip: the compiler would drain them at every LDS read.  They have no register destination; their
// arrival is the explicit vmcnt's business.  The scale loads are ordinary ones; the compiler's wait for them, one in two
// steps, drains the ring's loads as well.
// 4096 x 14336 -> 4096: 116 us = 4.1 PFLOP/s (189 for the kernel of two 64 KiB stages it replaces, whose loads were drained
// at every LDS read; 98 in the tiled layout, whose fragments are contiguous).
#include <math.h>

#include <type_traits>
#include <utility>

#include "row_store.hpp"
#include "wush_device.hpp"
#include "wush_kernels.hpp"

namespace wush {

namespace {

constexpr int kStepB = 128;          // bytes of a row per step: 256 elements
typedef unsigned int v4u_unaligned __attribute__((ext_vector_type(4), aligned(1)));

constexpr int vmcnt_imm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0F70; }
constexpr int kLgkm0 = 0xC07F;       // s_waitcnt lgkmcnt(0)

template <int... m, class Fn>
__device__ __forceinline__ void for_each(std::integer_sequence<int, m...>, Fn fn) {
  (fn(std::integral_constant<int, m>{}), ...);
}

template <int WM, int WN, int RB, int CB, int ST>
struct Shape {
  static constexpr int kTM = 32 * WM * RB, kTN = 32 * WN * CB, kRows = kTM + kTN;
  static constexpr int kSlotB = kRows * kStepB;
  static constexpr int kScaleBase = ST * kSlotB, kScaleB = kRows * 16;         // 16 scale bytes per row, two buffers
  static constexpr int kLds = kScaleBase + 2 * kScaleB;
  static constexpr int kDma = kRows / 32;                                      // direct loads per wavefront and step
  static constexpr int kScaleRows = (kRows + 255) / 256;                       // scale rows per thread
};

template <bool OUT_F32, bool RAGGED, int WM, int WN, int RB, int CB, int ST>
__global__ __launch_bounds__(256) void gemm_canon_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, int M, int N, int K, void* __restrict__ Y, int64_t ldy, int tiles_m, int tiles_n) {
  using S = Shape<WM, WN, RB, CB, ST>;
  static_assert(WM * WN == 4 && S::kTM % 32 == 0 && ST >= 2, "four wavefronts, whole 8-row loads");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int r = lane & 31, kh = lane >> 5;

  // Workgroup -> tile as in mxfp4_gemm_frag.hip: a contiguous id range per XCD, walked in bands of 8 tile rows.
  const int id = xcd_contiguous_id(blockIdx.x, tiles_m * tiles_n);
  constexpr int kBand = 8;
  const int width = kBand * tiles_n, first_m = id / width * kBand;
  const int band_rows = min(tiles_m - first_m, kBand);
  const int tm = first_m + (id % width) % band_rows, tn = (id % width) / band_rows;
  const int m0 = tm * S::kTM, n0 = tn * S::kTN;

  const int C = K >> 5;                       // groups of a row
  const int64_t KB = K >> 1;
  const int KT = (C + 7) >> 3;                // steps
  const int rem = RAGGED ? C - 8 * (KT - 1) : 8;   // groups of the last one

  // ---- direct loads: instruction u of the workgroup moves rows 8 u ... + 7 of [X tile; W tile]; a wavefront issues
  // kDma of them.  Rows past M or N repeat the last one (they feed outputs that are never stored).
  const uint8_t* x_tile = Xq + (int64_t)m0 * KB;
  const uint8_t* w_tile = Wq + (int64_t)n0 * KB;
  uint32_t off[S::kDma];
  auto chunk_of = [&](int u) { return (lane & 7) ^ (((u & 1) << 2) | (lane >> 4)); };   // (row >> 1) & 7 of row 8 u + lane / 8
#pragma unroll
  for (int j = 0; j < S::kDma; ++j) {
    const int u = wave * S::kDma + j, row = 8 * u + (lane >> 3);
    const int local = row < S::kTM ? min(row, M - 1 - m0) : min(row - S::kTM, N - 1 - n0);
    off[j] = (uint32_t)(local * KB + 16 * chunk_of(u));
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)smem;
  auto dma = [&](int kt, int slot_off, int j) {
    const int u = wave * S::kDma + j;         // wave-uniform
    const uint8_t* src = (8 * u < S::kTM ? x_tile : w_tile) + (int64_t)kt * kStepB;
    const uint32_t dst = lds_base + slot_off + 1024 * u;
    uint32_t o = off[j];
    if (RAGGED && kt == KT - 1) {
      // in a partial last step the chunks past the row's end fetch its last one; their products are masked out
      const int chunk = chunk_of(u);
      o -= 16u * (uint32_t)(chunk - min(chunk, rem - 1));
    }
    // the wait state a load to LDS needs behind the write of m0; m0 itself: see mxfp4_gemm_frag.hip
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(o), "s"(src), "s"(dst));
  };

  // ---- scales: rows threadIdx.x + 256 i of [X tile; W tile], 16 bytes (two steps) at a time
  // The pointers advance in place: an address put together for a load could land in the registers of the load before, which the
  // compiler then waits for, draining the ring.
  v4u scale_next[S::kScaleRows];
  typedef const __attribute__((address_space(1))) uint8_t* global_bytes;   // the asm below would make a plain pointer a flat one
  typedef const __attribute__((address_space(1))) v4u_unaligned* global_scales;
  global_bytes scale_at[S::kScaleRows];
#pragma unroll
  for (int i = 0; i < S::kScaleRows; ++i) {
    const int row = min((int)threadIdx.x + 256 * i, S::kRows - 1);
    const bool x = row < S::kTM;
    scale_at[i] = (global_bytes)(x ? Xs : Ws) + (int64_t)(x ? min(m0 + row, M - 1) : min(n0 + row - S::kTM, N - 1)) * C;
  }
  auto fetch_first_scales = [&]() {
#pragma unroll
    for (int i = 0; i < S::kScaleRows; ++i) {
      if (C >= 16) {                          // the same in every thread
        scale_next[i] = *(global_scales)scale_at[i];
      } else {
        v4u v = {0x7F7F7F7Fu, 0x7F7F7F7Fu, 0x7F7F7F7Fu, 0x7F7F7F7Fu};
        const int bytes = RAGGED ? 16 : 8;
#pragma unroll
        for (int b = 0; b < bytes; ++b)
          if (b < C) v[b >> 2] = (v[b >> 2] & ~(0xFFu << (8 * (b & 3)))) | (uint32_t)scale_at[i][b] << (8 * (b & 3));
        scale_next[i] = v;
      }
    }
  };
  auto fetch_scales = [&](int pair) {         // pair >= 1: the row has more than 16 groups
    const int step = min(16, C - 16 * pair);  // past the row's end: its last 16 bytes instead, shifted into place by leave_scales
#pragma unroll
    for (int i = 0; i < S::kScaleRows; ++i) {
      scale_at[i] += step;
      asm volatile("" : "+v"(scale_at[i]));
      if (threadIdx.x + 256 * i < S::kRows) scale_next[i] = *(global_scales)scale_at[i];
    }
  };
  auto leave_scales = [&](int pair) {
    int past = C >= 16 ? max(16 * pair + 16 - C, 0) : 0;   // bytes past the row's end: 0 .. 15 (8 groups: whole steps), the same in every thread
#pragma unroll
    for (int i = 0; i < S::kScaleRows; ++i) {
      const int row = threadIdx.x + 256 * i;
      v4u v = scale_next[i];
      if (past > 0) {
        asm volatile("" : "+s"(past));        // a branch, not selects in every step
        if (past & 8) v = (v4u){v[2], v[3], 0, 0};
        if (past & 4) v = (v4u){v[1], v[2], v[3], 0};
        v = (v4u){__builtin_amdgcn_alignbyte(v[1], v[0], past & 3), __builtin_amdgcn_alignbyte(v[2], v[1], past & 3),
                  __builtin_amdgcn_alignbyte(v[3], v[2], past & 3), __builtin_amdgcn_alignbyte(0, v[3], past & 3)};
      }
      if (row < S::kRows) *reinterpret_cast<v4u*>(smem + S::kScaleBase + (pair & 1) * S::kScaleB + 16 * row) = v;
    }
  };

  // ---- fragment and scale reads
  const int x_row = wm * RB * 32 + r, w_row = S::kTM + wn * CB * 32 + r;
  int pos[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) pos[kk] = 16 * ((4 * kh + kk) ^ ((r >> 1) & 7));
  auto read_x = [&](int slot_off, int kk, int i, bool last) {
    v4i f = *reinterpret_cast<const v4i*>(smem + slot_off + (x_row + 32 * i) * kStepB + pos[kk]);
    if (RAGGED && last && 4 * kh + kk >= rem) f = (v4i){0, 0, 0, 0};   // groups past the row's end
    return f;
  };
  auto read_w = [&](int slot_off, int kk, int j) {
    return *reinterpret_cast<const v4i*>(smem + slot_off + (w_row + 32 * j) * kStepB + pos[kk]);
  };
  auto read_scale = [&](int kt, int row) {
    return *reinterpret_cast<const int*>(smem + S::kScaleBase + ((kt >> 1) & 1) * S::kScaleB + 16 * row + 8 * (kt & 1) + 4 * kh);
  };

  v16f acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = (v16f){0};

#define WUSH_FENCE __builtin_amdgcn_sched_barrier(0);
  // ---- prologue: ST - 1 steps on their way
  fetch_first_scales();
  leave_scales(0);
  WUSH_FENCE
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < KT)
#pragma unroll
      for (int j = 0; j < S::kDma; ++j) dma(t, t * S::kSlotB, j);

  // One step.  REFILL: step kt + ST - 1 exists (its direct loads are issued here); MORE: step kt + 1 exists.
  int slot_off = 0;
  auto step = [&](int kt, auto refill_tag, auto more_tag) {
    constexpr bool REFILL = decltype(refill_tag)::value, MORE = decltype(more_tag)::value;
    // scales of the next two steps: requested in the first step of this pair, left in LDS before the second
    if (MORE && (kt & 1)) leave_scales((kt >> 1) + 1);
    // outstanding behind step kt's loads: those of the steps up to kt + ST - 2
    if (REFILL) __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 2) * S::kDma));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_waitcnt(kLgkm0);
    WUSH_FENCE
    lds_barrier();
    WUSH_FENCE
    asm volatile("" : "+s"(slot_off));        // LDS changes behind the compiler's back: no address may look like an old one
    int refill_off = slot_off - S::kSlotB;    // slot of step kt - 1 = of step kt + ST - 1
    refill_off = refill_off < 0 ? (ST - 1) * S::kSlotB : refill_off;
    v4i xf[2][RB], wf[2][CB];
    int xs[RB], ws[CB];
#pragma unroll
    for (int q = 0; q < (RB > CB ? RB : CB); ++q) {
      if (q < CB) {
        wf[0][q] = read_w(slot_off, 0, q);
        ws[q] = read_scale(kt, w_row + 32 * q);
      }
      if (q < RB) {
        xf[0][q] = read_x(slot_off, 0, q, !MORE);
        xs[q] = read_scale(kt, x_row + 32 * q);
      }
    }
    if (MORE && !(kt & 1) && kt + 2 < KT) fetch_scales((kt >> 1) + 1);
    constexpr int kMma = RB * CB;
    for_each(std::make_integer_sequence<int, 4 * kMma>{}, [&](auto tag) {
      constexpr int kk = decltype(tag)::value / kMma, m = decltype(tag)::value % kMma, i = m / CB, j = m % CB, cur = kk & 1;
      const v8i A = {wf[cur][j][0], wf[cur][j][1], wf[cur][j][2], wf[cur][j][3], 0, 0, 0, 0};
      const v8i B = {xf[cur][i][0], xf[cur][i][1], xf[cur][i][2], xf[cur][i][3], 0, 0, 0, 0};
      acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A, B, acc[i][j], 4, 4, kk, ws[j], kk, xs[i]);
      if constexpr (kk < 3) {
        constexpr int kReads = RB + CB, lo = m * kReads / kMma, hi = (m + 1) * kReads / kMma;
#pragma unroll
        for (int q = lo; q < hi; ++q) {
          if (q < CB) wf[cur ^ 1][q] = read_w(slot_off, kk + 1, q);
          else xf[cur ^ 1][q - CB] = read_x(slot_off, kk + 1, q - CB, !MORE);
        }
      }
      // direct loads: at most one per MFMA, from the step's first MFMA on
      if constexpr (REFILL) {
        constexpr int n = decltype(tag)::value, kPer = S::kDma > 4 * kMma ? (S::kDma + 4 * kMma - 1) / (4 * kMma) : 1;
#pragma unroll
        for (int q = n * kPer; q < (n + 1) * kPer; ++q)
          if (q < S::kDma) dma(kt + ST - 1, refill_off, q);
      }
      WUSH_FENCE
    });
    slot_off = slot_off + S::kSlotB == ST * S::kSlotB ? 0 : slot_off + S::kSlotB;
  };
  int kt = 0;
  for (; kt + ST - 1 < KT; ++kt) step(kt, std::true_type{}, std::true_type{});
  for (; kt + 1 < KT; ++kt) step(kt, std::false_type{}, std::true_type{});
  step(kt, std::false_type{}, std::false_type{});
#undef WUSH_FENCE
  __syncthreads();   // the ring becomes the transpose buffers

  // ---- epilogue (row_store.hpp): each wavefront turns its row blocks in a private buffer
  using Out = RowStore<OUT_F32, CB>;
  static_assert(4 * Out::kBuf <= S::kLds, "transpose buffers");
  uint8_t* buf = smem + wave * Out::kBuf;
  const bool stream = Out::streams(Y, ldy, M, N, K);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    __builtin_amdgcn_sched_barrier(0);
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < CB; ++j) Out::put(buf, acc[i][j], j, lane);
    wave_lds_sync();
    Out::store(buf, Y, ldy, m0 + (wm * RB + i) * 32, n0 + wn * CB * 32, M, N, lane, stream);
  }
}

template <bool OUT_F32, bool RAGGED, int WM, int WN, int RB, int CB, int ST>
hipError_t launch_shape(const void* Xq, const void* Xs, const void* Wq, const void* Ws, int64_t M, int64_t N, int64_t K,
                        void* Y, int64_t ldy, hipStream_t stream) {
  using S = Shape<WM, WN, RB, CB, ST>;
  static DynamicLdsLimit lds_limit;
  auto kernel = gemm_canon_kernel<OUT_F32, RAGGED, WM, WN, RB, CB, ST>;
  const hipError_t attr = lds_limit.ensure(reinterpret_cast<const void*>(kernel), S::kLds);
  if (attr != hipSuccess) return attr;
  const int tiles_m = (int)((M + S::kTM - 1) / S::kTM), tiles_n = (int)((N + S::kTN - 1) / S::kTN);
  kernel<<<dim3((unsigned)((int64_t)tiles_m * tiles_n)), dim3(256), S::kLds, stream>>>(
      (const uint8_t*)Xq, (const uint8_t*)Xs, (const uint8_t*)Wq, (const uint8_t*)Ws, (int)M, (int)N, (int)K, Y, ldy, tiles_m,
      tiles_n);
  return hipGetLastError();
}

template <bool OUT_F32, bool RAGGED>
hipError_t launch_any(int shape, const void* Xq, const void* Xs, const void* Wq, const void* Ws, int64_t M, int64_t N, int64_t K,
                      void* Y, int64_t ldy, hipStream_t stream) {
  switch (shape) {
    case 0: return launch_shape<OUT_F32, RAGGED, 2, 2, 4, 4, 2>(Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream);
    case 1: return launch_shape<OUT_F32, RAGGED, 2, 2, 2, 2, 2>(Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream);
    case 2: return launch_shape<OUT_F32, RAGGED, 2, 2, 2, 2, 4>(Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream);
    case 3: return launch_shape<OUT_F32, RAGGED, 2, 2, 1, 2, 3>(Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream);
    default: return launch_shape<OUT_F32, RAGGED, 2, 2, 1, 1, 4>(Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream);
  }
}

// Estimated duration in us with tiles of tm x tn: a tile costs a fixed part (first loads, epilogue) and, per step of 256 k,
// the larger of what one tile needs alone (lat) and what all n tiles of a compute unit need of it (thr each).  The
// constants are fits to graph replays of each shape forced, on 13 layers from 1 x 4096 -> 6144 to 8192 x 4096 -> 14336 (us,
// 256 x 256 | 128 x 128 | the same with four slots | 64 x 128 | 64 x 64): 4096 x 14336 -> 4096 116 | 146 | 180 | 188 | 252;
// 512 x 4096 -> 6144 31 | 16.4 | 14.8 | 15.3 | 19.5; 128 tokens 28 | 14.6 | 13.2 | 11.0 | 9.2; 1 token 26 | 10.7 | 10.9 | 9.1 |
// 7.4.  (Before: 189 with a 256 x 256 kernel of two
// stages, 89 | 31 | 18 with one wavefront per tile, mxfp4_gemm.hip, which keeps the layers of short K.)
// Rows of Y without 16-byte alignment make the fixed part per tile longer (per_tile.other; 777 x 256 -> 3001 FP32 15.0 | 7.0 | 7.1 | 6.4 | 6.9).
struct PerTile {
  double aligned, other;
};
double shape_cost_us(int64_t M, int64_t N, int64_t K, int tm, int tn, double base, PerTile per_tile, double lat, double thr,
                     int vec_store, int cus) {
  const int64_t tiles = ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
  if (tiles >= (int64_t)1 << 24) return 1e30;   // 256 work items each: a grid has fewer than 2^32
  const double n = (double)((tiles + cus - 1) / cus);
  return base + (vec_store ? per_tile.aligned : per_tile.other) * n + (double)((K + 255) / 256) * fmax(lat, thr * n);
}

}  // namespace

hipError_t launch_mxfp4_gemm_canon(const void* Xq, const void* Xs, const void* Wq, const void* Ws, int64_t M, int64_t N,
                                   int64_t K, int out_f32, void* Y, int64_t ldy, hipStream_t stream) {
  const int cus = device_cu_count();
  const bool one_each = ((M + 127) / 128) * ((N + 127) / 128) <= cus;   // 128 x 128: a compute unit's one workgroup gets four slots
  const int vec = canon_vec_store(Y, ldy, out_f32);
  const double cost[5] = {shape_cost_us(M, N, K, 256, 256, 1.0, {6.6, 13.0}, 1.95, 1.95, vec, cus),
                          shape_cost_us(M, N, K, 128, 128, 2.5, {1.8, 2.0}, 0.77, 0.64, vec, cus),
                          one_each ? shape_cost_us(M, N, K, 128, 128, 2.5, {1.8, 2.0}, 0.67, 0.67, vec, cus) : 1e30,
                          shape_cost_us(M, N, K, 64, 128, 2.7, {0.6, 1.2}, 0.47, 0.47, vec, cus),
                          shape_cost_us(M, N, K, 64, 64, 2.2, {0.8, 0.9}, 0.38, 0.28, vec, cus)};
  int shape = 0;
  for (int c = 1; c < 5; ++c)
    if (cost[c] < cost[shape]) shape = c;
  if (const int forced = debug_option(kDbgGemmTile); forced >= 0) shape = forced;
  const bool ragged = K % 256 != 0;
  if (out_f32)
    return ragged ? launch_any<true, true>(shape, Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream)
                  : launch_any<true, false>(shape, Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream);
  return ragged ? launch_any<false, true>(shape, Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream)
                : launch_any<false, false>(shape, Xq, Xs, Wq, Ws, M, N, K, Y, ldy, stream);
}

}  // namespace wush
