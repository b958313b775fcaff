// MXFP4 GEMM on canonical (row-major) operands where the layer has so few blocks of 32 tokens x 32 output channels that each gets a
// compute unit of its own: Y = deq(Xq,Xs) . deq(Wq,Ws)^T on v_mfma_scale_f32_32x32x64_f8f6f4, any M, N and K % 32 == 0.
//
// The pipelined tiles of mxfp4_gemm_canon.hip walk the whole K in one workgroup, 0.38 us per 256 elements at the least, with most compute
// units idle on such a layer.  Here the four wavefronts of a workgroup split K (the schedule of the tiled layout's kernel for few
// tokens), each with the operands of four K tiles of 256 in flight, straight from memory into registers: a lane's four fragments
// of a tile are 64 contiguous bytes of its row.  A load instruction touches 32 cache lines, four of them the same ones, and that
// is what bounds it where the tokens are many (16384 -> 1024: 1 token 14 us, 256 tokens 21.6; tiles 24 | 31).
#include "skinny_reduce.hpp"
#include "wush_kernels.hpp"

namespace wush {

namespace {

using skinny::kWaves;

struct Tile {   // (32 rows, 256 of K): a lane's four fragments and the scales of their groups
  v4i f[4];
  int s;
};
typedef int i32_any __attribute__((aligned(1)));

// Tile kt of block `blk` (32 rows) of an operand of `rows` rows and C groups of 32; a row past the last repeats it (never stored).
__device__ __forceinline__ void load_tile(Tile& t, const uint8_t* __restrict__ q, const uint8_t* __restrict__ s, int blk, int rows,
                                          int C, int kt, int lane) {
  const int64_t at = (int64_t)min(32 * blk + (lane & 31), rows - 1) * C + 8 * kt + 4 * (lane >> 5);
  const v4i* p = reinterpret_cast<const v4i*>(q + 16 * at);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) t.f[kk] = p[kk];
  t.s = *reinterpret_cast<const i32_any*>(s + at);
}
// The partial last tile of a row: groups past the row's end are zeros.
__device__ __forceinline__ void load_last_tile(Tile& t, const uint8_t* __restrict__ q, const uint8_t* __restrict__ s, int blk,
                                               int rows, int C, int lane) {
  const int g0 = (C & ~7) + 4 * (lane >> 5);
  const int64_t at = (int64_t)min(32 * blk + (lane & 31), rows - 1) * C + g0;
  t.s = 0x7F7F7F7F;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    t.f[kk] = (v4i){0, 0, 0, 0};
    if (g0 + kk < C) {
      t.f[kk] = *reinterpret_cast<const v4i*>(q + 16 * (at + kk));
      t.s = (t.s & ~(0xFF << (8 * kk))) | (int)s[at + kk] << (8 * kk);
    }
  }
}

__device__ __forceinline__ v16f multiply_tile(v16f acc, const Tile& w, const Tile& x) {
#define WUSH_ISSUE(KK)                                                                                 \
  {                                                                                                    \
    const v8i A_ = {w.f[KK][0], w.f[KK][1], w.f[KK][2], w.f[KK][3], 0, 0, 0, 0};                       \
    const v8i B_ = {x.f[KK][0], x.f[KK][1], x.f[KK][2], x.f[KK][3], 0, 0, 0, 0};                       \
    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A_, B_, acc, 4, 4, KK, w.s, KK, x.s);        \
  }
  WUSH_ISSUE(0)
  WUSH_ISSUE(1)
  WUSH_ISSUE(2)
  WUSH_ISSUE(3)
#undef WUSH_ISSUE
  return acc;
}

// Workgroup (x, y): output channels 32 x ..., tokens 32 y ...
template <bool OUT_F32>
__global__ __launch_bounds__(kWaves * 64) void gemm_canon_stream_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  constexpr int U = 4;                        // tiles in flight
  __shared__ v4f red[kWaves][1][4][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int C = K >> 5, j = blockIdx.x, rb = blockIdx.y;
  int kt0, kt1;
  skinny::wave_k_range(C >> 3, wave, kt0, kt1);
  v16f acc[1] = {{0}};
  for (int kt = kt0; kt < kt1; kt += U) {
    const int n = min(U, kt1 - kt);           // the same in every lane
    Tile w[U], x[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < n) load_tile(w[u], Wq, Ws, j, N, C, kt + u, lane);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < n) load_tile(x[u], Xq, Xs, rb, M, C, kt + u, lane);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u < n) acc[0] = multiply_tile(acc[0], w[u], x[u]);
  }
  if ((C & 7) && wave == kWaves - 1) {        // the wavefront with the fewest whole tiles
    Tile w, x;
    load_last_tile(w, Wq, Ws, j, N, C, lane);
    load_last_tile(x, Xq, Xs, rb, M, C, lane);
    acc[0] = multiply_tile(acc[0], w, x);
  }
  skinny::reduce_store_block<1, OUT_F32>(acc, red, j, M - 32 * rb, N, static_cast<uint8_t*>(Y) + 32 * (int64_t)rb * ldy * (OUT_F32 ? 4 : 2),
                                         ldy, lane, wave);
}

// At most 16 tokens, on v_mfma_scale_f32_16x16x128_f8f6f4: no padding to 32 rows.  Quarter q of the lanes has 32 of the 128 bytes of its row's
// line, 16 for each of a tile's two instructions, so an instruction of either operand touches 16 lines and the tile uses them whole; the scales of
// its two groups are bytes 0 and 1 of the row's dword shifted by the quarter.  HALVES and R as in the tiled layout's kernel: 16-channel halves of a
// block of 32 output channels a workgroup takes, K tiles a wavefront keeps in flight (three where both halves are taken from K = 4096 on; two in place
// of them within 1 %, four 0 to 2 % slower).  Replayed graphs, four sets of operands, us, 32 rows | this:
// 1 x 14336 -> 4096 15.1 | 7.9, 16 tokens 16.5 | 11.7; 1 x 24160 -> 1409 22.9 | 9.1; 16 x 16384 -> 1024 17.9 | 12.5; 1 x 4096 -> 4096 6.0 | 3.8;
// tiles | this: 1 x 28672 -> 8192 36.4 | 27.3, 1 x 8192 -> 8192 10.1 | 8.7, 1 x 2080 -> 20000 8.5 | 6.8.
struct HalfTile {   // (16 rows, 256 of K)
  v4i f[2];
  int s;
};
template <int HALVES, int R, bool OUT_F32>
__global__ __launch_bounds__(kWaves * 64) void gemm_canon_stream16_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const uint8_t* __restrict__ Wq,
    const uint8_t* __restrict__ Ws, int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  __shared__ v4f red[kWaves][HALVES][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, q = lane >> 4, C = K >> 5;
  const int NB = (N + 16 * HALVES - 1) / (16 * HALVES);
  int kt0, kt1;
  skinny::wave_k_range(C >> 3, wave, kt0, kt1);
  const int64_t x_at = (int64_t)min(l16, M - 1) * C;
  const int j = blockIdx.x + gridDim.x * blockIdx.z;
  if (j >= NB) return;                        // the grid's padding
  int64_t w_at[HALVES];
#pragma unroll
  for (int a = 0; a < HALVES; ++a) w_at[a] = (int64_t)min(16 * (HALVES * j + a) + l16, N - 1) * C;
  v4f acc[HALVES];
#pragma unroll
  for (int a = 0; a < HALVES; ++a) acc[a] = (v4f){0, 0, 0, 0};
  HalfTile w[R][HALVES], x[R];
  auto load_half = [&](HalfTile& t, const uint8_t* qp, const uint8_t* sp, int64_t at, int kt) {
    const v4i* p = reinterpret_cast<const v4i*>(qp + 16 * (at + 8 * kt + 2 * q));
    t.f[0] = p[0];
    t.f[1] = p[1];
    t.s = *reinterpret_cast<const i32_any*>(sp + at + 8 * kt + 4 * (q >> 1));   // shifted when it is multiplied: here it would be waited for
  };
  // the partial last tile of a row: groups past the row's end are zeros
  auto load_last = [&](HalfTile& t, const uint8_t* qp, const uint8_t* sp, int64_t at) {
    int two = 0x7F7F;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int g = (C & ~7) + 2 * q + p;
      t.f[p] = (v4i){0, 0, 0, 0};
      if (g < C) {
        t.f[p] = *reinterpret_cast<const v4i*>(qp + 16 * (at + g));
        two = (two & ~(0xFF << (8 * p))) | (int)sp[at + g] << (8 * p);
      }
    }
    t.s = two << (16 * (q & 1));
  };
  auto load = [&](int u, int kt) {
#pragma unroll
    for (int a = 0; a < HALVES; ++a) load_half(w[u][a], Wq, Ws, w_at[a], kt);
    load_half(x[u], Xq, Xs, x_at, kt);
  };
  auto multiply = [&](int u) {
    const int sx = x[u].s >> (16 * (q & 1));
#pragma unroll
    for (int a = 0; a < HALVES; ++a) {
      const int sw = w[u][a].s >> (16 * (q & 1));
#define WUSH_HALF_ISSUE(P)                                                                                                    \
  {                                                                                                                         \
    const v8i A_ = {w[u][a].f[P][0], w[u][a].f[P][1], w[u][a].f[P][2], w[u][a].f[P][3], 0, 0, 0, 0};                        \
    const v8i B_ = {x[u].f[P][0], x[u].f[P][1], x[u].f[P][2], x[u].f[P][3], 0, 0, 0, 0};                                    \
    acc[a] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(A_, B_, acc[a], 4, 4, P, sw, P, sx);                          \
  }
      WUSH_HALF_ISSUE(0)
      WUSH_HALF_ISSUE(1)
#undef WUSH_HALF_ISSUE
    }
  };
  skinny::ring<R>(kt0, kt1, load, multiply);
  if ((C & 7) && wave == kWaves - 1) {      // the wavefront with the fewest whole tiles
#pragma unroll
    for (int a = 0; a < HALVES; ++a) load_last(w[0][a], Wq, Ws, w_at[a]);
    load_last(x[0], Xq, Xs, x_at);
    multiply(0);
  }
  // the waves' sums in their order; accumulator v of lane (l16, q) is token l16, output channel 4 q + v of the half
#pragma unroll
  for (int a = 0; a < HALVES; ++a) red[wave][a][lane] = acc[a];
  __syncthreads();
  if (wave < HALVES) {
    const v4f sum = ((red[0][wave][lane] + red[1][wave][lane]) + red[2][wave][lane]) + red[3][wave][lane];
    const int col = 16 * (HALVES * j + wave) + 4 * q;
    const float v[4] = {sum[0], sum[1], sum[2], sum[3]};
    if (l16 < M && col < N) skinny::store_quad<OUT_F32>(Y, ldy, l16, col, N, col + 4 <= N, v);
  }
}

}  // namespace

// One workgroup per compute unit at the most (us, tiles | this kernel: 48 x 4096 -> 4096 9.2 | 7.5, 256 x 16384 -> 1024 29 | 20.8, 448 x 28672 -> 512
// 52 | 34; with more: 100 x 4096 -> 4096 8.8 | 12.4; 16-row kernel 16 x 1376 -> 3000 4.6 | 2.6, 1 x 4096 -> 4096 9.0 | 3.9, 1 x 14336 -> 4096
// 25.5 | 7.9).
bool canon_streams(int64_t M, int64_t N) {
  return M <= 8192 && N <= 8192 && ((M + 31) / 32) * ((N + 31) / 32) <= device_cu_count();
}

// More blocks of output channels than compute units, at most 16 tokens: where the 16-row kernel is ahead of the tiles, which read a layer's
// weights in larger pieces (us, tiles | 16 rows: 1 x 1024 -> 16384 4.6 | 3.9, 4 x 4096 -> 12288 9.7 | 8.9, 4 x 6144 -> 16384 13.8 | 12.0, 1 x 14336 ->
// 16384 36.7 | 26.4, 16 tokens 38.8 | 34.9; but 8 x 2048 -> 20000 7.3 | 7.8, 16 x 8192 -> 12000 16.6 | 18.2, 16 x 8192 -> 28672 32.8 | 36.9,
// 16 x 4096 -> 57344 25.7 | 32.8, 1 x 28672 -> 57344 151 | 173).  The lines were drawn with an earlier ring, 5 to 30 % slower, and the 16-row kernel is now
// ahead of the tiles on most layers beyond them too (1 x 8192 -> 28672 32.1 | 27.7, 8 x 832 -> 34416 8.4 | 5.3, 1 x 9088 -> 16789 33.8 | 24.3): on 629
// drawn layers of K from 512 on these lines are 10 % off the faster kernel in the mean; 16 rows up to 8 tokens until 6 blocks per compute unit or
// K = 12288, more tokens until 3 or K = 4096, would be 0.5 %.
bool canon_streams16(int64_t M, int64_t N, int64_t K) {
  const bool few = (N + 31) / 32 <= 2 * device_cu_count();
  return M <= 16 && ((M <= 4 && (K <= 2560 || few)) || (K >= 12288 && few));
}

hipError_t launch_mxfp4_gemm_canon_stream(const void* Xq, const void* Xs, const void* Wq, const void* Ws, int64_t M, int64_t N,
                                          int64_t K, int out_f32, void* Y, int64_t ldy, hipStream_t stream) {
  if (M <= 16) {
    const bool halves = (N + 15) / 16 <= device_cu_count();
    const int64_t blocks = halves ? (N + 15) / 16 : (N + 31) / 32;
    const int ring = K <= 2048 ? 1 : halves || K < 4096 ? 2 : 3;
#define WUSH_CANON16(HALVES, R) (out_f32 ? gemm_canon_stream16_kernel<HALVES, R, true> : gemm_canon_stream16_kernel<HALVES, R, false>)
    auto kernel = halves ? (ring == 1 ? WUSH_CANON16(1, 1) : WUSH_CANON16(1, 2))
                         : (ring == 1 ? WUSH_CANON16(2, 1) : ring == 2 ? WUSH_CANON16(2, 2) : WUSH_CANON16(2, 3));
#undef WUSH_CANON16
    kernel<<<skinny::wide_grid(blocks, 1), dim3(kWaves * 64), 0, stream>>>(
        (const uint8_t*)Xq, (const uint8_t*)Xs, (const uint8_t*)Wq, (const uint8_t*)Ws, (int)M, (int)N, (int)K, Y, ldy);
    return hipGetLastError();
  }
  auto kernel = out_f32 ? gemm_canon_stream_kernel<true> : gemm_canon_stream_kernel<false>;
  kernel<<<dim3((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32)), dim3(kWaves * 64), 0, stream>>>(
      (const uint8_t*)Xq, (const uint8_t*)Xs, (const uint8_t*)Wq, (const uint8_t*)Ws, (int)M, (int)N, (int)K, Y, ldy);
  return hipGetLastError();
}

}  // namespace wush
