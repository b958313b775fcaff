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
  __shared__ float red[kWaves][1][16][64];
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

}  // namespace

// One workgroup per compute unit at the most (us, tiles | this kernel: 1376 -> 3000, 16 tokens 6.3 | 4.2; 4096 -> 4096, 48 tokens 8.6 |
// 8.1; 14336 -> 4096, 1 token 26.8 | 14.5; 16384 -> 1024, 256 tokens 31 | 21.6; 28672 -> 512, 448 tokens 53 | 36; with more: 4096 ->
// 4096, 100 tokens 8.8 | 12.4; 1024 -> 16384, 1 token 4.6 | 4.6; 8192 -> 28672, 1 token 22.4 | 30.6).
bool canon_streams(int64_t M, int64_t N) {
  return M <= 8192 && N <= 8192 && ((M + 31) / 32) * ((N + 31) / 32) <= device_cu_count();
}

hipError_t launch_mxfp4_gemm_canon_stream(const void* Xq, const void* Xs, const void* Wq, const void* Ws, int64_t M, int64_t N,
                                          int64_t K, int out_f32, void* Y, int64_t ldy, hipStream_t stream) {
  auto kernel = out_f32 ? gemm_canon_stream_kernel<true> : gemm_canon_stream_kernel<false>;
  kernel<<<dim3((unsigned)((N + 31) / 32), (unsigned)((M + 31) / 32)), dim3(kWaves * 64), 0, stream>>>(
      (const uint8_t*)Xq, (const uint8_t*)Xs, (const uint8_t*)Wq, (const uint8_t*)Ws, (int)M, (int)N, (int)K, Y, ldy);
  return hipGetLastError();
}

}  // namespace wush
