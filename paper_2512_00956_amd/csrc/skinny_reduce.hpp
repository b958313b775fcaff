// Pieces shared by the weight-streaming GEMM kernels for few tokens (MXFP4: layer_decode.hip; NVFP4 and
// INT4: w4_gemm_skinny.hip): a workgroup of four waves owns 32 output channels at a time, its waves
// split K into four contiguous ranges and their partial 32 x 32 tiles are summed through LDS in a
// fixed order (deterministic).
#pragma once
#include "wush_device.hpp"

namespace wush {
namespace skinny {

constexpr int kWaves = 4;

// Four consecutive output channels of a token, in one store of 8 (BF16) or 16 bytes (FP32) whatever its alignment: gfx950 takes
// one at any address.  Element by element, rows off the vector's alignment took four times the store instructions, each
// touching the lines of the one (us, element by element | one store: NVFP4 1000 x 256 -> 4093 FP32 19.9 | 11.9, 2667 x 3328 -> 5899 FP32
// 149 | 123, INT4 4000 x 1024 -> 1021 FP32 28.4 | 20.0, MXFP4 512 x 1024 -> 2045 6.9 | 5.2).
// whole: all four channels exist.
template <bool OUT_F32>
__device__ __forceinline__ void store_quad(void* __restrict__ Y, int64_t ldy, int row, int col, int N, bool whole,
                                           const float (&v)[4]) {
  if constexpr (OUT_F32) {
    typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
    float* y = reinterpret_cast<float*>(Y) + (int64_t)row * ldy + col;
    if (whole || col + 4 <= N) {
      *reinterpret_cast<v4f_any*>(y) = (v4f){v[0], v[1], v[2], v[3]};
    } else {                                  // the last channels of a row
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (col + t < N) y[t] = v[t];
    }
  } else {
    typedef uint32_t v2u_any __attribute__((ext_vector_type(2), aligned(2)));
    uint16_t* y = reinterpret_cast<uint16_t*>(Y) + (int64_t)row * ldy + col;
    if (whole || col + 4 <= N) {
      v2u two;
      two[0] = (uint32_t)f32_to_bf16_bits(v[0]) | ((uint32_t)f32_to_bf16_bits(v[1]) << 16);
      two[1] = (uint32_t)f32_to_bf16_bits(v[2]) | ((uint32_t)f32_to_bf16_bits(v[3]) << 16);
      *reinterpret_cast<v2u_any*>(y) = two;
    } else {
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (col + t < N) y[t] = f32_to_bf16_bits(v[t]);
    }
  }
}

// Sum the four waves' partial tiles of column block j (fixed order 0,1,2,3), multiply by `scale` if
// SCALED (the product of the tensor scales of a format that has them), and store.  Accumulator e of lane (r, kh), row block rb is token 32*rb + r, output
// channel 32*j + 8*(e/4) + 4*kh + e%4; wave w finishes the quads e/4 == w.
template <int RB, bool OUT_F32, bool SCALED = false>
__device__ __forceinline__ void reduce_store_block(const v16f (&acc)[RB], v4f (*red)[RB][4][64], int j, int M, int N,
                                                   void* __restrict__ Y, int64_t ldy, int lane, int wave,
                                                   float scale = 1.0f) {
  const int r = lane & 31, kh = lane >> 5;
  const bool whole = 32 * j + 32 <= N;          // the same in every lane
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int q = 0; q < 4; ++q) red[wave][rb][q][lane] = (v4f){acc[rb][4 * q], acc[rb][4 * q + 1], acc[rb][4 * q + 2], acc[rb][4 * q + 3]};
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const v4f sum = ((red[0][rb][wave][lane] + red[1][rb][wave][lane]) + red[2][rb][wave][lane]) + red[3][rb][wave][lane];
    float v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = SCALED ? sum[t] * scale : sum[t];
    const int row = 32 * rb + r;
    const int col = 32 * j + 8 * wave + 4 * kh;
    if (row < M && (whole || col < N)) store_quad<OUT_F32>(Y, ldy, row, col, N, whole, v);
  }
  __syncthreads();   // red is rewritten by the next column block
}

// Contiguous K-tile range of a wave: the four waves split KT as evenly as possible.
__device__ __forceinline__ void wave_k_range(int KT, int wave, int& kt0, int& kt1) {
  const int q = (KT + kWaves - 1) / kWaves;
  kt0 = min(wave * q, KT);
  kt1 = min(kt0 + q, KT);
}

// A grid with `blocks` workgroups of 256 threads side by side and `groups` rows of them: 2^30 output channels are 2^25 blocks, which go on along z.
inline dim3 wide_grid(int64_t blocks, int groups) {
  constexpr int64_t kMost = 1 << 20;   // along x
  return dim3((unsigned)(blocks < kMost ? blocks : kMost), (unsigned)groups, (unsigned)((blocks + kMost - 1) / kMost));
}

// K tiles [kt, kt1) of a wavefront through a ring of R: load(u, t) requests tile t into slot u, multiply(u) multiplies slot u, which is then
// refilled at once.  The compiler's count of the loads in flight has to stay exact, or it waits for loads it has no need of.  Where the tiles are
// no multiple of R the first slots start out empty: a branch around a product does not touch the count, one around a refill at the
// end does, and so does a first load that may be missing (MXFP4, us, first loads and refills under branches | this:
// 48 x 27136 -> 379 13.0 | 11.1, 62 x 7168 -> 704 5.6 | 4.6, 18 x 26880 -> 128 11.4 | 9.9, 9 x 28672 -> 1024 9.0 | 7.8; 300 layers of K from 4096 on
// and up to 1024 channels, 17 to 256 tokens: geomean 0.89).
// With one slot there is nothing to count, and a way around all of it would have the accumulators cleared ahead of the first load.
template <int R, class Load, class Multiply>
__device__ __forceinline__ void ring(int kt, int kt1, const Load& load, const Multiply& multiply) {
  if (R > 1 && kt >= kt1) return;
  int t = kt1 - max((kt1 - kt + R - 1) / R, 1) * R;   // tile of slot 0
#pragma unroll
  for (int u = 0; u < R; ++u)
    if ((R > 1 && u == R - 1) || t + u >= kt) load(u, t + u);
  __builtin_amdgcn_sched_barrier(0);
  for (; t + R < kt1; t += R) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      if (u == R - 1 || t + u >= kt) multiply(u);
      load(u, t + R + u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < R; ++u)
    if ((R > 1 && u == R - 1) || t + u >= kt) multiply(u);
}

}  // namespace skinny
}  // namespace wush
