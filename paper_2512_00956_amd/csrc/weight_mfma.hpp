// The offline block products Wt_blk = W_blk inv(T_b) in FP64 on the FP64 MFMA (16 x 16 x 4), 16 rows of W at a
// time per wavefront.
//
// The product is taken transposed, D[j][n] = sum_k inv(T)[k][j] W[n][k], with the order of j (rows of the first
// operand) and of k (the four lane groups and the issues) chosen so that lane (l16, l4) = (lane % 16, lane / 16)
// reads 8 consecutive channels of row n = l16 -- one 16-byte load -- and ends up with 8 consecutive transformed
// channels of the same row: 32 bits of codes.  A quantization group of 32 lives in the four lanes l4 of one
// column, so its scale needs two cross-lane steps and nothing passes through LDS.
// v_mfma_f64_16x16x4_f64: first operand A[i = l16][k = l4], second B[k = l4][n = l16], accumulator element v is
// D[l4 + 4 v][l16].
#pragma once
#include "wush_device.hpp"

namespace wush {
namespace wm {

typedef double v4d __attribute__((ext_vector_type(4)));

// The other lanes' x: of lane ^ 16 (rows of 16 swapped in pairs), of lane ^ 32.
__device__ __forceinline__ float max_xor16(float x) {
  const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float max_xor32(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
// (even, odd): x of the even one and of the odd one of the two rows of 16 lanes that form a pair; (low, high):
// x of the lower and of the upper half of the wavefront.
struct PairF64 { double first, second; };
__device__ __forceinline__ PairF64 pair16(double a, double b) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return {__longlong_as_double((long long)((uint64_t)hi[0] << 32 | lo[0])),
          __longlong_as_double((long long)((uint64_t)hi[1] << 32 | lo[1]))};
}
__device__ __forceinline__ PairF64 pair32(double a) {
  const uint64_t x = (uint64_t)__double_as_longlong(a);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(x >> 32), false, false);
  return {__longlong_as_double((long long)((uint64_t)hi[0] << 32 | lo[0])),
          __longlong_as_double((long long)((uint64_t)hi[1] << 32 | lo[1]))};
}

// Eight BF16 (16 bytes) as FP64.
__device__ __forceinline__ void widen8(const v4u& raw, double (&w)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    w[2 * i] = (double)__uint_as_float(raw[i] << 16);
    w[2 * i + 1] = (double)__uint_as_float(raw[i] & 0xFFFF0000u);
  }
}

// ---- 32 x 32 blocks.  First operand of the lane: row i = l16 of tile t is j = 8 (i % 4) + 4 t + i / 4, k = 8 l4 + kk,
// so that accumulator v of tile t is j = 8 l4 + 4 t + v.
struct Block32 { double m[2][8]; };
// entry(k, j): element of the matrix the rows are multiplied with
template <class EntryFn>
__device__ __forceinline__ void load_block32(Block32& b, EntryFn entry, int lane) {
  const int l16 = lane & 15, l4 = lane >> 4;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) b.m[t][kk] = entry(8 * l4 + kk, 8 * (l16 & 3) + 4 * t + (l16 >> 2));
}
// w: channels 8 l4 ... + 7 of row l16; y += the transformed channels 8 l4 ... + 7 of the same row
__device__ __forceinline__ void multiply32(const Block32& b, const double (&w)[8], double (&y)[8]) {
  v4d acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) acc[t] = (v4d){y[4 * t], y[4 * t + 1], y[4 * t + 2], y[4 * t + 3]};
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
#pragma unroll
    for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(b.m[t][kk], w[kk], acc[t], 0, 0, 0);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v) y[4 * t + v] = acc[t][v];
}

// ---- two 16 x 16 blocks (channels 0..15 and 16..31 of a chunk of 32): k = 4 l4 + kk of either, accumulator v of
// tile a is channel 4 l4 + v of block a; the lane reads 8 bytes of each.
struct Block16x2 { double m[2][4]; };
__device__ __forceinline__ void load_block16x2(Block16x2& b, const double* __restrict__ inv0, int lane) {
  const int l16 = lane & 15, l4 = lane >> 4;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) b.m[a][kk] = inv0[256 * a + 16 * (4 * l4 + kk) + 4 * (l16 & 3) + (l16 >> 2)];
}
__device__ __forceinline__ void multiply16x2(const Block16x2& b, const v2u (&raw)[2], double (&y)[2][4]) {
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    v4d acc = {0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const uint32_t word = raw[a][kk >> 1];
      const double w = (double)__uint_as_float((kk & 1) ? (word & 0xFFFF0000u) : (word << 16));
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(b.m[a][kk], w, acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) y[a][v] = acc[v];
  }
}

// How many workgroups share the rows of one group of four 32-channel blocks: enough waves for four per SIMD, at
// least one 16-row tile each.  Step s of workgroup g takes tile s G + g, so that the grid as a whole moves
// down the rows once.
inline int row_groups(int64_t rows, int64_t blocks32, int cus) {
  const int64_t tiles = (rows + 15) / 16, per = (blocks32 + 3) / 4;
  int64_t g = (4 * (int64_t)cus + per - 1) / per;
  if (g > tiles) g = tiles;
  return (int)(g < 1 ? 1 : g);
}

}  // namespace wm
}  // namespace wush
