// Offline construction of the per-block WUSH transforms on the GPU
// (Alg. 2, RTN case, first two steps, and Alg. 1):
//   M_W = d_out^-1 W_(i) W_(i)^T,  M_X = d_batch^-1 X_(i) X_(i)^T     (per block i)
//   W' W'^T = M_W + lambda d^-1 tr(M_W) I,  X' X'^T = likewise         (Cholesky)
//   U S V^T = W'^T X'                                                  (SVD)
//   T_wush = H S^(-1/2) U^T W'^T                                       (the WUSH construction equation)
// Everything is FP64.  Products of two BF16 inputs are exact, so the second
// moments differ from an FP64 reference only in summation order.
//
//   1. second_moment_kernel: grid (block, row split, {W, X}); a workgroup
//      streams its rows of one 32-channel block through LDS and accumulates the
//      32x32 moment on the FP64 MFMA, each wave every fourth group of 4 rows; partial
//      sums go to the workspace (fixed split -> fixed summation order, no atomics).
//   2. wush_block_kernel: one workgroup of four wavefronts per block (two for 16 x 16
//      blocks): reduce the partials, damp, Cholesky of both moments side by side, A = W'^T X',
//      SVD of A by right rotations (sweeps of one-sided Jacobi, then all small
//      angles at once; V is never needed), sort, sign convention
//      (largest-magnitude entry of each column of U positive), then
//      T = H diag(s^-1/2) U^T W'^T, rounded to BF16 (nearest even, straight from
//      FP64).
#include "wush_block.hpp"
#include "wush_kernels.hpp"

namespace wush {

namespace {

constexpr int kRowsPerStep = 128;

// Row of the 16 x 16 result block that accumulator element v of a lane holds (v_mfma_f64_16x16x4_f64;
// its column is lane % 16).  Checked by the parity tests of the transforms: the other candidate,
// 4 (lane / 16) + v, gives moments that are not positive definite.
__device__ __forceinline__ int mfma_f64_row(int lane, int v) { return (lane >> 4) + 4 * v; }

__global__ __launch_bounds__(256) void second_moment_kernel(
    const uint16_t* __restrict__ W, int64_t ldw, int N, const uint16_t* __restrict__ X, int64_t ldx, int Mc,
    int rows_per_split_w, int rows_per_split_x, int S, int C, double* __restrict__ partial, int* __restrict__ status) {
  // the kernel behind this one may set the status word
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x < 4) status[threadIdx.x] = 0;
  // 2 * 1024 FP64 flop per row and block against 64 bytes read: arithmetic bound, so the products run
  // on the FP64 MFMA (16 x 16 x 4: four rows of the block at a time).  With A[i][k] = x[row k][channel i]
  // and B[k][j] = x[row k][channel j] a lane feeds both operands from the element (row lane / 16,
  // channel lane % 16) of a 16-channel half; the moment is symmetric, so the two diagonal 16 x 16
  // blocks and one off-diagonal block are computed (3 MFMAs per 4 rows) and the fourth is its mirror.  c2 layer: 42 us, the
  // MFMAs alone 26 (47 with twice the splits and the waves' sums in LDS of their own: three workgroups per CU instead of six).
  // A wave takes every fourth group of 4 rows; the four waves' sums are added at the end in wave order.
  __shared__ __attribute__((aligned(16))) float tile[kRowsPerStep][48];   // row stride 48: the 4-row reads hit 32 distinct banks per half wave
  static_assert(sizeof(tile) >= 3 * 768 * sizeof(double), "the waves' sums fit the tile");
  double (*red)[768] = reinterpret_cast<double (*)[768]>(tile);
  const int b = blockIdx.x, s = blockIdx.y, z = blockIdx.z;
  const uint16_t* A = z == 0 ? W : X;
  const int64_t ld = z == 0 ? ldw : ldx;
  const int rows = z == 0 ? N : Mc;
  const int per = z == 0 ? rows_per_split_w : rows_per_split_x;
  const int r_begin = min(s * per, rows), r_end = min(r_begin + per, rows);
  if (r_begin == r_end) return;   // a split with no rows left: its partial moment is not read
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int k = lane >> 4, c = lane & 15;
  v4d acc00 = {0, 0, 0, 0}, acc01 = {0, 0, 0, 0}, acc11 = {0, 0, 0, 0};
  // 128 rows x 4 chunks of 8 BF16 per step: two chunks per thread (rows past the end contribute zeros);
  // the chunks of the next step are fetched while this one is multiplied
  const int rr0 = threadIdx.x >> 2, ch = threadIdx.x & 3;
  v4u raw[2];
  auto fetch = [&](int r0) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int row = r0 + rr0 + 64 * u;
      raw[u] = (v4u){0, 0, 0, 0};
      if (row < r_end) raw[u] = *reinterpret_cast<const v4u*>(A + (int64_t)row * ld + 32 * b + 8 * ch);
    }
  };
  fetch(r_begin);
  for (int r0 = r_begin; r0 < r_end; r0 += kRowsPerStep) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float4 lo, hi;
      lo.x = __uint_as_float(raw[u][0] << 16); lo.y = __uint_as_float(raw[u][0] & 0xFFFF0000u);
      lo.z = __uint_as_float(raw[u][1] << 16); lo.w = __uint_as_float(raw[u][1] & 0xFFFF0000u);
      hi.x = __uint_as_float(raw[u][2] << 16); hi.y = __uint_as_float(raw[u][2] & 0xFFFF0000u);
      hi.z = __uint_as_float(raw[u][3] << 16); hi.w = __uint_as_float(raw[u][3] & 0xFFFF0000u);
      *reinterpret_cast<float4*>(&tile[rr0 + 64 * u][8 * ch]) = lo;
      *reinterpret_cast<float4*>(&tile[rr0 + 64 * u][8 * ch + 4]) = hi;
    }
    __syncthreads();
    if (r0 + kRowsPerStep < r_end) fetch(r0 + kRowsPerStep);
#pragma unroll
    for (int t = 0; t < kRowsPerStep / 16; ++t) {
      const int rr = 4 * (wave + 4 * t) + k;
      const double x0 = tile[rr][c], x1 = tile[rr][16 + c];
      acc00 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x0, acc00, 0, 0, 0);
      acc01 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x1, acc01, 0, 0, 0);
      acc11 = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x1, acc11, 0, 0, 0);
    }
  }
  __syncthreads();
  // waves 1..3 hand their sums to wave 0, which adds them in wave order and writes the 32 x 32 partial
  if (wave > 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      red[wave - 1][4 * lane + v] = acc00[v];
      red[wave - 1][256 + 4 * lane + v] = acc01[v];
      red[wave - 1][512 + 4 * lane + v] = acc11[v];
    }
  }
  __syncthreads();
  if (wave == 0) {
    double* out = partial + (((int64_t)z * S + s) * C + b) * kMomentSize;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = 4 * lane + v, i = mfma_f64_row(lane, v);
      const double m00 = ((acc00[v] + red[0][e]) + red[1][e]) + red[2][e];
      const double m01 = ((acc01[v] + red[0][256 + e]) + red[1][256 + e]) + red[2][256 + e];
      const double m11 = ((acc11[v] + red[0][512 + e]) + red[1][512 + e]) + red[2][512 + e];
      out[moment_beside(i, c)] = m01;
      if (c <= i) {
        out[lower16(i, c)] = m00;
        out[moment_second(i, c)] = m11;
      }
    }
  }
}

// The first S_W splits of S hold rows of W, the first S_X rows of X.
// FLIGHT = partial moments of either operand in flight.  16 of them take a wavefront's 404 registers, a compute unit's one workgroup; 4, all there are
// where the blocks are so many that they go round by round, 122 (16 x 16 blocks 270 and 89), and three workgroups share a compute unit.
template <int FLIGHT>
__global__ __launch_bounds__(256) void wush_block_kernel(const double* __restrict__ partial, int S, int S_W, int S_X,
                                                         int C, int N, int Mc, double lambda, uint16_t* __restrict__ T_out,
                                                         double* __restrict__ T_f64, int* __restrict__ status) {
  const int b = blockIdx.x;
  // the partial moments are added in a fixed order and normalized
  auto load = [&](int half, int e, int, int, int s) { return partial[(((int64_t)half * S + s) * C + b) * kMomentSize + e]; };
  auto finish = [&](int half, double sum) { return sum * (1.0 / (double)(half ? Mc : N)); };
  __shared__ BlockShared<32> sh;
  wush_block_group<32, 0, FLIGHT, FLIGHT>(sh, load, finish, S_W, S_X, lambda, nullptr, T_out + (int64_t)b * 1024,
                                          T_f64 ? T_f64 + (int64_t)b * 1024 : nullptr, nullptr, status);
}

// The same for 16 x 16 blocks (the NVFP4 variant: transform block = quantization group of 16).  The
// moments of block b are the diagonal 16 x 16 sub-block (b & 1) of the 32-channel moments of block b / 2.
template <int FLIGHT>
__global__ __launch_bounds__(128) void wush_block16_kernel(const double* __restrict__ partial, int S, int S_W, int S_X,
                                                           int C, int N, int Mc, double lambda, uint16_t* __restrict__ T_out,
                                                           double* __restrict__ T_f64, int* __restrict__ status) {
  const int b = blockIdx.x, b32 = b >> 1, off = b & 1 ? moment_second(0, 0) : 0;
  auto load = [&](int half, int e, int, int, int s) {
    return partial[(((int64_t)half * S + s) * C + b32) * kMomentSize + off + e];
  };
  auto finish = [&](int half, double sum) { return sum * (1.0 / (double)(half ? Mc : N)); };
  __shared__ BlockShared<16> sh;
  wush_block_group<16, 0, FLIGHT, FLIGHT>(sh, load, finish, S_W, S_X, lambda, nullptr, T_out + (int64_t)b * 256,
                                          T_f64 ? T_f64 + (int64_t)b * 256 : nullptr, nullptr, status);
}

// Splits of the rows, for about four workgroups of each moment per compute unit.  Every split costs a partial moment of 4.1 KiB per
// block, written and read back (both kernels together, us, 2048 / C | 1024 / C | 512 / C: c2 layer 107.3 | 104.6 | 102.9,
// 8192 x 8192 -> 57344 495 | 502 | 539, 512 x 1024 -> 1024 70.2 | 70.2 | 70.1); partials of splits without rows are not read.
int splits_for(int64_t C) {
  int64_t s = 1024 / C;
  if (s < 1) s = 1;
  if (s > 256) s = 256;
  return (int)s;
}

// Partial moments in flight, by how many there are: four at most from 205 blocks of 32 channels on, where the blocks start to outnumber the compute
// units (both kernels, us, 16 | 4 in flight, 32 x 32 blocks; 16 x 16: 8192 channels, 8192 + 2048 rows 143 | 141; 109 | 109; 12288, 2048 + 2048 rows
// 159 | 131; 100 | 82; 16384, 4096 + 2048 rows 205 | 169; 148 | 123; 28672, 1024 + 1024 rows 268 | 206; 148 | 101, 8192 + 2048 rows 465 | 399; 353 | 311).
constexpr int kFewSplits = 4, kManySplits = 16;

}  // namespace

size_t build_transforms_status_offset(int64_t K) {
  const int64_t C = K / 32;
  return (size_t)(2 * splits_for(C) * C) * 1024 * sizeof(double);
}

size_t build_transforms_workspace_bytes(int64_t K) { return build_transforms_status_offset(K) + 16; }

hipError_t launch_build_transforms(const void* W, int64_t N, int64_t ldw, const void* X, int64_t Mc, int64_t ldx,
                                   int64_t K, double lambda, int block, void* T_out, double* T_f64, void* workspace,
                                   hipStream_t stream) {
  const int C = (int)(K / 32);
  const int S = splits_for(C);
  double* partial = reinterpret_cast<double*>(workspace);
  int* status = reinterpret_cast<int*>(reinterpret_cast<char*>(workspace) + build_transforms_status_offset(K));
  auto per = [&](int64_t rows) { return (int)(((rows + S - 1) / S + kRowsPerStep - 1) / kRowsPerStep * kRowsPerStep); };
  auto used = [&](int64_t rows) { return (int)((rows + per(rows) - 1) / per(rows)); };
  second_moment_kernel<<<dim3(C, S, 2), dim3(256), 0, stream>>>((const uint16_t*)W, ldw, (int)N, (const uint16_t*)X,
                                                               ldx, (int)Mc, per(N), per(Mc), S, C, partial, status);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool few = used(N) <= kFewSplits && used(Mc) <= kFewSplits;
  if (block == 16) {
    auto kernel = few ? wush_block16_kernel<kFewSplits> : wush_block16_kernel<kManySplits>;
    kernel<<<dim3(2 * C), dim3(128), 0, stream>>>(partial, S, used(N), used(Mc), C, (int)N, (int)Mc, lambda, (uint16_t*)T_out, T_f64, status);
  } else {
    auto kernel = few ? wush_block_kernel<kFewSplits> : wush_block_kernel<kManySplits>;
    kernel<<<dim3(C), dim3(256), 0, stream>>>(partial, S, used(N), used(Mc), C, (int)N, (int)Mc, lambda, (uint16_t*)T_out, T_f64, status);
  }
  return hipGetLastError();
}

}  // namespace wush
