// Offline weight path, GPTQ case of Alg. 2: WUSH transforms interleaved with
// GPTQ's intra-block and inter-block error propagation.  Everything is FP64; the
// path runs once per layer.
//
// The paper's schedule uses L, the lower Cholesky factor of the inverse of the
// damped Hessian Hd = H + lambda tr(H)/d_in I, through three quantities per
// block i: (L_ii L_ii^T)^-1, and L_ji L_ii^-1 for j > i.  This file never
// inverts Hd.  With the reverse Cholesky factorization Hd = U U^T (U upper
// triangular) and V = U^-1 one has L = V^T, hence
//     (L_ii L_ii^T)^-1       = U_ii U_ii^T
//     (L_ji L_ii^-1)^T       = U_ii V_ij                (j > i),
// so block j enters its step as W_j + D_j with D_j = sum_{i<j} E_i U_ii V_ij, E_i the error of block i against what it
// entered with.  With F_i = E_i U_ii the D_j + E_j are the blocks of F V, and (F V) U = F gives, block by block,
//     D_j = -(sum_{i<j} G_i U_ij) V_jj,   G_i = E_i + D_i = (deq T)_i - W_i (the ORIGINAL weights):
// the propagation needs the factor U and the inverses of its diagonal blocks, no other part of U^-1 (whose
// computation, a triangular inverse, took 5.6 ms of the c2 layer's 70).
//
// Steps: H; its factor (one launch per 32 columns); then the sequential loop over blocks, two launches each:
//     M_W of block i's current weights, Alg. 1 -> T_i (rounded to BF16);  Hbar = (T_i U_ii)(T_i U_ii)^T, R = inverse of its
//       reverse Cholesky factor (R^T R = inv(Hbar));  inv(T_i);   beside it errors G U onto later S
//     per output channel: transformed weights, GPTQ subroutine (32 steps of quantize at a static group scale,
//     err = (w - q)/R[r][r], w[r'] -= err R[r][r']), G_i, and block i + 1: S += G_i U, current weights, M_W.
// c2 (4096 calibration tokens, 4096 -> 6144): 70.4 -> 12.2 ms, of which the loop 128 x 61 us, the factor 3.0 ms and H 1.3.
// Summation orders are fixed (no atomics), so the result is reproducible.
#include <algorithm>

#include "weight_mfma.hpp"
#include "wush_block.hpp"
#include "wush_kernels.hpp"

namespace wush {

namespace {

using wm::Block32;
using wm::v4d;

// Eight consecutive doubles (64 bytes, 16-byte aligned).
__device__ __forceinline__ void load8(const double* __restrict__ p, double (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const v2d v = reinterpret_cast<const v2d*>(p)[i];
    x[2 * i] = v[0];
    x[2 * i + 1] = v[1];
  }
}
__device__ __forceinline__ void store8(double* __restrict__ p, const double (&x)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) reinterpret_cast<v2d*>(p)[i] = (v2d){x[2 * i], x[2 * i + 1]};
}

// ------------------------------------------------------------------ Hessian
// H = Xc^T Xc / M, 64 x 64 tile per workgroup, tiles on or above the diagonal (the factorization reads no other).
// Products of BF16 values are exact.  Arithmetic bound (K^2 M multiply-adds): FP64 MFMA, a wavefront per 32 x 32
// quarter, operands widened as they come out of LDS; row pitch 80 floats: the four rows of an operand read hit
// distinct banks.  The tiles are numbered along the triangle and every XCD takes a contiguous run of them: as a square grid whose lower
// half leaves at once, an XCD got up to a tenth more of them than the mean.  Two LDS stages, one barrier per 32 rows, with the fetches left in
// flight.  4096 x 4096: 1.37 ms = 50 TFLOP/s (square grid 1.75, one stage 1.40; the MFMAs alone 67 TFLOP/s; operands
// staged as the upper words of their FP64 values, without a conversion behind LDS: 1.54).
__global__ __launch_bounds__(256) void gptq_hessian_kernel(const uint16_t* __restrict__ X, int64_t ldx, int Mc, int K,
                                                           double* __restrict__ H, int* __restrict__ status) {
  if (blockIdx.x == 0 && threadIdx.x < 4) status[threadIdx.x] = 0;   // later kernels set it
  const int id = xcd_contiguous_id((int)blockIdx.x, (int)gridDim.x);
  int tj = (int)((sqrt(8.0 * (double)id + 1.0) - 1.0) * 0.5);
  while ((int64_t)tj * (tj + 1) / 2 > id) --tj;
  while ((int64_t)(tj + 1) * (tj + 2) / 2 <= id) ++tj;
  const int ti = id - (int)((int64_t)tj * (tj + 1) / 2);
  __shared__ __attribute__((aligned(16))) float side_a[2][32][80], side_b[2][32][80];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
  const int wr = 32 * (wave >> 1), wc = 32 * (wave & 1);
  v4d acc[2][2] = {};
  const int lr = threadIdx.x >> 3, lc = (threadIdx.x & 7) * 8;   // one 16-byte chunk per thread and side
  const int ca = 64 * ti + lc, cb = 64 * tj + lc;
  v4u ra, rb;
  auto fetch = [&](int m0) {
    const v4u zero = {0, 0, 0, 0};
    const bool row = m0 + lr < Mc;
    ra = row && ca < K ? *reinterpret_cast<const v4u*>(X + (int64_t)(m0 + lr) * ldx + ca) : zero;
    rb = row && cb < K ? *reinterpret_cast<const v4u*>(X + (int64_t)(m0 + lr) * ldx + cb) : zero;
  };
  auto widen = [&](const v4u& raw, float* dst) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      dst[2 * i] = __uint_as_float(raw[i] << 16);
      dst[2 * i + 1] = __uint_as_float(raw[i] & 0xFFFF0000u);
    }
  };
  fetch(0);
  widen(ra, &side_a[0][lr][lc]);
  widen(rb, &side_b[0][lr][lc]);
  fetch(32);
  lds_barrier();
  int stage = 0;
  for (int m0 = 0; m0 < Mc; m0 += 32) {
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      double a[2], b[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        a[u] = (double)side_a[stage][4 * kk + l4][wr + 16 * u + l16];
        b[u] = (double)side_b[stage][4 * kk + l4][wc + 16 * u + l16];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[v], acc[u][v], 0, 0, 0);
      if (kk == 4) {   // the other stage was read last before the barrier
        widen(ra, &side_a[stage ^ 1][lr][lc]);
        widen(rb, &side_b[stage ^ 1][lr][lc]);
        fetch(m0 + 64);
      }
    }
    lds_barrier();
    stage ^= 1;
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 64 * ti + wr + 16 * u + l4 + 4 * e, c = 64 * tj + wc + 16 * v + l16;
        if (r < K && c < K) H[(int64_t)r * K + c] = acc[u][v][e] / (double)Mc;
      }
}

// tr(H) in a fixed order, then: keep the undamped diagonal blocks (the M_X of
// every block) and add lambda tr(H)/K to the diagonal.
__global__ __launch_bounds__(256) void gptq_trace_kernel(const double* __restrict__ H, int K, double* __restrict__ tr_out) {
  __shared__ double part[256];
  double s = 0.0;
  for (int d = threadIdx.x; d < K; d += 256) s += H[(int64_t)d * K + d];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) tr_out[0] = part[0];
}

__global__ __launch_bounds__(256) void gptq_damp_kernel(double* __restrict__ H, int K, double lambda,
                                                        const double* __restrict__ tr, double* __restrict__ MX) {
  const int b = blockIdx.x;
  const double add = lambda * tr[0] / (double)K;
  for (int o = threadIdx.x; o < 1024; o += 256) {
    const int r = o >> 5, c = o & 31;
    const int64_t idx = (int64_t)(32 * b + r) * K + 32 * b + c;
    const double v = H[idx];
    MX[(int64_t)b * 1024 + o] = v;
    if (r == c) H[idx] = v + add;
  }
}

// ------------------------------------------------ reverse Cholesky of Hd
// Step i (C, C - 1, ..., 1) takes block column i out of what is left of Hd: U_ki = H_ki V_ii^T and
// H_kl -= U_ki U_li^T for all k <= l < i, and, in workgroup 0, the factor U_dd, V_dd of the next diagonal block
// d = i - 1 right behind that block's update -- the chain of diagonal factors never waits for the rest, and a step is
// one launch (c2: 62 us on average as three kernels that waited for each other, now 24).  Step C only factors block C - 1.  A
// wavefront per pair (k, l); the panel products U_ki, U_li are repeated by every pair rather than fetched from
// another launch.  U goes to its own buffer: other wavefronts of the step still read H_ki.
__global__ __launch_bounds__(256) void gptq_rchol_kernel(double* __restrict__ H, double* __restrict__ U,
                                                         double* __restrict__ Vd, int K, int i, int* __restrict__ status) {
  __shared__ double Sd[32][33];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
  const int d = i - 1;
  int k = d, l = d, a_begin = wave, a_end = wave < 2 ? wave + 1 : wave;   // workgroup 0: one 16-row half per wavefront
  if (blockIdx.x > 0) {
    const int64_t idx = ((int64_t)blockIdx.x - 1) * 4 + wave;
    if (idx >= (int64_t)i * (i + 1) / 2 - 1) return;   // wave-uniform; no barrier follows in these workgroups
    l = (int)((sqrt(8.0 * (double)idx + 1.0) - 1.0) * 0.5);
    while ((int64_t)l * (l + 1) / 2 > idx) --l;
    while ((int64_t)(l + 1) * (l + 2) / 2 <= idx) ++l;
    k = (int)(idx - (int64_t)l * (l + 1) / 2);
    a_begin = 0;
    a_end = 2;
  }
  const bool update = 32 * i < K;
  if (update && a_begin < a_end) {
    Block32 v, ul;
    wm::load_block32(v, [&](int kk, int j) { return Vd[(int64_t)i * 1024 + 32 * j + kk]; }, lane);
    // U_li with its rows where the next product wants its first operand's (weight_mfma.hpp)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      double w[8], y[8] = {};
      load8(H + (int64_t)(32 * l + 8 * (l16 & 3) + 4 * t + (l16 >> 2)) * K + 32 * i + 8 * l4, w);
      wm::multiply32(v, w, y);
#pragma unroll
      for (int q = 0; q < 8; ++q) ul.m[t][q] = -y[q];
    }
    for (int a = a_begin; a < a_end; ++a) {
      const int64_t row = (int64_t)(32 * k + 16 * a + l16) * K;
      double w[8], uk[8] = {}, y[8];
      load8(H + row + 32 * i + 8 * l4, w);
      load8(H + row + 32 * l + 8 * l4, y);
      wm::multiply32(v, w, uk);
      if (k == l) store8(U + row + 32 * i + 8 * l4, uk);
      wm::multiply32(ul, uk, y);
      if (blockIdx.x > 0) {
        store8(H + row + 32 * l + 8 * l4, y);
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) Sd[16 * a + l16][8 * l4 + q] = y[q];
      }
    }
  }
  if (blockIdx.x > 0) return;
  if (!update)
    for (int o = threadIdx.x; o < 1024; o += 256) Sd[o >> 5][o & 31] = H[(int64_t)(32 * d + (o >> 5)) * K + 32 * d + (o & 31)];
  __syncthreads();
  const bool good = reverse_factor_group([&](int r, int c) { return Sd[r][c]; },
                                         [&](int r, int c, double x) { U[(int64_t)(32 * d + r) * K + 32 * d + c] = x; },
                                         [&](int r, int c, double x) { Vd[(int64_t)d * 1024 + 32 * r + c] = x; });
  if (!good && threadIdx.x == 0) atomicExch(status, 1);
}

// ------------------------------------------------------ per-block kernels
// Second moment of 32 channels over tiles of 16 rows, by the wavefronts of a workgroup: a lane brings channels
// 8 l4 ... + 7 of row l16, the tile is turned through the wavefront's own LDS area into operands whose contraction
// runs over the rows, and the three distinct 16 x 16 blocks are accumulated on the FP64 MFMA.
constexpr int kAreaDoubles = 768;    // LDS per wavefront: a 16 x 34 tile and 16 x 8 errors, at the end its three sums
struct Moment {
  v4d acc00 = {0, 0, 0, 0}, acc01 = {0, 0, 0, 0}, acc11 = {0, 0, 0, 0};
  __device__ __forceinline__ void add(const double (&x)[8], double* area, int l16, int l4) {
    store8(area + 34 * l16 + 8 * l4, x);
    wave_lds_sync();
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const double x0 = area[34 * (4 * kk + l4) + l16], x1 = area[34 * (4 * kk + l4) + 16 + l16];
      acc00 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x0, acc00, 0, 0, 0);
      acc01 = __builtin_amdgcn_mfma_f64_16x16x4f64(x0, x1, acc01, 0, 0, 0);
      acc11 = __builtin_amdgcn_mfma_f64_16x16x4f64(x1, x1, acc11, 0, 0, 0);
    }
    wave_lds_sync();
  }
  // sums of the workgroup's WAVES wavefronts in wave order -> out [kMomentSize]
  template <int WAVES>
  __device__ __forceinline__ void reduce(double* areas, int wave, int lane, double* __restrict__ out) {
    __syncthreads();
    double* mine = areas + wave * kAreaDoubles;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      mine[4 * lane + v] = acc00[v];
      mine[256 + 4 * lane + v] = acc01[v];
      mine[512 + 4 * lane + v] = acc11[v];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 768; e += 64 * WAVES) {
      double s = areas[e];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) s += areas[w * kAreaDoubles + e];
      const int el = (e & 255) >> 2, i = (el >> 4) + 4 * (e & 3), c = el & 15;   // row, column of the 16 x 16 block
      if (e >= 256 && e < 512) out[moment_beside(i, c)] = s;
      else if (c <= i) out[e < 256 ? lower16(i, c) : moment_second(i, c)] = s;
    }
  }
};

constexpr int kWarmSplits = 8;    // row splits of the moments of the original weights
constexpr int kChainFlight = 24;  // partial moments of the chain's block in flight

// Second moments of all blocks of the original weights (grid: splits of the rows x blocks), for the warm start.
__global__ __launch_bounds__(256) void gptq_moment0_kernel(const uint16_t* __restrict__ W, int64_t ldw, int N,
                                                           double* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) double areas[4 * kAreaDoubles];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
  const int b = blockIdx.y, tiles = (N + 15) / 16;
  Moment m;
  for (int t = 4 * blockIdx.x + wave; t < tiles; t += 4 * gridDim.x) {
    const int n = 16 * t + l16;
    double x[8];
    wm::widen8(*reinterpret_cast<const v4u*>(W + (int64_t)min(n, N - 1) * ldw + 32 * b + 8 * l4), x);
    if (n >= N)
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = 0.0;
    m.add(x, areas + wave * kAreaDoubles, l16, l4);
  }
  m.reduce<4>(areas, wave, lane, partial + ((int64_t)b * gridDim.x + blockIdx.x) * kMomentSize);
}

// Right singular vectors of W'^T X' of every block of the ORIGINAL weights: what the SVD inside the loop starts from.
// All blocks at once (they fill the chip), while inside the loop a block waits for its SVD alone: there the 4096 x 4096 -> 6144
// layer's blocks take 0.1 sweeps and 3.8 steps (orthogonalize_group) instead of 1.9 and 4.2; how much is left to do depends on how far a layer's
// errors move its weights' moments.
__global__ __launch_bounds__(256) void gptq_warm_kernel(const double* __restrict__ partial, int splits, int N,
                                                        const double* __restrict__ MX, double lambda, double* __restrict__ V0) {
  const int b = blockIdx.x;
  auto load = [&](int half, int e, int r, int c, int s) {
    return half ? MX[(int64_t)b * 1024 + r * 32 + c] : partial[((int64_t)b * splits + s) * kMomentSize + e];
  };
  auto finish = [&](int half, double sum) { return half ? sum : sum / (double)N; };
  __shared__ BlockShared<32> sh;
  wush_block_group<32, 1, kWarmSplits, 1>(sh, load, finish, splits, 1, lambda, nullptr, nullptr, nullptr, V0 + (int64_t)b * 1024, nullptr);
}

// What the sums S_l still lack travels in groups of kGroup blocks: S is N x K doubles, and adding every block's error to
// all of it at once made that traffic the longest part of a step (190 us at the start of the c2 layer, against a chain of
// 70).  Step i (i = kGroup q + s) brings
//   block i + 1    up to date for its own step: the errors of group q so far, before them those of group q - 1;
//   every kGroup-th later block, from kGroup (q + 1) + s on: the errors of group q - 1
// so that each block has each group's errors added once, groups in order, and the steps share the work evenly.
constexpr int kGroup = 4;
struct Pending { int l, lo, hi; };    // block l takes the errors of blocks lo ... hi - 1
__host__ __device__ inline int pending_columns(int i, int C) {
  const int q = i / kGroup, s = i % kGroup, first = kGroup * (q + 1) + s;
  const int far = q > 0 && first < C ? (C - first + kGroup - 1) / kGroup : 0;
  return (i > 0 && i + 1 < C ? 1 : 0) + far;
}
__host__ __device__ inline Pending pending_of(int i, int C, int index) {
  const int q = i / kGroup, s = i % kGroup;
  if (i > 0 && i + 1 < C) {
    if (index == 0) return {i + 1, s < kGroup - 1 && q > 0 ? kGroup * (q - 1) : kGroup * q, i};
    --index;
  }
  return {kGroup * (q + 1) + s + kGroup * index, kGroup * (q - 1), kGroup * q};
}
constexpr int kMostPending = 2 * kGroup - 2;

// Workgroup 0: Alg. 1 on (M_W of block i's current weights, M_X = diagonal block of H) -> T_i, then inv(T_i) and R, a chain of some 40 us on
// one compute unit.  The others meanwhile: S_l += sum_b G_b U_bl for the pending blocks l.  A workgroup holds its U_bl
// in LDS in operand order, its wavefronts walk tiles of 16 rows (64 bytes per lane and operand, the next tile's
// requested before this one's products); the panels G_b (the errors; block b's, whose S is used up) and S_l are [N][32].
__global__ __launch_bounds__(256) void gptq_chain_kernel(const double* __restrict__ partial, int splits, int N, int K, int i,
                                                         const double* __restrict__ MX_i, double lambda,
                                                         const double* __restrict__ V0_i, uint16_t* __restrict__ T_bits_i,
                                                         int given, const double* __restrict__ U, double* __restrict__ S,
                                                         int near_groups, int far_groups, double* __restrict__ Tinv, double* __restrict__ R,
                                                         int* __restrict__ status) {
  extern __shared__ __attribute__((aligned(16))) double smem[];   // workgroup 0: BlockShared; others [block][pair of operand registers][lane][2]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
  if (blockIdx.x == 0) {
    BlockShared<32>& sh = *reinterpret_cast<BlockShared<32>*>(smem);
    __builtin_amdgcn_s_setprio(3);   // ahead of wavefronts that may share its compute unit
    const int t = threadIdx.x, i0 = 16 * (wave >> 1), j0 = 16 * (wave & 1);
    double u[4];                     // U_ii, fetched ahead
#pragma unroll
    for (int q = 0; q < 4; ++q) u[q] = U[(int64_t)(32 * i + (t >> 5) + 8 * q) * K + 32 * i + (t & 31)];
    auto load = [&](int half, int e, int r, int c, int s) { return half ? MX_i[r * 32 + c] : partial[(int64_t)s * kMomentSize + e]; };
    auto finish = [&](int half, double sum) { return half ? sum : sum / (double)N; };
    double (*T)[34] = sh.scratch[1], (*Um)[34] = sh.scratch[2], (*B)[34] = sh.scratch[0], (*Hb)[34] = sh.LX;
    if (!given) {
      wush_block_group<32, 0, kChainFlight, 1>(sh, load, finish, splits, 1, lambda, V0_i, T_bits_i, nullptr, nullptr, status);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) T[(t >> 5) + 8 * q][t & 31] = (double)bf16_bits_to_f32(T_bits_i[t + 256 * q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) Um[(t >> 5) + 8 * q][t & 31] = u[q];
    __syncthreads();
    // R = the inverse of the reverse factor of Hbar = B B^T, B = T_i U_ii, and inv(T_i) = U_ii B^T inv(Hbar) = (U_ii B^T R^T) R, which
    // squares the condition of B, and a Newton step X (2 I - T_i X) or two, which bring it back; should they not start close
    // enough, by elimination.  (Elimination always, beside R's: 1200 cycles a step of 32, 16 us a block.)
    const v4d zero = {0, 0, 0, 0};
    auto put = [&](double (*m)[34], const v4d& x) {
#pragma unroll
      for (int v = 0; v < 4; ++v) m[i0 + l4 + 4 * v][j0 + l16] = x[v];
    };
    double (*Q)[34] = sh.A, (*Rm)[34] = Um, (*Z)[34] = B;
    put(B, product_tile<32, true>(T, i0, Um, j0, zero));
    __syncthreads();
    put(Hb, product_tile<32>(B, i0, B, j0, zero));
    put(Q, product_tile<32>(Um, i0, B, j0, zero));
    __syncthreads();
    if (t < 8) sh.votes[t] = 0;
    const bool definite = reverse_factor_group([&](int r, int c) { return Hb[r][c]; }, [](int, int, double) {},
                                               [&](int r, int c, double x) {
                                                 Rm[r][c] = x;
                                                 R[32 * r + c] = x;
                                               });
    if (!definite && t == 0) atomicExch(status, 1);
    __syncthreads();
    put(Z, product_tile<32>(Q, i0, Rm, j0, zero));
    __syncthreads();
    double (*X)[34] = sh.LW, (*E)[34] = sh.LX, (*other)[34] = sh.A;
    put(X, product_tile<32, true>(Z, i0, Rm, j0, zero));
    __syncthreads();
    bool close = false;
    for (int newton = 0; newton < 4 && !close; ++newton) {
      v4d e = product_tile<32, true>(T, i0, X, j0, zero);
      bool far = false, lost = false;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double one = i0 + l4 + 4 * v == j0 + l16 ? 1.0 : 0.0, off = fabs(e[v] - one);
        far |= off > 1e-9;           // squared by the step, 32 terms at most: far below rounding
        lost |= !(off < 1e-2);
        e[v] = 2.0 * one - e[v];
      }
      put(E, e);
      if (far) sh.votes[newton] = 1;
      if (lost) sh.votes[4 + newton] = 1;
      __syncthreads();
      if (sh.votes[4 + newton]) break;
      close = !sh.votes[newton];
      const v4d x = product_tile<32, true>(X, i0, E, j0, zero);
      if (close) {
#pragma unroll
        for (int v = 0; v < 4; ++v) Tinv[32 * (i0 + l4 + 4 * v) + j0 + l16] = x[v];
      } else {
        put(other, x);
        double (*swap)[34] = X;
        X = other;
        other = swap;
        __syncthreads();
      }
    }
    if (!close) {
      const bool good = invert_block_group<32>([&](int r, int c) { return T[r][c]; }, [&](int r, int c, double v) { Tinv[32 * r + c] = v; });
      if (!good && t == 0) atomicExch(status, 1);
    }
    return;
  }
  // the first near_groups workgroups share the rows of block i + 1, every far_groups behind them those of a later one
  const int id = (int)blockIdx.x - 1;
  const bool near = id < near_groups;
  const int row_groups = near ? near_groups : far_groups, g = near ? id : (id - near_groups) % far_groups;
  const Pending job = pending_of(i, K >> 5, near ? 0 : (near_groups > 0 ? 1 : 0) + (id - near_groups) / far_groups);
  const int nb = job.hi - job.lo;
  for (int b = wave; b < nb; b += 4) {
    Block32 u;
    wm::load_block32(u, [&](int k, int j) { return U[(int64_t)(32 * (job.lo + b) + k) * K + 32 * job.l + j]; }, lane);
#pragma unroll
    for (int p = 0; p < 8; ++p)
      *reinterpret_cast<v2d*>(&smem[((b * 8 + p) * 64 + lane) * 2]) = (v2d){u.m[p >> 2][2 * (p & 3)], u.m[p >> 2][2 * (p & 3) + 1]};
  }
  __syncthreads();
  const int64_t panel = (int64_t)N * 32;
  double* sum = S + job.l * panel;
  const double* err = S + job.lo * panel;
  const int tiles = (N + 15) / 16, stride = 4 * row_groups;
  const bool fresh = job.lo == 0;    // the block's first errors: nothing to add to
  auto at = [&](int t) { return (int64_t)min(16 * t + l16, N - 1) * 32 + 8 * l4; };
  int t = 4 * g + wave;
  if (t >= tiles) return;
  // fetched one product ahead: the next block's errors, behind the last the next tile's first errors and sums
  double en[8], sn[8] = {};
  load8(err + at(t), en);
  if (!fresh) load8(sum + at(t), sn);
  for (; t < tiles; t += stride) {
    const int64_t here = at(t), next = at(min(t + stride, tiles - 1));
    double s[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) s[q] = sn[q];
    if (!fresh) load8(sum + next, sn);   // other rows than this tile's, except behind the last one, where it is not used
    for (int b = 0; b < nb; ++b) {
      double e[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) e[q] = en[q];
      load8(b + 1 < nb ? err + (b + 1) * panel + here : err + next, en);
      Block32 u;
#pragma unroll
      for (int p = 0; p < 8; ++p) {
        const v2d v = *reinterpret_cast<const v2d*>(&smem[((b * 8 + p) * 64 + lane) * 2]);
        u.m[p >> 2][2 * (p & 3)] = v[0];
        u.m[p >> 2][2 * (p & 3) + 1] = v[1];
      }
      wm::multiply32(u, e, s);
    }
    if (16 * t + l16 < N) store8(sum + here, s);
  }
}

// One element of the GPTQ subroutine: code of v at the group's scale (in float range: through the hardware converts, which
// agree with FP64 comparisons, f64_to_f32_sticky), its value.
template <bool SAFE>
__device__ __forceinline__ uint32_t gptq_code(double v, float sc, double inv_scale, double scale, double& value) {
  if constexpr (SAFE) {
    const uint32_t code = pack2_e2m1<0>(0, f64_to_f32_sticky(v), 0.0f, sc) & 0xFu;
    typedef float v2f __attribute__((ext_vector_type(2)));
    const v2f q = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(code, sc, 0);
    value = (double)q[0];
    return code;
  } else {
    const uint32_t sign = (uint32_t)(((uint64_t)__double_as_longlong(v)) >> 63);
    const uint32_t code = e2m1_code_f64(fabs(v) * inv_scale);
    const double mag = (code < 4 ? 0.5 * (double)code : (code == 4 ? 2.0 : (code == 5 ? 3.0 : (code == 6 ? 4.0 : 6.0)))) * scale;
    value = sign ? -mag : mag;
    return (sign << 3) | code;
  }
}

struct RowOperands {            // in LDS, the same for the workgroup
  double r[32][34];             // R
  double rinv[32];              // 1 / R[r][r]
};

// The GPTQ subroutine on 16 rows: lane (l16, l4) holds channels 8 l4 ... + 7 of row l16 (y).  The channels go in index
// order: the lanes l4 = g take their eight steps among themselves, hand the eight errors to the lanes with later channels
// through LDS, and those subtract them in the same order.  The quotient (v - q) / R[r][r] from the correctly rounded
// reciprocal, corrected once, is the correctly rounded one (Markstein).  err holds 16 x 8 doubles.
template <bool SAFE>
__device__ __forceinline__ uint32_t gptq_subroutine(double (&y)[8], double (&dq)[8], int byte, const RowOperands& op,
                                                    double* err, int l16, int l4) {
  const float sc = scale_as_f32(byte);
  const double inv_scale = __longlong_as_double((int64_t)(uint64_t)(1023 + 127 - byte) << 52);   // 2^(127-byte)
  const double scale = __longlong_as_double((int64_t)(uint64_t)(1023 - 127 + byte) << 52);       // 2^(byte-127)
  uint32_t word = 0;
  for (int g = 0; g < 4; ++g) {
    if (l4 == g) {
#pragma unroll
      for (int s = 0; s < 8; ++s) {
#pragma clang fp contract(off)   // the reference subtracts a rounded product: no fused multiply-add here
        const int r = 8 * g + s;
        const double v = y[s];
        word |= gptq_code<SAFE>(v, sc, inv_scale, scale, dq[s]) << (4 * s);
        const double a = v - dq[s], q0 = a * op.rinv[r];
        const double e = __builtin_fma(__builtin_fma(-op.r[r][r], q0, a), op.rinv[r], q0);
        err[8 * l16 + s] = e;
#pragma unroll
        for (int q = s + 1; q < 8; ++q) {
          const double p = e * op.r[r][8 * g + q];
          y[q] = y[q] - p;
        }
      }
    }
    wave_lds_sync();
    if (l4 > g) {
      double e[8];
      load8(err + 8 * l16, e);
#pragma unroll
      for (int s = 0; s < 8; ++s) {
#pragma clang fp contract(off)
        double rr[8];
        load8(&op.r[8 * g + s][8 * l4], rr);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const double p = e[s] * rr[q];
          y[q] = y[q] - p;
        }
      }
    }
    wave_lds_sync();
  }
  return word;
}

constexpr int kRowWaves = 8;
struct RowShared {
  double areas[kRowWaves * kAreaDoubles];
  RowOperands op;
  double inv[32][33], tm[32][33], u[32][33], v[32][33];   // inv(T_i), T_i, U_{i,i+1}, -V_{i+1,i+1}
};

// Block i of all rows (i = -1: none, the first block's moment only): from the current weights to codes, scale and G_i =
// (deq T)_i - W_i, and on to block i + 1: S += G_i U_{i,i+1} (S_{i+1} is complete then), current weights W - S V, their
// moment.  Everything of a row stays in the four lanes that hold it (weight_mfma.hpp); a wavefront takes 16 rows at a time.
// A chain as well: 32 quantize-and-divide steps of some 170 cycles and five block products.  c2: 19 us; as three
// kernels (moment, quantize with a thread per row, propagate) 90 us.
// The errors G_i take the place of S_i, which block i has used up.
__global__ __launch_bounds__(64 * kRowWaves) void gptq_rows_kernel(
    const uint16_t* __restrict__ W, int64_t ldw, int N, int K, int i, double* __restrict__ S, const double* __restrict__ U,
    const double* __restrict__ Vd, const uint16_t* __restrict__ T, const double* __restrict__ Tinv,
    const double* __restrict__ R, int rule, int tiled, uint8_t* __restrict__ Wq, uint8_t* __restrict__ Ws,
    double* __restrict__ current, double* __restrict__ partial) {
  extern __shared__ __attribute__((aligned(16))) double smem[];
  RowShared& sh = *reinterpret_cast<RowShared*>(smem);
  RowOperands& op = sh.op;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
  const int next = i + 1, C = K >> 5, tiles = (N + 15) / 16;
  double* area = sh.areas + wave * kAreaDoubles;
  // what the first rows need is on its way while the matrices are brought to LDS
  v4u raw, raw_next;
  double s[8], w[8];
  auto fetch = [&](int t) {
    const int64_t nc = min(16 * t + l16, N - 1);
    const uint16_t* wrow = W + nc * ldw + 8 * l4;
    raw = *reinterpret_cast<const v4u*>(wrow + 32 * max(i, 0));
    raw_next = *reinterpret_cast<const v4u*>(wrow + 32 * min(next, C - 1));
    if (i > 0) {
      load8(current + nc * 32 + 8 * l4, w);
      if (next < C) load8(S + ((int64_t)next * N + nc) * 32 + 8 * l4, s);
    }
  };
  fetch(kRowWaves * blockIdx.x + wave);
  if (i >= 0) {
    constexpr int kPer = 1024 / (64 * kRowWaves);
    double r[kPer], inv[kPer], u[kPer], v[kPer], rinv = 0.0;
    uint16_t tm[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int o = threadIdx.x + 64 * kRowWaves * q;
      r[q] = R[o];
      inv[q] = Tinv[o];
      tm[q] = T[o];
      u[q] = U[(int64_t)(32 * i + (o >> 5)) * K + 32 * min(next, C - 1) + (o & 31)];
      v[q] = Vd[(int64_t)min(next, C - 1) * 1024 + o];
    }
    if (threadIdx.x < 32) rinv = R[33 * threadIdx.x];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int o = threadIdx.x + 64 * kRowWaves * q, k = o >> 5, j = o & 31;
      op.r[k][j] = r[q];
      sh.inv[k][j] = inv[q];
      sh.tm[k][j] = (double)bf16_bits_to_f32(tm[q]);
      sh.u[k][j] = u[q];
      sh.v[k][j] = -v[q];
    }
    if (threadIdx.x < 32) op.rinv[threadIdx.x] = 1.0 / rinv;
    lds_barrier();
  }
  // y += w M, M one of the four matrices in LDS (in registers they would take 128 of a lane's 256)
  auto multiply = [&](const double (*m)[33], const double (&w)[8], double (&y)[8]) {
    Block32 b;
    wm::load_block32(b, [&](int k, int j) { return m[k][j]; }, lane);
    wm::multiply32(b, w, y);
  };
  Moment m;
  for (int t = kRowWaves * blockIdx.x + wave; t < tiles; t += kRowWaves * gridDim.x) {
    const int n = 16 * t + l16;
    const int64_t at = (int64_t)min(n, N - 1) * 32 + 8 * l4;
    if (t != kRowWaves * (int)blockIdx.x + wave) fetch(t);
    double wn[8];   // current weights of block i + 1
    if (i >= 0) {
      double y[8] = {}, dq[8], g[8];
      wm::widen8(raw, g);
      if (i == 0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          w[q] = g[q];
          s[q] = 0.0;
        }
      }
      multiply(sh.inv, w, y);
      // static group scale: taken before any update
      float amax = 0.0f;
#pragma unroll
      for (int q = 0; q < 8; ++q) amax = fmaxf(amax, fabsf(f64_to_f32_sticky(y[q])));
      amax = wm::max_xor32(wm::max_xor16(amax));
      int byte = scale_byte_f32(amax, rule);
      uint32_t word;
      if (!__any(byte < kSafeByteLo || byte > kSafeByteHi)) {
        word = gptq_subroutine<true>(y, dq, byte, op, area + 16 * 34, l16, l4);
      } else {
        double am = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) am = fmax(am, fabs(y[q]));
        wm::PairF64 p = wm::pair16(am, am);
        p = wm::pair32(fmax(p.first, p.second));
        byte = scale_byte_f64(fmax(p.first, p.second), rule);
        word = gptq_subroutine<false>(y, dq, byte, op, area + 16 * 34, l16, l4);
      }
      if (n < N) {
        const int KT = K >> 8;
        uint8_t* cq = tiled ? Wq + tiled_chunk_offset(n, i, KT) : Wq + (int64_t)n * (K / 2) + 16 * i;
        *reinterpret_cast<uint32_t*>(cq + 4 * l4) = word;
        if (l4 == 0) Ws[tiled ? tiled_scale_offset(n, i, KT) : (int64_t)n * C + i] = (uint8_t)byte;
      }
      if (next < C) {
#pragma unroll
        for (int q = 0; q < 8; ++q) g[q] = -g[q];
        multiply(sh.tm, dq, g);
        if (n < N) store8(S + (int64_t)i * N * 32 + at, g);
        multiply(sh.u, g, s);
        wm::widen8(raw_next, wn);
        multiply(sh.v, s, wn);
        if (n < N) store8(current + at, wn);
      }
    } else {
      wm::widen8(raw, wn);
    }
    if (next < C) {
      if (n >= N)
#pragma unroll
        for (int q = 0; q < 8; ++q) wn[q] = 0.0;
      m.add(wn, area, l16, l4);
    }
  }
  if (next < C) m.reduce<kRowWaves>(sh.areas, wave, lane, partial + (int64_t)blockIdx.x * kMomentSize);
}

// Partial moments of a block: at most this many workgroups of gptq_rows_kernel.
constexpr int kMomentSplits = 64, kMomentSplitsLarge = 128;
// From this K on the Hessian's buffer, free behind the factorization, has room for the warm start (V0, its partial
// moments) and for more partial moments: (32 + 8 * 32) K + 128 * 1024 <= K^2.
constexpr int64_t kLargeK = 1024;

struct Layout {
  size_t H, U, S, MX, partial, spare, Tinv, R, Vd, current, tr, status, total;
};

Layout layout(int64_t N, int64_t K) {
  Layout L{};
  size_t off = 0;
  auto take = [&](size_t doubles) { const size_t o = off; off += (doubles * sizeof(double) + 255) / 256 * 256; return o; };
  const size_t C = (size_t)(K / 32);
  L.H = take((size_t)K * K);
  L.U = take((size_t)K * K);
  L.S = take((size_t)N * K);
  L.MX = take(C * 1024);
  L.partial = take((size_t)kMomentSplits * 1024);
  L.spare = take(1024);
  L.Tinv = take(1024);
  L.R = take(1024);
  L.Vd = take(C * 1024);
  L.current = take((size_t)N * 32);
  L.tr = take(4);
  L.status = take(4);
  L.total = off;
  return L;
}

}  // namespace

size_t gptq_prep_workspace_bytes(int64_t N, int64_t K) { return layout(N, K).total; }
size_t gptq_prep_status_offset(int64_t N, int64_t K) { return layout(N, K).status; }

#define WUSH_GPTQ_CHECK()                 \
  {                                       \
    const hipError_t e_ = hipGetLastError(); \
    if (e_ != hipSuccess) return e_;      \
  }

hipError_t launch_gptq_prep(const void* W, int64_t N, int64_t K, int64_t ldw, const void* Xc, int64_t Mc, int64_t ldx,
                            double lambda, int transform_given, int rule, int tiled, void* T_blocks, void* Wq, void* Ws,
                            void* workspace, hipStream_t st) {
  const Layout L = layout(N, K);
  char* base = static_cast<char*>(workspace);
  auto D = [&](size_t off) { return reinterpret_cast<double*>(base + off); };
  double *H = D(L.H), *U = D(L.U), *S = D(L.S), *MX = D(L.MX), *partial = D(L.partial), *Tinv = D(L.Tinv), *R = D(L.R),
         *Vd = D(L.Vd), *current = D(L.current), *tr = D(L.tr);
  int* status = reinterpret_cast<int*>(base + L.status);
  const int C = (int)(K / 32), Ki = (int)K, Ni = (int)N;
  const uint16_t* Wb = static_cast<const uint16_t*>(W);
  uint16_t* Tbits = static_cast<uint16_t*>(T_blocks);

  const int64_t t64 = (K + 63) / 64;
  gptq_hessian_kernel<<<(unsigned)(t64 * (t64 + 1) / 2), 256, 0, st>>>((const uint16_t*)Xc, ldx, (int)Mc, Ki, H, status);
  WUSH_GPTQ_CHECK()
  gptq_trace_kernel<<<1, 256, 0, st>>>(H, Ki, tr);
  WUSH_GPTQ_CHECK()
  gptq_damp_kernel<<<C, 256, 0, st>>>(H, Ki, lambda, tr, MX);
  WUSH_GPTQ_CHECK()
  for (int i = C; i >= 1; --i) {
    const int64_t pairs = i < C ? (int64_t)i * (i + 1) / 2 - 1 : 0;
    gptq_rchol_kernel<<<(unsigned)(1 + (pairs + 3) / 4), 256, 0, st>>>(H, U, Vd, Ki, i, status);
    WUSH_GPTQ_CHECK()
  }
  static DynamicLdsLimit rows_lds;
  hipError_t attr = rows_lds.ensure(reinterpret_cast<const void*>(gptq_rows_kernel), (int)sizeof(RowShared));
  if (attr != hipSuccess) return attr;
  constexpr int kPendingLds = kMostPending * 1024 * (int)sizeof(double), kBlockLds = (int)sizeof(BlockShared<32>);
  constexpr int kChainLds = kPendingLds > kBlockLds ? kPendingLds : kBlockLds;
  static DynamicLdsLimit chain_lds;
  attr = chain_lds.ensure(reinterpret_cast<const void*>(gptq_chain_kernel), kChainLds);
  if (attr != hipSuccess) return attr;
  const bool large = K >= kLargeK;
  double* V0 = nullptr;
  if (large) {
    partial = H;
    if (!transform_given) {
      V0 = H + (size_t)kMomentSplitsLarge * 1024;
      double* partial0 = V0 + (size_t)C * 1024;
      gptq_moment0_kernel<<<dim3(kWarmSplits, C), 256, 0, st>>>(Wb, ldw, Ni, partial0);
      WUSH_GPTQ_CHECK()
      gptq_warm_kernel<<<C, 256, 0, st>>>(partial0, kWarmSplits, Ni, MX, lambda, V0);
      WUSH_GPTQ_CHECK()
    }
  }
  const int64_t tiles = (N + 15) / 16;
  const int64_t groups = (tiles + kRowWaves - 1) / kRowWaves, most = large ? kMomentSplitsLarge : kMomentSplits;
  const int splits = (int)(groups < most ? groups : most);
  for (int i = -1; i < C; ++i) {
    if (i >= 0) {
      // workgroup 0: T_i; the others: pending errors, one workgroup per compute unit (their LDS would let two share one), dealt out by the products
      // they have to form: block i + 1 lacks up to six blocks' errors where the others take four (as many workgroups for each: the steps of the
      // first third of the c2 layer took 44 to 61 us, by that number, where the chain itself takes 40)
      const bool near = i > 0 && i + 1 < C;
      const int far = pending_columns(i, C) - near, others = device_cu_count() - 1, most = (int)((tiles + 3) / 4);
      int near_groups = 0, far_groups = 0;
      if (near) {
        const Pending job = pending_of(i, C, 0);
        const int nb = job.hi - job.lo;
        near_groups = std::min(most, std::max(1, others * nb / (nb + kGroup * far)));
      }
      if (far > 0) far_groups = std::min(most, std::max(1, (others - near_groups) / far));
      gptq_chain_kernel<<<(unsigned)(1 + near_groups + far * far_groups), 256, kChainLds, st>>>(
          partial, splits, Ni, Ki, i, MX + (int64_t)i * 1024, lambda, V0 ? V0 + (int64_t)i * 1024 : nullptr,
          Tbits + (int64_t)i * 1024, transform_given, U, S, near_groups, far_groups, Tinv, R, status);
      WUSH_GPTQ_CHECK()
    }
    gptq_rows_kernel<<<(unsigned)splits, 64 * kRowWaves, sizeof(RowShared), st>>>(Wb, ldw, Ni, Ki, i, S, U, Vd,
                                                                  Tbits + (int64_t)(i < 0 ? 0 : i) * 1024, Tinv, R, rule, tiled,
                                                                  (uint8_t*)Wq, (uint8_t*)Ws, current, partial);
    WUSH_GPTQ_CHECK()
  }
  return hipSuccess;
}
#undef WUSH_GPTQ_CHECK

}  // namespace wush
