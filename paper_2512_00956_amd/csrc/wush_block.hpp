// FP64 pieces of the offline path shared by the RTN-case and the GPTQ-case kernels: Alg. 1 on one
// block and the inverse of one block, each by a workgroup.
#pragma once
#include "wush_device.hpp"

namespace wush {

// 1 / x for a normal x: the hardware estimate (some 2^-24) and one cubic step (a few 2^-53).
__device__ __forceinline__ double rcp_refined(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}

// a / d for a normal d, corrected to the rounded quotient (Markstein): in an elimination a / a has to be 1, or what is left of a
// singular matrix is rounding noise instead of zero.
__device__ __forceinline__ double div_refined(double a, double d) {
  const double y = rcp_refined(d), q = a * y;
  return fma(fma(-d, q, a), y, q);
}

// The value of x in another lane of the same row of 16, chosen by a DPP control word (no LDS round trip).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// Sum / maximum of x over the 16 lanes of a DPP row, the same in each of them: partner lane ^ 1, lane ^ 2
// (quad permutes), the mirrored lane of the other quad, the mirrored lane of the other half row.  Every addition has the same two
// operands in the lanes it joins; no multiplication of the caller's may be fused into the first one, or x stays unrounded on one
// side of it and rounded on the other, and the lanes get different sums.
__device__ __forceinline__ double row_sum(double x) {
#pragma clang fp contract(off)
  x += dpp_f64<0xB1>(x);    // quad_perm [1, 0, 3, 2]
  x += dpp_f64<0x4E>(x);    // quad_perm [2, 3, 0, 1]
  x += dpp_f64<0x141>(x);   // row_half_mirror: lane i <-> 7 - i
  x += dpp_f64<0x140>(x);   // row_mirror: lane i <-> 15 - i
  return x;
}
__device__ __forceinline__ double row_max(double x) {
  x = fmax(x, dpp_f64<0xB1>(x));
  x = fmax(x, dpp_f64<0x4E>(x));
  x = fmax(x, dpp_f64<0x141>(x));
  return fmax(x, dpp_f64<0x140>(x));
}
__device__ __forceinline__ int row_min(int x) {
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true));
  x = min(x, __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true));
  return min(x, __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, true));
}
__device__ __forceinline__ int row_sum_int(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, true);
  return x + __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, true);
}
__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

typedef double v2d __attribute__((ext_vector_type(2)));
typedef double v4d __attribute__((ext_vector_type(4)));

// Largest of the keys of the D lanes that hold the rows of a block (the upper lanes repeat them), in every lane.
template <int D>
__device__ __forceinline__ uint32_t row_group_max(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true));
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true));
  if constexpr (D == 32) {
    const auto s = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = max(s[0], s[1]);
  }
  return x;
}

// A pivot below 1e-290 makes a block singular (the upper word of that FP64 number).
constexpr uint32_t kPivotKey = 0x03B8F2B1u;

// Inverse of one D x D block (D = 32 or 16) by Gauss-Jordan elimination in place with partial pivoting, by a
// group of D * D / 4 threads (256 or 64; all of the workgroup).  Thread t owns row t / (D / 4), columns
// 4 (t % (D / 4)) ... + 3, in registers.  entry(r, c): element of T; store(r, c, v): element of the inverse
// (zeros if the block is singular; the result says whether it is regular).
// What bounds it is the chain of D dependent steps, so a step is one barrier: every thread publishes its
// elements (two LDS buffers in turn), and behind the barrier reads the pivot column, the pivot row and its own
// factor.  Rows are not swapped: pos = the position the row would have after the swaps.  Pivot candidates are
// compared by their upper words less 5 bits (15 fraction bits: enough for a pivot), which those 5 bits, the first position,
// make unique; a singular block is found at the end.  128 blocks of 32 x 32: 14 us against 91 us for one wavefront that swapped
// rows in LDS and synchronized per row.
template <int D, class EntryFn, class StoreFn>
__device__ __forceinline__ bool invert_block_group(EntryFn entry, StoreFn store) {
  static_assert(D == 32 || D == 16, "block size");
  constexpr int kTpr = D / 4;                      // threads per row
  __shared__ __attribute__((aligned(16))) double buf[2][D][D + 2];
  __shared__ int pivot_row[D];
  const int t = threadIdx.x, r = t / kTpr, c0 = 4 * (t % kTpr);
  const int lane = t & 63, row = lane % D;         // the row whose pivot candidate this lane looks at
  double a[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = entry(r, c0 + i);
  int pos = row;
  uint32_t least = ~0u, most = 0;
  for (int p = 0; p < D; ++p) {
    double (*b)[D + 2] = buf[p & 1];
    *reinterpret_cast<v2d*>(&b[r][c0]) = (v2d){a[0], a[1]};
    *reinterpret_cast<v2d*>(&b[r][c0 + 2]) = (v2d){a[2], a[3]};
    __syncthreads();
    const double cand = b[row][p], f = b[r][p];
    const uint32_t mag = (uint32_t)((uint64_t)__double_as_longlong(cand) >> 32) & 0x7FFFFFFFu;
    const uint32_t key = pos >= p ? (mag & ~31u) | (31u - (uint32_t)pos) : 0u;
    const uint32_t best = row_group_max<D>(key);
    const int idx = __builtin_ctzll(__ballot(key == best) | (1ull << (D - 1)));   // never past the rows
    least = min(least, best);
    most = max(most, best);
    const double inv_piv = rcp_refined(readlane_f64(cand, idx));
    const v2d r0 = *reinterpret_cast<const v2d*>(&b[idx][c0]), r1 = *reinterpret_cast<const v2d*>(&b[idx][c0 + 2]);
    const int ipos = 31 - (int)(best & 31u);
    if (row == idx) pos = p;
    else if (pos == p) pos = ipos;
    if (t == 0) pivot_row[p] = idx;
    const double prow[4] = {r0[0], r0[1], r1[0], r1[1]};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      // column p of what was T becomes the column of the inverse that the pivot row stands for
      const double q = c0 + i == p ? inv_piv : prow[i] * inv_piv;
      const double old = c0 + i == p ? 0.0 : a[i];
      a[i] = r == idx ? q : old - f * q;
    }
  }
  __syncthreads();
  const bool good = (least & ~31u) >= (kPivotKey & ~31u) && most < 0x7FF00000u;   // the same in every thread
  const int rpos = good ? __shfl(pos, r, 64) : r;
#pragma unroll
  for (int i = 0; i < 4; ++i) store(rpos, good ? pivot_row[c0 + i] : c0 + i, good ? a[i] : 0.0);
  return good;
}

// x / root from the root's reciprocal, corrected.
__device__ __forceinline__ double over_root(double x, double root, double inv) {
  const double q = x * inv;
  return fma(fma(-root, q, x), inv, q);
}

// Reverse Cholesky factor of a symmetric positive definite 32 x 32 S and its inverse, by 256 threads: S = U U^T with
// U upper triangular, V = U^-1, from the elimination of [S | I] row by row from the last: with d the diagonal entry
// of row j of what is left, row j over sqrt(d) is column j of U (left half) and row j of V (right half), and a row
// r < j loses row j times its own entry over d -- which is row j's entry r, S being symmetric.  Thread t owns row
// t / 8, columns 8 (t % 8) ... + 7 of the 64.  Two rows per barrier: j and j - 1 go out together, and every thread takes row j off its part of
// row j - 1 by itself (one row per barrier: 520 cycles a row, most of them the way through LDS).  Returns false if S is not positive
// definite (the same in every thread).
template <class EntryFn, class StoreUFn, class StoreVFn>
__device__ __forceinline__ bool reverse_factor_group(EntryFn entry, StoreUFn store_u, StoreVFn store_v) {
  __shared__ __attribute__((aligned(16))) double rowb[2][2][64];
  const int t = threadIdx.x, r = t >> 3, c0 = 8 * (t & 7);
  double a[8], diag = 1.0;
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = c0 < 32 ? entry(r, c0 + i) : (c0 - 32 + i == r ? 1.0 : 0.0);
  bool good = true;
  for (int j = 31; j > 0; j -= 2) {
    double (*rows)[64] = rowb[(j >> 1) & 1];
    if ((r | 1) == j) {
#pragma unroll
      for (int i = 0; i < 8; i += 2) *reinterpret_cast<v2d*>(&rows[r & 1][c0 + i]) = (v2d){a[i], a[i + 1]};
    }
    __syncthreads();
    const double *hi = rows[1], *lo = rows[0];         // rows j and j - 1
    double x[8], y[8];
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      const v2d u = *reinterpret_cast<const v2d*>(&hi[c0 + i]), v = *reinterpret_cast<const v2d*>(&lo[c0 + i]);
      x[i] = u[0];
      x[i + 1] = u[1];
      y[i] = v[0];
      y[i + 1] = v[1];
    }
    const double beside = hi[j - 1], hi_r = hi[r], lo_r = lo[r];
    double d1 = hi[j];
    if (!(d1 > 0.0)) { good = false; d1 = 1.0; }
    const double g = div_refined(beside, d1), f1 = r < j ? div_refined(hi_r, d1) : 0.0;
    double d0 = fma(-g, beside, lo[j - 1]);
    if (!(d0 > 0.0)) { good = false; d0 = 1.0; }
    const double f0 = r < j - 1 ? div_refined(fma(-g, hi_r, lo_r), d0) : 0.0;
    if (r == j) diag = d1;
    if (r == j - 1) diag = d0;
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = fma(-f0, fma(-g, x[i], y[i]), fma(-f1, x[i], a[i]));
  }
  const double root = sqrt(diag), inv = 1.0 / root;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (c0 < 32) store_u(c0 + i, r, c0 + i <= r ? over_root(a[i], root, inv) : 0.0);
    else store_v(r, c0 - 32 + i, c0 - 32 + i >= r ? over_root(a[i], root, inv) : 0.0);
  }
  return good;
}

// One sweep of one-sided Jacobi over the columns of A (A[column][row], D = 32 or 16) by the first 4 D of a workgroup's 8 D threads (for
// D = 32 all of them call it, the barriers are everybody's; for D = 16 the first wavefront alone).
//
// A sweep is D - 1 rounds of D / 2 rotations, each round waiting for the one before.  With 16 lanes per column pair and a round trip
// through LDS and a barrier per round it took 850 cycles a round: some 60 instructions of 4 cycles, 16 the square roots and
// reciprocals, on the chain or not, the round trip, the barrier.  So:
//   * A slot of 16 lanes takes four columns, two blocks of two, and turns all four pairs between the blocks before the columns go
//     back to LDS: two rounds per round trip, one more trip per sweep for the pairs inside the blocks.
//   * The two pairs of a round are computed side by side: a lane holds D / 16 rows of all four columns and adds up both scalar
//     products; each half of the slot gathers and evaluates one pair ("own") and hands cosine and sine to the other half, so
//     that a wavefront's 60 instructions serve eight pairs instead of four.  One wavefront for all (four rows per lane) is slower: it
//     is the issue of instructions that bounds that.
// (x1, y1) is the own pair of a lane's half, (x2, y2) the other half's; the second round of a trip pairs x1 with y2.
// 32 x 32 blocks: some 650 cycles a round with the sweep's norms.
template <int D>
__device__ __forceinline__ void jacobi_sweep(double (*A)[D + 2], double* norm2) {
  constexpr int NT = 8 * D, R = D / 16, B = D / 2;
  const int t = threadIdx.x, slot = t / 16, l = t % 16;
  const bool hi = l >= 8, active = t < 4 * D;
  auto sync = [&]() {
    if constexpr (D == 32) __syncthreads();
    else wave_lds_sync();
  };
  typedef double rows_t[R];
  auto load = [&](rows_t& v, int c) {
    const double* p = &A[0][0] + __umul24(c, D + 2) + R * l;
    if constexpr (R == 2) {
      const v2d w = *reinterpret_cast<const v2d*>(p);
      v[0] = w[0];
      v[1] = w[1];
    } else {
      v[0] = p[0];
    }
  };
  auto store = [&](const rows_t& v, int c) {
    double* p = &A[0][0] + __umul24(c, D + 2) + R * l;
    if constexpr (R == 2) *reinterpret_cast<v2d*>(p) = (v2d){v[0], v[1]};
    else p[0] = v[0];
  };
  auto dot = [&](const rows_t& a, const rows_t& b) {
    double s = a[0] * b[0];
    if constexpr (R == 2) s = fma(a[1], b[1], s);
    return s;
  };
  double nx, ny;                                       // squared norms of the own pair
  // The rotation by the angle of smaller magnitude that makes two columns orthogonal:
  // tan(2 theta) = 2 ga / (be - al), |theta| <= pi / 4.  With h = hypot(be - al, 2 ga):
  // cos^2 = (1 + |be - al| / h) / 2 and tan = (|ga| / h) / cos^2.  The tangent only has to be about
  // right (the hardware's estimates, some 2^-24: the next sweep sees what is left); that cos and sin form a
  // rotation to FP64 accuracy is the last reciprocal square root's business, refined by a cubic step.
  auto rotate = [&](rows_t& x1, rows_t& y1, rows_t& x2, rows_t& y2) {
    double ga = dot(x1, y1);
    {
#pragma clang fp contract(off)
      ga += dpp_f64<0x140>(dot(x2, y2));               // row_mirror: the other half's partial sums of this half's pair
      ga += dpp_f64<0xB1>(ga);
      ga += dpp_f64<0x4E>(ga);
      ga += dpp_f64<0x141>(ga);
    }
    const double dd = ny - nx, ab = nx * ny, gg = ga * ga, ga2 = ga + ga;
    const double ih = __builtin_amdgcn_rsq(fma(ga2, ga2, dd * dd));
    const double c2 = fma(0.5 * fabs(dd), ih, 0.5);
    double tn = ga * ih * __builtin_amdgcn_rcp(c2);
    tn = __longlong_as_double(__double_as_longlong(tn) ^ (__double_as_longlong(dd) & (1ll << 63)));
    tn = gg > 1e-30 * ab ? tn : 0.0;                   // |ga| <= 1e-15 sqrt(al be): left alone
    const double x = fma(tn, tn, 1.0);
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    const double cs = fma(y * e, fma(e, 0.375, 0.5), y), sn = tn * cs;
    const double cp = dpp_f64<0x140>(cs), sp = dpp_f64<0x140>(sn);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const double a = fma(-sn, y1[i], cs * x1[i]);
      y1[i] = fma(sn, x1[i], cs * y1[i]);
      x1[i] = a;
      const double b = fma(-sp, y2[i], cp * x2[i]);
      y2[i] = fma(sp, x2[i], cp * y2[i]);
      x2[i] = b;
    }
    nx = fma(-tn, ga, nx);
    ny = fma(tn, ga, ny);
  };
  // squared norms of the columns: computed once a sweep, updated by the rotations in between (they only
  // decide angles, so the updates' cancellation costs no accuracy of U)
  constexpr int kGroups = D == 32 ? NT / 16 : 4;
  for (int c = slot; c < D; c += kGroups) {
    rows_t v;
    load(v, c);
    const double n2 = row_sum(dot(v, v));
    if (l == 0) norm2[c] = n2;
  }
  sync();
  rows_t x1, y1, x2, y2;
  int cx, cy;                                        // columns of the own pair
  auto fetch = [&](int ax, int ay, int bx, int by) { // low half: pair (ax, ay), high half: pair (bx, by)
    cx = hi ? bx : ax;
    cy = hi ? by : ay;
    load(x1, cx);
    load(y1, cy);
    load(x2, hi ? ax : bx);
    load(y2, hi ? ay : by);
    nx = norm2[cx];
    ny = norm2[cy];
  };
  auto leave = [&](int ox, int oy, const rows_t& yo, const rows_t& yp) {   // the other pair's columns; the own pair's second, the other's
    store(x1, cx);
    store(yo, cy);
    store(x2, ox);
    store(yp, oy);
    norm2[cx] = nx;                                  // the same from every lane of the half
    norm2[cy] = ny;
  };
  // the pair inside every block
  if (active) {
    fetch(4 * slot, 4 * slot + 1, 4 * slot + 2, 4 * slot + 3);
    rotate(x1, y1, x2, y2);
    leave(hi ? 4 * slot : 4 * slot + 2, hi ? 4 * slot + 1 : 4 * slot + 3, y1, y2);
  }
  sync();
  // the blocks against each other, circle method: position 0 fixed, the other B - 1 rotate
  int p = slot, q = B - 1 - slot;
  for (int rnd = 0; rnd < B - 1; ++rnd) {
    if (active) {
      fetch(2 * p, 2 * q, 2 * p + 1, 2 * q + 1);
      rotate(x1, y1, x2, y2);
      ny = dpp_f64<0x140>(ny);                       // the halves swap their second columns
      cy ^= 1;
      rotate(x1, y2, x2, y1);
      leave(cx ^ 1, cy ^ 1, y2, y1);
      p = slot == 0 ? 0 : (p == B - 1 ? 1 : p + 1);
      q = q == B - 1 ? 1 : q + 1;
    }
    sync();
  }
}

// Tile (rows x0 ..., columns y0 ...) of X Y^T, added to acc, on the FP64 MFMA (16 x 16 x 4): a lane's operands are D / 4 consecutive
// elements of row l16 of either matrix; accumulator v is element (x0 + l4 + 4 v, y0 + l16).  Stored across == true: Y instead of Y^T.
template <int D, bool ACROSS = false>
__device__ __forceinline__ v4d product_tile(const double (*X)[D + 2], int x0, const double (*Y)[D + 2], int y0, v4d acc) {
  constexpr int kPer = D / 4;
  const int l16 = threadIdx.x & 15, k0 = kPer * ((threadIdx.x & 63) >> 4);
  double x[kPer], y[kPer];
#pragma unroll
  for (int k = 0; k < kPer; k += 2) {
    const v2d u = *reinterpret_cast<const v2d*>(&X[x0 + l16][k0 + k]);
    x[k] = u[0];
    x[k + 1] = u[1];
    if constexpr (ACROSS) {
      y[k] = Y[k0 + k][y0 + l16];
      y[k + 1] = Y[k0 + k + 1][y0 + l16];
    } else {
      const v2d w = *reinterpret_cast<const v2d*>(&Y[y0 + l16][k0 + k]);
      y[k] = w[0];
      y[k + 1] = w[1];
    }
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[k], y[k], acc, 0, 0, 0);
  return acc;
}

// The columns of A made orthogonal by right rotations, A V = U S (V is never needed): sweeps of Jacobi until all that is left are small
// angles, then all pairs at once.
//
// The simultaneous step: with K[i][j] = the tangent that makes columns i and j orthogonal by themselves (antisymmetric), A <- A P with
// P = exp(K) nearly, orthogonal to FP64's resolution; what it leaves is of second order in K, as behind a sweep.  Its 32 x 32 products
// are on the FP64 MFMA, a tile per wavefront: three for tangents up to 1e-5, four up to 3e-4, two more with every step of correction, 1.5 to 4 us where a
// sweep is a chain of 31 dependent rounds of 650 cycles, 8.7 us.
//   G = A^T A gives the angles;  K^2;  P = I + K + K^2 / 2, + K^3 / 6 + K^4 / 24 beyond 1e-5;  beyond 3e-4 Newton-Schulz steps
//   P <- P (3 I - P^T P) / 2 until P^T P differs from I by 2e-9 at most before the last one;  A P.
// Everything behind relies on A P having A's singular values, so a P that is not orthogonal is never applied.  What decides is the norm of K, which
// 31 tangents of one size in every row make up to 20.4 times as large as one of them: there P^T P - I is ||K||^4 / 4 = 4e-16 at 1e-5 and
// ||K||^6 / 72 = 7e-16 at 3e-4 (5e-13 with that line at 1e-3), and the correction takes one to four steps for angles as they come, but up to eight
// for such rows of 0.05 to 0.15; behind the eighth, or with an entry of P^T P - I at 0.1 or more, the step is refused and a sweep takes its place.
// Everything is graded as A's columns are (K[i][j] is about cosine x ratio of the norms), so small columns keep their relative accuracy.
// P is kept transposed, so that both operands of all products but two are read along their rows.
// It is taken up to tangents of 0.4 (blocks of the 4096 -> 6144 layer, sweeps + steps from the Cholesky factors: never 5.9 + 0, 0.003: 3.3 +
// 2.1, 0.05: 2.7 + 3.1, 0.1: 2.5 + 3.4, 0.4: 1.9 + 4.2, 0.6: 1.7 + 4.5; from a warm start 3.9 + 0, 1.3 + 2.5, 0.7 + 3.1, 0.4 + 3.4, 0.05 + 3.8, 0 + 3.8),
// at most eight times: on blocks of nearly equal singular values, where second order is not small against their distance, the sweeps end it.  (A bound:
// 28000 blocks drawn to have such values, in a model of this on the CPU, took seven at most.)
//
// End: a step or sweep that met cosines up to 1e-10 and tangents up to 1e-7 only is the last one: it turns what earlier rotations
// zeroed by a tangent times the cosines it mixes in (the ratio of the two columns' norms is in the tangent), 2 D of them per pair at
// most, and so leaves cosines of some 1e-16, and its own ones, 2^-24 of what they were.  Equal or nearly equal singular values turn by
// large angles at any cosine; there the sweeps go on until no cosine is above 1e-15.
//
// All threads of the workgroup call it (D = 16: the first wavefront does the work).  K, Q, R: scratch; votes: 8 words; cold: nothing is
// known of A's columns, so a sweep comes first.
template <int D>
__device__ __forceinline__ void orthogonalize_group(double (*A)[D + 2], double (*K)[D + 2], double (*Q)[D + 2], double (*R)[D + 2],
                                                    double* norm2, int* votes, bool cold) {
  constexpr int kTurn = 1, kSweep = 2, kMore = 4, kFourth = 8, kFix = 16, kMostFixes = 8;
  if (D == 16 && threadIdx.x >= 64) return;            // one wavefront: nobody to wait for
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, l4 = lane >> 4;
  const int i0 = D == 32 ? 16 * (wave >> 1) : 0, j0 = D == 32 ? 16 * (wave & 1) : 0;   // this wavefront's tile of every product
  auto sync = [&]() {
    if constexpr (D == 32) __syncthreads();
    else wave_lds_sync();
  };
  int round = 0;
  // the bits set by any lane, in every lane; a barrier for LDS as well
  auto vote = [&](int bits) {
    int mine = 0;
#pragma unroll
    for (int b = 1; b <= kFix; b *= 2)
      if (__any(bits & b)) mine |= b;
    if constexpr (D == 32) {
      int* v = votes + 4 * (round++ & 1);              // read by everybody before the barrier of the next vote
      if (lane == 0) v[wave] = mine;
      __syncthreads();
      mine = __builtin_amdgcn_readfirstlane(v[0] | v[1] | v[2] | v[3]);
    } else {
      wave_lds_sync();
    }
    return mine;
  };
  auto put = [&](double (*m)[D + 2], const v4d& x) {
#pragma unroll
    for (int v = 0; v < 4; ++v) m[i0 + l4 + 4 * v][j0 + l16] = x[v];
  };
  const v4d zero = {0, 0, 0, 0};
  v4d one;
#pragma unroll
  for (int v = 0; v < 4; ++v) one[v] = i0 + l4 + 4 * v == j0 + l16 ? 1.0 : 0.0;
  if (cold) {
    jacobi_sweep<D>(A, norm2);
  }
  int steps_left = 8;
  for (int pass = 0; pass < 40; ++pass) {
    const v4d G = product_tile<D>(A, i0, A, j0, zero);
    if (i0 == j0) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (l16 == l4 + 4 * v) norm2[j0 + l16] = G[v];
    }
    sync();
    const double nj = norm2[j0 + l16];
    v4d k;
    int bits = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      // tan(theta) as in jacobi_sweep's rotation of columns x = i, y = j
      const double ni = norm2[i0 + l4 + 4 * v], ga = G[v], dd = nj - ni, ab = ni * nj, gg = ga * ga, ga2 = ga + ga;
      const double ih = __builtin_amdgcn_rsq(fma(ga2, ga2, dd * dd));
      const double c2 = fma(0.5 * fabs(dd), ih, 0.5);
      double tn = ga * ih * __builtin_amdgcn_rcp(c2);
      tn = __longlong_as_double(__double_as_longlong(tn) ^ (__double_as_longlong(dd) & (1ll << 63)));
      const bool turn = one[v] == 0.0 && gg > 1e-30 * ab;
      k[v] = turn ? tn : 0.0;
      const double mag = fabs(k[v]);
      bits |= (turn ? kTurn : 0) | (mag > 0.4 ? kSweep : 0) | (turn && (gg > 1e-20 * ab || mag > 1e-7) ? kMore : 0) |
              (mag > 1e-5 ? kFourth : 0) | (mag > 3e-4 ? kFix : 0);
    }
    put(K, k);
    const int seen = vote(bits);
    if (!(seen & kTurn)) break;
    bool step = !(seen & kSweep) && steps_left-- > 0;
    if (step) {
      // Q = K^2 = -K K^T
      v4d k2 = product_tile<D>(K, i0, K, j0, zero);
      double (*P)[D + 2] = Q;                          // P^T, all along
      v4d p;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        k2[v] = -k2[v];
        p[v] = fma(0.5, k2[v], one[v] - k[v]);
      }
      if (seen & kFourth) {
        // P^T += K^2 (K^2 / 24 - K / 6); the second factor's transpose is K^2 / 24 + K / 6
        v4d m;
#pragma unroll
        for (int v = 0; v < 4; ++v) m[v] = fma(k2[v], 1.0 / 24.0, k[v] * (1.0 / 6.0));
        put(Q, k2);
        put(R, m);
        sync();
        p = product_tile<D>(Q, i0, R, j0, p);
        P = K;
      }
      put(P, p);
      sync();
      if (seen & kFix) {
        double (*other)[D + 2] = R;
        for (int fix = 0; fix < kMostFixes; ++fix) {
          v4d s = product_tile<D>(P, i0, P, j0, zero);
          bool off = false, lost = false;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double e = fabs(s[v] - one[v]);
            off |= e > 2e-9;
            lost |= !(e < 0.1);
            s[v] = fma(-0.5, s[v], 1.5 * one[v]);
          }
          put(Q, s);
          const int left = vote((off ? kMore : 0) | (lost ? kSweep : 0));
          step = !(left & kSweep) && (fix + 1 < kMostFixes || !(left & kMore));
          if (!step) break;                            // not orthogonal: a sweep instead, A is as it was
          p = product_tile<D, true>(Q, i0, P, j0, zero);
          put(other, p);
          sync();
          double (*swap)[D + 2] = P;
          P = other;
          other = swap;
          if (!(left & kMore)) break;
        }
      }
      if (step) {
        const v4d a = product_tile<D, true>(P, i0, A, j0, zero);
        sync();
        put(A, a);
        sync();
      }
    }
    if (!step) jacobi_sweep<D>(A, norm2);
    if (!(seen & kMore)) break;
  }
}

// Second moments go from kernel to kernel as the 528 entries on or below the diagonal of a symmetric 32 x 32: the lower triangle of the first
// 16 x 16 block by rows, then the block beside it (channel i of the first half, c of the second: row i, column c), then the lower
// triangle of the second diagonal block.  A partial moment is then half the bytes: what one compute unit has to fetch of 48 of them is 8 us of
// the GPTQ chain's step otherwise.
constexpr int kMomentSize = 528;
__host__ __device__ __forceinline__ int lower16(int i, int c) { return i * (i + 1) / 2 + c; }           // c <= i < 16
__host__ __device__ __forceinline__ int moment_beside(int i, int c) { return 136 + 16 * i + c; }        // entry (16 + c, i)
__host__ __device__ __forceinline__ int moment_second(int i, int c) { return 392 + lower16(i, c); }     // entry (16 + i, 16 + c)
// row and column (row >= column) of entry e of the lower triangle of a 16 x 16
__device__ __forceinline__ void lower16_at(int e, int& r, int& c) {
  r = (int)((sqrtf(8.0f * (float)e + 1.5f) - 1.0f) * 0.5f);   // 8 e + 1 is a square at c = 0
  c = e - r * (r + 1) / 2;
}

// Alg. 1 for one D x D block (D = 32, or 16 for the NVFP4 variant), by a workgroup of 8 D threads:
//   W' W'^T = M_W + lambda d^-1 tr(M_W) I,  X' X'^T likewise  (Cholesky, side by side)
//   U S V^T = W'^T X'  (orthogonalize_group on the columns; V never needed)
//   T = H S^(-1/2) U^T W'^T, singular values descending, the entry of largest
//   magnitude of every column of U positive.
// load(h, e, r, c, s): partial sum s (of S_W for h = 0, S_X for h = 1) of entry (r, c), r >= c, of the second moment, e its index in the lower
// triangle (kMomentSize's order, or lower16 for D = 16); finish(h, sum): the normalized, undamped entry, h = 0 for M_W, 1 for M_X.  T goes out as
// BF16 bits (T_bits) and, where the pointer is non-null, as FP64 before rounding (T_f64), each [D][D] row-major.  A moment
// that is not positive definite sets *status.
// V0 (may be null): an orthogonal [D][D] the SVD starts from, A V0 in place of A; U and S are the same, and a V0 close
// to the right singular vectors leaves little to do.  MODE 1 computes such a V0 in place of T (into
// V_out; the identity where the moments give none) and leaves the status alone.
//
// A block is one chain of dependent steps (2 x D columns of the factors, the SVD's sweeps and steps), so what counts is the
// latency of each.  The factors are taken by a wavefront each, without a barrier: a lane has D^2 / 64 entries of a row in registers, a
// step's pivot goes to everybody through the scalar registers, its column through LDS; the registers are shifted so that the loop stays a loop
// (unrolled over the columns it took 290 cycles a step, bound by instruction fetch).  Products are on the FP64 MFMA, a tile per wavefront.
// c2 layer, 128 blocks: 83 us with Jacobi to the end, products and factors by all threads with a barrier per column; now 61, half of it the SVD.
template <int N>
struct Count { static constexpr int value = N; };

template <int D>
struct __attribute__((aligned(16))) BlockShared {
  typedef double matrix_t[D][D + 2];
  matrix_t LW;          // M_W, then W'^T: LW[column][row]
  matrix_t LX;          // M_X, then X'^T
  matrix_t A;           // columns of W'^T X', then of U S: A[column][row]; then B
  matrix_t scratch[3];  // [0]: V0^T, at the end U sorted and sign-normalized, U[column][row]; [1]: T as rounded to BF16 (MODE 0)
  double diag[2][D], inv_root[2][D];
  double norm2[D], sv[D], ssort[D];
  int votes[8];
};
template <int D, int MODE, int FW, int FX, class LoadFn, class FinishFn>
__device__ __forceinline__ void wush_block_group(BlockShared<D>& sh, LoadFn load, FinishFn finish, int S_W, int S_X, double lambda,
                                                 const double* __restrict__ V0, uint16_t* __restrict__ T_bits,
                                                 double* __restrict__ T_f64, double* __restrict__ V_out,
                                                 int* __restrict__ status) {
  static_assert(D == 32 || D == 16, "block size");
  constexpr int NT = 8 * D;
  constexpr int kRpl = D / 16;           // rows of a column per lane, 16 lanes per column
  typedef typename BlockShared<D>::matrix_t matrix_t;
  matrix_t &LW = sh.LW, &LX = sh.LX, &A = sh.A, &U = sh.scratch[0];
  matrix_t (&scratch)[3] = sh.scratch;
  double (&diag)[2][D] = sh.diag, (&inv_root)[2][D] = sh.inv_root;
  double (&norm2)[D] = sh.norm2, (&sv)[D] = sh.sv, (&ssort)[D] = sh.ssort;
  int (&votes)[8] = sh.votes;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, l16 = lane & 15, l4 = lane >> 4;
  // this wavefront's tile of the products (one tile for D = 16: the first wavefront's)
  const bool tiles = D == 32 || wave == 0;
  const int i0 = D == 32 ? 16 * (wave >> 1) : 0, j0 = D == 32 ? 16 * (wave & 1) : 0;
  const v4d zero = {0, 0, 0, 0};
  auto put = [&](matrix_t& m, const v4d& x) {
#pragma unroll
    for (int v = 0; v < 4; ++v) m[i0 + l4 + 4 * v][j0 + l16] = x[v];
  };
  double v0[D * D / NT];                 // fetched ahead: the same for the whole workgroup whether there is one
#pragma unroll
  for (int u = 0; u < D * D / NT; ++u) v0[u] = V0 ? V0[t + NT * u] : 0.0;
  {
    // a thread's entries of both moments and FW, FX of their partial sums are in flight at a time, added in ascending order
    constexpr int kEntries = D == 32 ? kMomentSize : 136, kPer = (kEntries + NT - 1) / NT;
    double acc[2][kPer];
    int row[kPer], col[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      acc[0][u] = acc[1][u] = 0.0;
      const int e = min(t + NT * u, kEntries - 1);
      if (D == 32 && e >= 136 && e < 392) {
        row[u] = 16 + ((e - 136) & 15);
        col[u] = (e - 136) >> 4;
      } else {
        const bool second = D == 32 && e >= 392;
        lower16_at(second ? e - 392 : e, row[u], col[u]);
        if (second) {
          row[u] += 16;
          col[u] += 16;
        }
      }
    }
    for (int w0 = 0, x0 = 0; w0 < S_W || x0 < S_X; w0 += FW, x0 += FX) {
      double vw[kPer][FW], vx[kPer][FX];
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if (u + 1 < kPer || NT * u + 64 * wave < kEntries) {   // wave-uniform; the last lanes' repeats are dropped below
          const int e = min(t + NT * u, kEntries - 1);
#pragma unroll
          for (int i = 0; i < FX; ++i) vx[u][i] = x0 + i < S_X ? load(1, e, row[u], col[u], x0 + i) : 0.0;
#pragma unroll
          for (int i = 0; i < FW; ++i) vw[u][i] = w0 + i < S_W ? load(0, e, row[u], col[u], w0 + i) : 0.0;
        }
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
#pragma unroll
        for (int i = 0; i < FX; ++i) acc[1][u] += vx[u][i];
#pragma unroll
        for (int i = 0; i < FW; ++i) acc[0][u] += vw[u][i];
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      matrix_t& L = h ? LX : LW;
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if (t + NT * u < kEntries) {
          const double m = finish(h, acc[h][u]);
          L[row[u]][col[u]] = m;
          L[col[u]][row[u]] = m;
        }
    }
  }
  __syncthreads();
  // ---- damping and Cholesky (lower), the first wavefront M_W, the second M_X.  Lane q owns row q / kLpr, columns q % kLpr, + kLpr, ... of its
  // matrix.  Step j publishes column j of what is left (in place of row j of the matrix, which is read no more); with d its diagonal entry,
  // entry (r, c) loses col[r] col[c] / d, and column j of the factor is col / sqrt(d), formed at the end.
  if (wave < 2) {
    constexpr int kLpr = 64 / D, kCpl = D / kLpr;
    matrix_t& L = wave ? LX : LW;
    double* window = &scratch[wave][0][0];             // column j by the lanes that read it: row r at (r % kLpr) 2 kCpl + r / kLpr
    const int r = lane / kLpr, g = lane % kLpr;
    double* const at = window + 2 * kCpl * (r % kLpr) + r / kLpr;
    double a[kCpl + 1], m[kCpl], f = 0.0;
    double tr = row_sum(L[l16][l16]);
    if constexpr (D == 32) tr += row_sum(L[16 + l16][16 + l16]);
    const double add = lambda * tr / (double)D;
#pragma unroll
    for (int i = 0; i < kCpl; ++i) {
      a[i + 1] = L[r][kLpr * i + g] + (kLpr * i + g == r ? add : 0.0);
      m[i] = 0.0;
    }
    a[0] = 0.0;
    wave_lds_sync();
    double now = a[1];
    // steps j = kLpr q ... + kLpr - 1, SIZE registers of columns still to do.  What step j takes off them is taken off in step j + 1, beside
    // that one's quotient; behind the last owner's with a shift.
    auto steps = [&](int q, auto size) {
      constexpr int SIZE = decltype(size)::value;
      const double* mine_at = window + 2 * kCpl * g + q;
#pragma unroll
      for (int o = 0; o < kLpr; ++o) {
        const int j = kLpr * q + o;
        if (g == o) {
          L[j][r] = now;
          *at = now;
        }
        wave_lds_sync();
        double fetched[SIZE];
#pragma unroll
        for (int i = 0; i < SIZE; ++i) fetched[i] = mine_at[i];
#pragma unroll
        for (int i = 0; i < SIZE; ++i) {
          if (o > 0) a[i] = fma(-f, m[i], a[i]);
          else a[i] = i + 1 < kCpl ? fma(-f, m[i + 1], a[i + 1]) : a[i + 1];
        }
        double d = readlane_f64(now, kLpr * j + o);
        d = d > 0.0 ? d : 1.0;
        // the row's entry of column j, from the lane of the row that has it
        const double mine = D == 32 ? (o ? dpp_f64<0xF5>(now) : dpp_f64<0xA0>(now))
                                    : (o == 0 ? dpp_f64<0x00>(now) : o == 1 ? dpp_f64<0x55>(now) : o == 2 ? dpp_f64<0xAA>(now) : dpp_f64<0xFF>(now));
        f = div_refined(mine, d);
        now = fma(-f, readlane_f64(now, (kLpr * (j + 1) + o) & 63), a[o + 1 < kLpr ? 0 : 1]);
#pragma unroll
        for (int i = 0; i < SIZE; ++i) m[i] = fetched[i];
        wave_lds_sync();
      }
    };
#pragma unroll 1
    for (int q = 0; q < kCpl / 2; ++q) steps(q, Count<kCpl>{});
#pragma unroll 1
    for (int q = kCpl / 2; q < kCpl; ++q) steps(q, Count<kCpl / 2>{});
  }
  __syncthreads();
  if (t < 2 * D) {
    double d = (t / D ? LX : LW)[t % D][t % D];
    const bool bad = !(d > 0.0);
    if (bad) d = 1.0;
    const double root = sqrt(d);
    diag[t / D][t % D] = root;
    inv_root[t / D][t % D] = 1.0 / root;
    if (MODE == 0 && __any(bad) && lane == 0) atomicExch(status, 1);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 2 * D * D / NT; ++u) {
    const int e = t + NT * u, h = e / (D * D), j = e / D % D, r = e % D;
    matrix_t& L = h ? LX : LW;
    const double root = diag[h][j];
    L[j][r] = r > j ? over_root(L[j][r], root, inv_root[h][j]) : (r == j ? root : 0.0);
  }
  if (V0) {
#pragma unroll
    for (int u = 0; u < D * D / NT; ++u) U[(t + NT * u) % D][(t + NT * u) / D] = v0[u];
  }
  __syncthreads();
  // ---- A = W'^T X':  A[j][i] = sum_k X'[k][j] W'[k][i]
  if (tiles) {
    const v4d a = product_tile<D>(LX, i0, LW, j0, zero);
    put(V0 ? scratch[1] : A, a);
  }
  if (V0) {
    __syncthreads();
    if (tiles) put(A, product_tile<D, true>(U, i0, scratch[1], j0, zero));
  }
  __syncthreads();
  // ---- columns of A made orthogonal by right rotations: A V = U S
  orthogonalize_group<D>(A, scratch[0], scratch[1], scratch[2], norm2, votes, V0 == nullptr);
  __syncthreads();
  // ---- singular values, descending order, U with the sign convention (16 lanes per column, two columns one after the other)
  {
    constexpr int kGroups = NT / 16;
    static_assert(D == 2 * kGroups, "two columns per 16 lanes");
    const int pr = t / 16, sub = t % 16;               // column; rows kRpl sub ... of it
    double x[2][kRpl], s[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c = pr + kGroups * u;
      double n2 = 0.0, best = 0.0;
#pragma unroll
      for (int i = 0; i < kRpl; ++i) {
        x[u][i] = A[c][kRpl * sub + i];
        n2 = fma(x[u][i], x[u][i], n2);
      }
      s[u] = sqrt(row_sum(n2));
      if (sub == 0) sv[c] = s[u];
#pragma unroll
      for (int i = 0; i < kRpl; ++i) {
        x[u][i] /= s[u];
        best = fmax(best, fabs(x[u][i]));
      }
      best = row_max(best);
      int first = 1 << 20;                             // 2 row + sign bit of the first row of largest magnitude
#pragma unroll
      for (int i = kRpl - 1; i >= 0; --i)
        if (fabs(x[u][i]) == best) first = 2 * (kRpl * sub + i) + (x[u][i] < 0.0);
      first = row_min(first);
#pragma unroll
      for (int i = 0; i < kRpl; ++i) x[u][i] = (first & 1) ? -x[u][i] : x[u][i];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c = pr + kGroups * u;
      int rank = 0;
#pragma unroll
      for (int i = 0; i < kRpl; ++i) {
        const int k = kRpl * sub + i;
        rank += (sv[k] > s[u]) || (sv[k] == s[u] && k < c);
      }
      rank = row_sum_int(rank);
      if (sub == 0) ssort[rank] = MODE == 1 ? 1.0 / s[u] : 1.0 / sqrt(s[u]);
#pragma unroll
      for (int i = 0; i < kRpl; ++i) U[rank][kRpl * sub + i] = x[u][i];
    }
  }
  __syncthreads();
  // ---- U^T W'^T, row i times s_i^-1/2 (B), or s_i^-1
  if (tiles) {
    v4d b = product_tile<D, true>(U, i0, LW, j0, zero);
#pragma unroll
    for (int v = 0; v < 4; ++v) b[v] *= ssort[i0 + l4 + 4 * v];
    put(A, b);
  }
  __syncthreads();
  if constexpr (MODE == 1) {
    // V = A^T U S^-1 = X'^T (S^-1 U^T W'^T)^T, made orthogonal to FP64 accuracy by one Newton-Schulz step
    // V (3 I - V^T V) / 2; the identity if it is not close to orthogonal (a singular moment).  V^T all along.
    v4d x, e;
    if (t == 0) votes[0] = 0;
    if (tiles) {
      x = product_tile<D>(A, i0, LX, j0, zero);        // V^T[c][r] = sum_k (W' U S^-1)[k][c] X'[k][r]
      put(U, x);
    }
    __syncthreads();
    if (tiles) {
      e = product_tile<D>(U, i0, U, j0, zero);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double one = i0 + l4 + 4 * v == j0 + l16 ? 1.0 : 0.0;
        if (!(fabs(e[v] - one) < 1e-3)) votes[0] = 1;
        e[v] = fma(-0.5, e[v], 1.5 * one);
      }
      put(scratch[1], e);
    }
    __syncthreads();
    if (tiles) {
      x = product_tile<D, true>(scratch[1], i0, U, j0, zero);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = i0 + l4 + 4 * v, r = j0 + l16;
        V_out[r * D + c] = votes[0] ? (r == c ? 1.0 : 0.0) : x[v];
      }
    }
    return;
  }
  // ---- T = H B with the normalized Sylvester matrix H[j][i] = (-1)^popcount(j & i) / sqrt(D)
  if (tiles) {
    constexpr int kPer = D / 4;
    const double hn = 1.0 / sqrt((double)D);
    v4d acc = zero;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = kPer * l4 + k;
      const double sign = (__popc((i0 + l16) & i) & 1) ? -1.0 : 1.0;
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sign, A[i][j0 + l16], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = (i0 + l4 + 4 * v) * D + j0 + l16;
      const double x = acc[v] * hn;
      const uint16_t bits = f64_to_bf16_bits(x);
      T_bits[o] = bits;
      scratch[1][i0 + l4 + 4 * v][j0 + l16] = (double)bf16_bits_to_f32(bits);
      if (T_f64) T_f64[o] = x;
    }
  }
}

}  // namespace wush
