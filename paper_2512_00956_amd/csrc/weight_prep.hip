// Offline weight path (Alg. 2, RTN case): T_xvsh = T_wush^{-T}, then
// q(T_xvsh W).  Also the quantizer-only test tap on FP32 values.
//
//   1. invert_blocks_kernel: one workgroup per 32x32 block, FP64 Gauss-Jordan
//      with partial pivoting on the augmented matrix [T | I].
//   2. weight_apply_quant_kernel: Wt = W_blk . inv(T_b) on the FP64 MFMA, then the
//      same RTN AbsMax MXFP4 rules as the activation kernel, decided on the FP64 values.
#include "nvfp4_layout.hpp"
#include "weight_mfma.hpp"
#include "wush_block.hpp"
#include "wush_device.hpp"
#include "wush_kernels.hpp"

namespace wush {

namespace {

// inv(T_b) of every block; the status word is cleared here and set by the kernel behind this one, which
// knows a singular block by its zero inverse.
__global__ __launch_bounds__(256) void invert_blocks_kernel(const uint16_t* __restrict__ T, double* __restrict__ Tinv,
                                                            int* __restrict__ status) {
  const int b = blockIdx.x;
  if (b == 0 && threadIdx.x < 4) status[threadIdx.x] = 0;
  auto entry = [&](int r, int c) { return (double)bf16_bits_to_f32(T[((int64_t)b * 32 + r) * 32 + c]); };
  auto store = [&](int r, int c, double v) { Tinv[((int64_t)b * 32 + r) * 32 + c] = v; };
  invert_block_group<32>(entry, store);
}

// Wt_blk = W_blk inv(T_b) and its codes.  Bound by the FP64 matrix arithmetic (1024 multiply-adds per row and
// block): a wavefront keeps its block's inverse in registers and walks tiles of 16 rows (weight_mfma.hpp), the
// four of a workgroup on adjacent blocks, so that a tile is 16 runs of 256 bytes.  Everything behind the product
// is decided on the FP64 values, in 32-bit arithmetic: f64_to_f32_sticky keeps every comparison with a midpoint of
// the grid and with 1.5 x a power of two what it was.  4096 -> 6144: 44 us (one thread per row and block, inverse in
// LDS, FP64 comparisons: 72).
template <int FMT>   // 0: MXFP4, 1: INT4
__global__ __launch_bounds__(256) void weight_apply_quant_kernel(
    const uint16_t* __restrict__ W, int64_t ldw, const double* __restrict__ Tinv,
    uint8_t* __restrict__ Wq, uint8_t* __restrict__ Ws, int N, int K, int C, int rule, int tiled,
    int* __restrict__ status) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, l4 = lane >> 4;
  const int b = 4 * blockIdx.y + (threadIdx.x >> 6);
  if (b >= C) return;
  const double* ti = Tinv + (int64_t)b * 1024;
  // row 0 of a block's inverse is zero only if the block was singular
  if (blockIdx.x == 0 && !__any(ti[lane & 31] != 0.0) && lane == 0) atomicExch(status, 1);
  wm::Block32 inv;
  wm::load_block32(inv, [&](int k, int j) { return ti[32 * k + j]; }, lane);
  const int tiles = (N + 15) / 16;
  auto fetch = [&](int t) {
    const int n = min(16 * t + l16, N - 1);
    return *reinterpret_cast<const v4u*>(W + (int64_t)n * ldw + 32 * b + 8 * l4);
  };
  v4u raw = fetch(blockIdx.x);
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int n = 16 * t + l16;
    double w[8], y[8] = {};
    wm::widen8(raw, w);
    raw = fetch(min(t + (int)gridDim.x, tiles - 1));
    wm::multiply32(inv, w, y);
    uint32_t word = 0, scale;   // this lane's 8 codes; the group's scale bits
    if constexpr (FMT == 0) {
      float v[8], amax = 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        v[i] = f64_to_f32_sticky(y[i]);
        amax = fmaxf(amax, fabsf(v[i]));
      }
      amax = wm::max_xor32(wm::max_xor16(amax));
      int byte = scale_byte_f32(amax, rule);
      if (!__any(byte < kSafeByteLo || byte > kSafeByteHi)) {
        word = pack8_e2m1(v, scale_as_f32(byte));
      } else {
        // some row's values leave FP32's range: the same rules on the FP64 values
        double am = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) am = fmax(am, fabs(y[i]));
        wm::PairF64 p = wm::pair16(am, am);
        p = wm::pair32(fmax(p.first, p.second));
        byte = scale_byte_f64(fmax(p.first, p.second), rule);
        const double inv_scale = __longlong_as_double((int64_t)(uint64_t)(1023 + 127 - byte) << 52);  // 2^(127-byte)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t sign = (uint32_t)(((uint64_t)__double_as_longlong(y[i])) >> 63);
          word |= ((sign << 3) | e2m1_code_f64(fabs(y[i]) * inv_scale)) << (4 * i);
        }
      }
      scale = (uint32_t)byte;
    } else {
      // INT4 (Table 1: 4-bit integers, BF16 scale per 32 = Gaussian-MSE-optimal step times the group's root mean
      // square): one IEEE operation per step and no fused multiply-add in the sum of squares (channels 0..15 left to
      // right, channels 16..31 left to right, the two sums added).  Lanes l4 = 0 and 2 begin the two sums, 1 and 3 go on.
#pragma clang fp contract(off)
      double sq[8], s = 0.0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        sq[i] = y[i] * y[i];
        s = i == 0 ? sq[0] : s + sq[i];
      }
      double half = wm::pair16(s, s).first;
#pragma unroll
      for (int i = 0; i < 8; ++i) half = half + sq[i];
      const wm::PairF64 sums = wm::pair32(wm::pair16(half, half).second);
      const double sigma = sqrt((sums.first + sums.second) * 0.03125);
      uint32_t bits = f64_to_bf16_bits(0.33860793 * sigma);
      bits = bits < 0x80u ? 0u : bits;
      const double q = 1.0 / (double)__uint_as_float(bits << 16);
      const double rcp = bits == 0 ? 0.0 : q;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const double c = fmin(fmax(y[i] * rcp, -8.0), 7.0);
        word |= ((uint32_t)(int)rint(c) & 0xFu) << (4 * i);
      }
      scale = bits;
    }
    if (n >= N) continue;
    if (FMT == 0 && tiled) {
      *reinterpret_cast<uint32_t*>(Wq + tiled_chunk_offset(n, b, K >> 8) + 4 * l4) = word;
      if (l4 == 0) Ws[tiled_scale_offset(n, b, K >> 8)] = (uint8_t)scale;
    } else if (tiled) {
      const int KT = K >> 6;
      *reinterpret_cast<uint32_t*>(Wq + nv_tiled_chunk_offset(n, b >> 1, b & 1, KT) + 4 * l4) = word;
      if (l4 == 0) reinterpret_cast<uint16_t*>(Ws + nv_tiled_scale_offset(n, b >> 1, KT))[b & 1] = (uint16_t)scale;
    } else {
      *reinterpret_cast<uint32_t*>(Wq + (int64_t)n * (K / 2) + 16 * b + 4 * l4) = word;
      if (FMT == 0 && l4 == 0) Ws[(int64_t)n * C + b] = (uint8_t)scale;
      if (FMT == 1 && l4 == 0) reinterpret_cast<uint16_t*>(Ws)[(int64_t)n * C + b] = (uint16_t)scale;
    }
  }
}

// Tiled -> canonical copy of packed codes and scales (inspection / tests).
__global__ __launch_bounds__(256) void unpack_tiled_kernel(const uint8_t* __restrict__ qt,
                                                           const uint8_t* __restrict__ st,
                                                           uint8_t* __restrict__ q, uint8_t* __restrict__ s,
                                                           int64_t rows, int C) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;   // one (row, group) per thread
  if (idx >= rows * C) return;
  const int row = (int)(idx / C), g = (int)(idx % C);
  *reinterpret_cast<v4u*>(q + (int64_t)row * C * 16 + 16 * g) =
      *reinterpret_cast<const v4u*>(qt + tiled_chunk_offset(row, g, C >> 3));
  s[(int64_t)row * C + g] = st[tiled_scale_offset(row, g, C >> 3)];
}

// Quantizer-only tap: one thread per group of 32 FP32 values.
__global__ __launch_bounds__(256) void quantize_f32_kernel(const float* __restrict__ Y,
                                                           uint8_t* __restrict__ q,
                                                           uint8_t* __restrict__ s,
                                                           int64_t groups, int C, int rule, int tiled) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (g >= groups) return;
  float v[32];
  const v4f* src = reinterpret_cast<const v4f*>(Y + g * 32);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const v4f t = src[i];
    v[4 * i] = t[0]; v[4 * i + 1] = t[1]; v[4 * i + 2] = t[2]; v[4 * i + 3] = t[3];
  }
  float amax = 0.f;
#pragma unroll
  for (int i = 0; i < 32; ++i) amax = fmaxf(amax, fabsf(v[i]));
  const int byte = scale_byte_f32(amax, rule);
  const float sc = scale_as_f32(byte);
  v4u out;
#pragma unroll
  for (int i = 0; i < 4; ++i) out[i] = pack8_e2m1(v + 8 * i, sc);
  if (tiled) {
    const int row = (int)(g / C), grp = (int)(g % C);
    *reinterpret_cast<v4u*>(q + tiled_chunk_offset(row, grp, C >> 3)) = out;
    s[tiled_scale_offset(row, grp, C >> 3)] = (uint8_t)byte;
  } else {
    *reinterpret_cast<v4u*>(q + g * 16) = out;
    s[g] = (uint8_t)byte;
  }
}

}  // namespace

size_t weight_prep_status_offset(int64_t K) { return (size_t)(K / 32) * 1024 * sizeof(double); }

size_t weight_prep_workspace_bytes(int64_t /*N*/, int64_t K) { return weight_prep_status_offset(K) + 16; }

namespace {

template <int FMT>
hipError_t launch_prep(const void* W, int64_t N, int64_t K, int64_t ldw, const void* T, int rule, int tiled, void* Wq,
                       void* Ws, void* workspace, hipStream_t stream) {
  const int C = (int)(K / 32);
  double* tinv = reinterpret_cast<double*>(workspace);
  int* status = reinterpret_cast<int*>(reinterpret_cast<char*>(workspace) + weight_prep_status_offset(K));
  invert_blocks_kernel<<<dim3(C), dim3(256), 0, stream>>>((const uint16_t*)T, tinv, status);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 grid((unsigned)wm::row_groups(N, C, device_cu_count()), (unsigned)((C + 3) / 4));
  weight_apply_quant_kernel<FMT><<<grid, dim3(256), 0, stream>>>((const uint16_t*)W, ldw, tinv, (uint8_t*)Wq, (uint8_t*)Ws,
                                                                (int)N, (int)K, C, rule, tiled, status);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_weight_prep(const void* W, int64_t N, int64_t K, int64_t ldw, const void* T, int rule,
                              int tiled, void* Wq, void* Ws, void* workspace, hipStream_t stream) {
  return launch_prep<0>(W, N, K, ldw, T, rule, tiled, Wq, Ws, workspace, stream);
}

hipError_t launch_int4_weight_prep(const void* W, int64_t N, int64_t K, int64_t ldw, const void* T, int tiled, void* Wq,
                                   void* Ws, void* workspace, hipStream_t stream) {
  return launch_prep<1>(W, N, K, ldw, T, 0, tiled, Wq, Ws, workspace, stream);
}

hipError_t launch_quantize_f32(const float* Y, int64_t M, int64_t K, int rule, int tiled, void* q, void* s,
                               hipStream_t stream) {
  const int64_t groups = M * (K / 32);
  quantize_f32_kernel<<<dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, stream>>>(
      Y, (uint8_t*)q, (uint8_t*)s, groups, (int)(K / 32), rule, tiled);
  return hipGetLastError();
}

hipError_t launch_unpack_tiled(const void* qt, const void* st, int64_t rows, int64_t K, void* q, void* s,
                               hipStream_t stream) {
  const int64_t n = rows * (K / 32);
  unpack_tiled_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(
      (const uint8_t*)qt, (const uint8_t*)st, (uint8_t*)q, (uint8_t*)s, rows, (int)(K / 32));
  return hipGetLastError();
}

}  // namespace wush
