// Weight-streaming GEMM of the NVFP4 and INT4 variants (gfx950), for few tokens and for layers whose 256-row tiles leave
// most compute units idle:
//   Y = tsx tsw * deq(Xq, Xs) . deq(Wq, Ws)^T
// (the sum over blocks of the layer forward-pass equation in the formats of the paper's
// experiments that have no block-scaled MFMA path: E2M1 x E4M3 per 16 x FP32 per tensor, and
// two's-complement codes x BF16 per 32).  At these sizes the layer is bound by reading the packed
// weights once (K/2 + K/16 bytes per output channel); the activations are a few hundred KiB that
// stay in the L2.
//
// Schedule: that of the MXFP4 kernel for few tokens.  A workgroup of four waves owns one block of 32
// output channels at a time; its waves split the K steps (64 channels each) into four contiguous
// ranges, so that a wave's weights are one contiguous run of the tiled layout, and the four partial
// tiles are summed through LDS in a fixed order.
// Arithmetic: that of the tiled kernels of these formats.  Element x group scale is exact in FP16, so
// both operands are dequantized in registers (hardware fp4 -> f16 convert or the magic-number INT4
// conversion, one packed multiply by the scale) and contracted on v_mfma_f32_32x32x16_f16 with FP32
// accumulators.  Which 16 channels an MFMA contracts is free as long as both operands agree: lane
// half h of a K step takes the step's 16-byte half h of its row (32 codes, ONE 128-bit load per lane
// and operand), and MFMA d = 0..3 of the step takes dword d of it.  The W fragment is the first
// operand, so a lane's accumulator quad is four consecutive output channels of one token.
// A wave loads its K steps in chunks of U and multiplies one chunk while the next is on its way; several
// workgroups share a CU.
// Every step costs a wave 32 vector operations per 32 x 64 block of codes it converts (W once, X once
// per 32 tokens) against 1152 bytes of weights: up to 64 tokens the conversion keeps pace with HBM.
#include "nvfp4_layout.hpp"
#include "skinny_reduce.hpp"
#include "w4_dequant.hpp"
#include "wush_kernels.hpp"

namespace wush {

namespace {

using skinny::kWaves;

struct RawStep {   // what a lane holds of one (32-row block, K step): its row's 16-byte half and scale dword
  v4u q;
  uint32_t s;
};

// K steps per chunk of loads; a wave keeps two chunks in flight (one being multiplied, one on its way).  Two, which leaves registers for
// more workgroups (four | two steps, one row block: 32 x 8192 -> 28672 NVFP4 38.2 | 33.8, INT4 42.0 | 38.0; 32 x 14336 -> 4096 15.6 | 14.8;
// two row blocks, two | one: 128 x 14336 -> 4096 25.5 | 29.7), but four of canonical rows, whose steps share lines (64.4 | 70.2).
template <int RB, bool TILED>
struct Depth { static constexpr int U = RB == 1 && !TILED ? 4 : 2; };

// Block `blk` (32 rows) of a tiled operand with KT K steps: codes at
// (((blk KT + kt) 2 + h) 32 + r) 16, scale dword at ((blk KT + kt) 32 + r) 4.
__device__ __forceinline__ void load_step(RawStep& t, const uint8_t* __restrict__ q, const uint8_t* __restrict__ s,
                                          int64_t blk_kt, int r, int h) {
  t.q = *reinterpret_cast<const v4u*>(q + ((blk_kt * 2 + h) * 32 + r) * 16);
  t.s = *reinterpret_cast<const uint32_t*>(s + (blk_kt * 32 + r) * 4);
}

// The same of either layout.  Canonical rows: K / 2 bytes of codes, 32 per K step, and K / 16 of scales, 4 per step (K is a
// multiple of 64, so the 16-byte and 4-byte loads are aligned); a row past the operand's last repeats it (never stored).  A load
// instruction then touches 32 lines instead of 8; the K steps of a chunk share them.
template <bool TILED>
__device__ __forceinline__ void load_step(RawStep& t, const uint8_t* __restrict__ q, const uint8_t* __restrict__ s, int blk,
                                          int rows, int KT, int kt, int r, int h) {
  if constexpr (TILED) {
    load_step(t, q, s, (int64_t)blk * KT + kt, r, h);
  } else {
    const int64_t at = (int64_t)min(32 * blk + r, rows - 1) * KT + kt;
    t.q = *reinterpret_cast<const v4u*>(q + at * 32 + 16 * h);
    t.s = *reinterpret_cast<const uint32_t*>(s + at * 4);
  }
}

// The lane's 32 codes of a step as four MFMA operands (8 FP16 each).
template <int FMT>
__device__ __forceinline__ void dequant_step(const RawStep& t, int h, uint32_t sel, v8h (&f)[4]) {
  const v2h sc = w_step_scales<FMT>(t.s, h, sel);   // NVFP4: [0] groups 0, 1 of the half, [1] groups 2, 3; INT4: one scale
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const v2h s2 = {sc[d >> 1], sc[d >> 1]};
    const v4u u = FMT == kNvfp4 ? dequant8(t.q[d], s2) : dequant8_int4(t.q[d], s2);
    f[d] = __builtin_bit_cast(v8h, u);
  }
}

// CBW = blocks of 32 output channels a workgroup takes at a time: the X fragments of a K step are
// converted once and multiplied with CBW weight blocks (the conversion of X is the same work in every
// workgroup; with one block per pass it costs as much as that of the weights).
template <int RB, int CBW, int FMT, bool OUT_F32, bool TILED>
__global__ __launch_bounds__(kWaves * 64) void w4_skinny_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const float* __restrict__ tsx,
    const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ Ws, const float* __restrict__ tsw,
    int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  __shared__ v4f red[kWaves][RB][4][64];
  constexpr int U = Depth<RB, TILED>::U;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int KT = K >> 6, NB = (N + 31) >> 5;
  // row blocks RB blockIdx.y ... of the tokens
  const int64_t row_block = (int64_t)RB * blockIdx.y;
  Xq += row_block * KT * 1024;             // 32 rows, in either layout
  Xs += row_block * KT * 128;
  Y = static_cast<uint8_t*>(Y) + 32 * row_block * ldy * (OUT_F32 ? 4 : 2);
  M -= 32 * (int)row_block;
  const int nrb = (M + 31) >> 5;   // row blocks the X buffers hold: a block past them re-reads the last, never stored
  const int groups = (NB + CBW - 1) / CBW;
  const uint32_t sel = 0x05040C0Cu + 0x02020000u * h;
  const float scale = FMT == kNvfp4 ? *tsx * *tsw : 1.0f;   // INT4 has no tensor scales (null pointers)
  int kt0, kt1;
  skinny::wave_k_range(KT, wave, kt0, kt1);

  struct Chunk {
    RawStep w[CBW][U], x[RB][U];
  };
  for (int g = blockIdx.x; g < groups; g += gridDim.x) {
    int jb[CBW];   // weight blocks of this pass; one past the end repeats the last (never stored)
#pragma unroll
    for (int c = 0; c < CBW; ++c) jb[c] = min(g * CBW + c, NB - 1);
    v16f acc[CBW][RB];
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[c][rb] = (v16f){0};

    // Every load is unconditional (a step past the wave's range re-reads its last step), so the compiler
    // counts the loads in flight exactly and a chunk is multiplied while the next one is on its way.  Not so a whole chunk past the
    // range of canonical rows, whose loads cost too much to be for nothing (16 x 512 -> 512 7.3 -> 4.9 us, 40 x 16384 -> 1024 33.9 ->
    // 32.6; one token, all lanes' activations in the same lines, loses up to 10 % of 9 us at 4096 channels).
    auto load_chunk = [&](Chunk& ch, int kt) {
      if (!TILED && kt >= kt1) return;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(kt + u, kt1 - 1);
#pragma unroll
        for (int c = 0; c < CBW; ++c) load_step<TILED>(ch.w[c][u], Wq, Ws, jb[c], N, KT, k, r, h);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(kt + u, kt1 - 1);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) load_step<TILED>(ch.x[rb][u], Xq, Xs, min(rb, nrb - 1), M, KT, k, r, h);
      }
    };
    auto multiply_chunk = [&](const Chunk& ch, int kt) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (kt + u < kt1) {
          v8h fx[RB][4];
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) dequant_step<FMT>(ch.x[rb][u], h, sel, fx[rb]);
#pragma unroll
          for (int c = 0; c < CBW; ++c) {
            v8h fw[4];
            dequant_step<FMT>(ch.w[c][u], h, sel, fw);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
              for (int d = 0; d < 4; ++d)
                acc[c][rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[d], fx[rb][d], acc[c][rb], 0, 0, 0);
          }
        }
    };
    if (kt0 < kt1) {
      Chunk a, b;
      load_chunk(a, kt0);
      for (int kt = kt0; kt < kt1; kt += 2 * U) {
        load_chunk(b, kt + U);
        multiply_chunk(a, kt);
        load_chunk(a, kt + 2 * U);
        multiply_chunk(b, kt + U);
      }
    }
#pragma unroll
    for (int c = 0; c < CBW; ++c)
      if (g * CBW + c < NB)
        skinny::reduce_store_block<RB, OUT_F32, FMT == kNvfp4>(acc[c], red, g * CBW + c, M, N, Y, ldy, lane,
                                                               wave, scale);
  }
}

// The K split for at most 16 tokens, on v_mfma_f32_16x16x32_f16: a row block's upper half would be padding, half of the activations' loads
// and conversions and half of every MFMA.  A lane is (row l16 of 16, quarter l4): quarters 0, 1 hold the two halves of the row's first K step
// of a pair, 2 and 3 those of the second, 16 bytes each as above; MFMA d of the pair takes dword d of all four.  A weight block is two operands
// of 16 output channels.  Behind the last K step of an odd number the activations' scales are zero, and for INT4 the weights' too: theirs may be
// infinite there.  Replayed graphs, four sets of operands, us,
// 32 x 32 | this: NVFP4 16 x 8192 -> 28672 36.6 | 31.3 (132 MB of weights: 4.2 TB/s), 8192 -> 57344 65.9 | 59.3, 14336 -> 4096 15.6 | 12.0, 1 x 4096 ->
// 6144 7.0 | 6.0, canonical 16 x 8192 -> 28672 58.5 | 49.0; INT4 40.6 | 32.8, 73.2 | 60.4, 20.0 | 15.2, 8.4 | 6.7, canonical 1 x 8192 -> 28672
// 52.6 | 44.5.
// U = pairs of K steps per chunk, of which two are in flight: one where two weight blocks share the activations or a wave's range is four pairs or
// less (canonical rows two), two otherwise (U = 2 | 1: NVFP4 16 x 8192 -> 57344 59.3 | 57.6, 16 x 704 -> 28672 6.5 | 5.5, 8 x 2048 -> 20480
// 7.8 | 7.3, 1 x 4096 -> 6144 6.0 | 6.9, 16 x 14336 -> 4096 11.9 | 15.8; canonical 3 x 512 -> 1000 INT4 3.4 | 2.8, 16 x 8192 -> 28672 49.0 | 51.6;
// three 12.5, 62.0 on 16 x 14336 -> 4096 and 8192 -> 57344).
// Accumulator v of lane (l16, l4), half a of block c: token l16, output channel 32 c + 16 a + 4 l4 + v.
template <int CBW, int U, int FMT, bool OUT_F32, bool TILED>
__global__ __launch_bounds__(kWaves * 64) void w4_skinny16_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const float* __restrict__ tsx,
    const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ Ws, const float* __restrict__ tsw,
    int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  __shared__ v4f red[kWaves][CBW][2][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, l4 = lane >> 4, h = l4 & 1;
  const int KT = K >> 6, NB = (N + 31) >> 5;
  const int groups = (NB + CBW - 1) / CBW;
  const uint32_t sel = 0x05040C0Cu + 0x02020000u * h;
  const float scale = FMT == kNvfp4 ? *tsx * *tsw : 1.0f;
  int kp0, kp1;
  skinny::wave_k_range((KT + 1) >> 1, wave, kp0, kp1);

  struct Chunk {
    RawStep w[CBW][2][U], x[U];
  };
  for (int g = blockIdx.x; g < groups; g += gridDim.x) {
    int jb[CBW];   // weight blocks of this pass; one past the end repeats the last (never stored)
#pragma unroll
    for (int c = 0; c < CBW; ++c) jb[c] = min(g * CBW + c, NB - 1);
    v4f acc[CBW][2];
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int a = 0; a < 2; ++a) acc[c][a] = (v4f){0, 0, 0, 0};
    // as above: every load is unconditional, but for a whole chunk past the range of canonical rows
    auto load_chunk = [&](Chunk& ch, int kp) {
      if (!TILED && kp >= kp1) return;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(2 * min(kp + u, kp1 - 1) + (l4 >> 1), KT - 1);
#pragma unroll
        for (int c = 0; c < CBW; ++c)
#pragma unroll
          for (int a = 0; a < 2; ++a) load_step<TILED>(ch.w[c][a][u], Wq, Ws, jb[c], N, KT, k, 16 * a + l16, h);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(2 * min(kp + u, kp1 - 1) + (l4 >> 1), KT - 1);
        load_step<TILED>(ch.x[u], Xq, Xs, 0, M, KT, k, l16, h);
      }
    };
    auto multiply_chunk = [&](Chunk& ch, int kp) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (kp + u < kp1) {
          const bool past = 2 * (kp + u) + (l4 >> 1) >= KT;
          if (FMT == kNvfp4 && past) ch.x[u].s = 0;
          const uint32_t from = FMT == kInt4 && past ? 0x0C0C0C0Cu : sel;   // zero bytes
          v8h fx[4];
          dequant_step<FMT>(ch.x[u], h, from, fx);
#pragma unroll
          for (int c = 0; c < CBW; ++c)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
              v8h fw[4];
              dequant_step<FMT>(ch.w[c][a][u], h, from, fw);
#pragma unroll
              for (int d = 0; d < 4; ++d) acc[c][a] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fw[d], fx[d], acc[c][a], 0, 0, 0);
            }
        }
    };
    if (kp0 < kp1) {
      Chunk a, b;
      load_chunk(a, kp0);
      for (int kp = kp0; kp < kp1; kp += 2 * U) {
        load_chunk(b, kp + U);
        multiply_chunk(a, kp);
        load_chunk(a, kp + 2 * U);
        multiply_chunk(b, kp + U);
      }
    }
    // the waves' sums in their order; wave w finishes the half blocks w, w + 4, ...
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int a = 0; a < 2; ++a) red[wave][c][a][lane] = acc[c][a];
    __syncthreads();
    for (int ca = wave; ca < 2 * CBW; ca += kWaves) {
      const int j = g * CBW + (ca >> 1), col = 32 * j + 16 * (ca & 1) + 4 * l4;
      const v4f* part = &red[0][ca >> 1][ca & 1][lane];
      constexpr int kNext = CBW * 2 * 64;    // the next wave's
      const v4f sum = ((part[0] + part[kNext]) + part[2 * kNext]) + part[3 * kNext];
      const bool whole = 32 * j + 32 <= N;
      if (l16 < M && j < NB && (whole || col < N)) {
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = FMT == kNvfp4 ? sum[t] * scale : sum[t];
        skinny::store_quad<OUT_F32>(Y, ldy, l16, col, N, whole, v);
      }
    }
    __syncthreads();   // red is rewritten by the next blocks
  }
}

// Second schedule, for 65..128 tokens on layers with many output channels.  Above, every wave converts the
// X fragments it multiplies, RB row blocks per K step and workgroup of 32 output channels: with four row blocks the
// activations, read from the L2 and converted once per workgroup, outweigh the weight stream (four times its bytes
// and conversions).  Here the four waves of a workgroup take four different groups of CBW output-channel blocks
// and all walk the WHOLE K range in step, so that they multiply the same X fragments: each wave converts a quarter
// of them (two (row block, K step) pairs of a chunk of eight) to FP16 and leaves them in LDS in MFMA operand order
// (lane-linear 16-byte accesses, conflict free); a chunk is double buffered, one barrier per chunk; the barrier's
// fences name LDS only, so the weight loads of the chunks ahead stay in flight across it.  Per 32 x 64 block of
// weights a wave now spends its 32 conversion operations, RB x 4 LDS reads and RB x 4 MFMAs; the raw X traffic and
// its conversion drop by four.  No partial sums across waves: a wave's accumulators are final and go straight to
// Y (one FP32 chain over K per element).
// It needs a workgroup per 4 CBW blocks of output channels, so few channels leave CUs idle, and every MFMA reads
// its X fragment from LDS (with CBW = 1): the launcher takes it where it was measured faster (launch()).  The
// kernel is written for any RB and CBW; only RB = 4, CBW = 1 is instantiated.
// Accumulator e of lane (r, h), row block rb: token 32 rb + r, output channel 32 j + 8 (e / 4) + 4 h + e % 4.
template <int RB, bool OUT_F32>
__device__ __forceinline__ void store_block(const v16f (&acc)[RB], int j, int M, int N, void* __restrict__ Y,
                                            int64_t ldy, int r, int h, float scale) {
  const bool whole = 32 * j + 32 <= N;          // the same in every lane of a wavefront
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = 32 * rb + r;
    if (row >= M) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int col = 32 * j + 8 * q + 4 * h;
      if (!whole && col >= N) continue;
      float v[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = acc[rb][4 * q + t] * scale;
      skinny::store_quad<OUT_F32>(Y, ldy, row, col, N, whole, v);
    }
  }
}

// (row block, K step) pairs of X per chunk, 4 KiB of FP16 fragments each: four K steps up to 64 tokens, two beyond
template <int RB>
struct Chunk {
  static constexpr int kPairs = RB == 1 ? 4 : 8;
};
// chunks of weights in flight ahead of the multiply: what the registers next to the accumulators allow
template <int RB, int CBW>
struct Ahead { static constexpr int kChunks = RB == 1 ? 2 : (CBW == 2 ? 1 : (RB == 4 ? 3 : 2)); };
static_assert(Chunk<4>::kPairs % kWaves == 0, "every wave converts the same number of pairs");

template <int RB, int CBW, int FMT, bool OUT_F32, bool TILED>
__global__ __launch_bounds__(kWaves * 64, 2) void w4_shared_x_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs, const float* __restrict__ tsx,
    const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ Ws, const float* __restrict__ tsw,
    int M, int N, int K, void* __restrict__ Y, int64_t ldy) {
  constexpr int kPairs = Chunk<RB>::kPairs;
  constexpr int U = kPairs / RB;            // K steps per chunk
  constexpr int kMine = kPairs / kWaves;    // pairs a wave converts per chunk
  __shared__ v4u xf[2][kPairs][4][64];      // [buffer][pair = step RB + row block][MFMA of the step][lane]: 32 or 64 KiB
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int KT = K >> 6, NB = (N + 31) >> 5;
  // row blocks RB blockIdx.y ... of the tokens
  const int64_t row_block = (int64_t)RB * blockIdx.y;
  Xq += row_block * KT * 1024;             // 32 rows, in either layout
  Xs += row_block * KT * 128;
  Y = static_cast<uint8_t*>(Y) + 32 * row_block * ldy * (OUT_F32 ? 4 : 2);
  M -= 32 * (int)row_block;
  const int nrb = (M + 31) >> 5;   // row blocks the X buffers hold: a block past them re-reads the last, never stored
  const int groups = (NB + kWaves * CBW - 1) / (kWaves * CBW);
  const int nch = (KT + U - 1) / U;
  const uint32_t sel = 0x05040C0Cu + 0x02020000u * h;
  const float scale = FMT == kNvfp4 ? *tsx * *tsw : 1.0f;

  for (int g = blockIdx.x; g < groups; g += gridDim.x) {
    int jb[CBW];   // this wave's weight blocks; one past the end repeats the last (never stored)
#pragma unroll
    for (int c = 0; c < CBW; ++c) jb[c] = min((g * kWaves + wave) * CBW + c, NB - 1);
    v16f acc[CBW][RB];
#pragma unroll
    for (int c = 0; c < CBW; ++c)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) acc[c][rb] = (v16f){0};

    // All loads are unconditional (a step past the end re-reads the last one): exact wait counts.
    RawStep xr[kMine];
    auto load_x = [&](int ch) {
#pragma unroll
      for (int m = 0; m < kMine; ++m) {
        const int p = wave + kWaves * m, u = p / RB, rb = p % RB;
        load_step<TILED>(xr[m], Xq, Xs, min(rb, nrb - 1), M, KT, min(ch * U + u, KT - 1), r, h);
      }
    };
    auto convert_x = [&](int buf) {
#pragma unroll
      for (int m = 0; m < kMine; ++m) {
        v8h f[4];
        dequant_step<FMT>(xr[m], h, sel, f);
#pragma unroll
        for (int d = 0; d < 4; ++d) xf[buf][wave + kWaves * m][d][lane] = __builtin_bit_cast(v4u, f[d]);
      }
    };
    auto load_w = [&](RawStep (&w)[CBW][U], int ch) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < CBW; ++c) load_step<TILED>(w[c][u], Wq, Ws, jb[c], N, KT, min(ch * U + u, KT - 1), r, h);
    };
    auto multiply = [&](const RawStep (&w)[CBW][U], int ch, int buf) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (ch * U + u < KT) {
          v2h sc[CBW];
#pragma unroll
          for (int c = 0; c < CBW; ++c) sc[c] = w_step_scales<FMT>(w[c][u].s, h, sel);
          // one MFMA of the step (8 of the lane's 32 codes per operand) at a time: few registers in flight
#pragma unroll
          for (int d = 0; d < 4; ++d) {
            v8h fw[CBW];
#pragma unroll
            for (int c = 0; c < CBW; ++c) {
              const v2h s2 = {sc[c][d >> 1], sc[c][d >> 1]};
              fw[c] = __builtin_bit_cast(v8h, FMT == kNvfp4 ? dequant8(w[c][u].q[d], s2) : dequant8_int4(w[c][u].q[d], s2));
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
              const v8h fx = __builtin_bit_cast(v8h, xf[buf][u * RB + rb][d][lane]);
#pragma unroll
              for (int c = 0; c < CBW; ++c)
                acc[c][rb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fw[c], fx, acc[c][rb], 0, 0, 0);
            }
          }
        }
    };
    // The weights of D chunks are in flight ahead of the one being multiplied (D + 1 register sets that take
    // turns by unrolling); the X fragments of the next chunk are converted while this one is multiplied.
    constexpr int D = Ahead<RB, CBW>::kChunks, NBUF = D + 1;
    RawStep w[NBUF][CBW][U];
#pragma unroll
    for (int s = 0; s < D; ++s) load_w(w[s], s);
    load_x(0);
    convert_x(0);
    load_x(1);
    lds_barrier();
    for (int base = 0; base < nch; base += NBUF) {
#pragma unroll
      for (int s = 0; s < NBUF; ++s) {
        const int ch = base + s;           // past the last chunk: loads repeat the last step, nothing is multiplied,
        load_w(w[(s + D) % NBUF], ch + D); // and every wave still meets the barrier
        convert_x((ch + 1) & 1);
        load_x(ch + 2);
        multiply(w[s], ch, ch & 1);
        lds_barrier();
      }
    }
#pragma unroll
    for (int c = 0; c < CBW; ++c) {
      const int j = (g * kWaves + wave) * CBW + c;
      if (j < NB) store_block<RB, OUT_F32>(acc[c], j, M, N, Y, ldy, r, h, scale);
    }
  }
}

// Tiled operands, at most 128 tokens: row blocks of 32 tokens (rb) and weight blocks (cbw) a workgroup takes at a time.
// Every workgroup converts all of its tokens' activations, so with few output channels the tokens are dealt out to idle compute
// units, and with many two weight blocks share the conversion (us, NVFP4 | INT4, a workgroup with all tokens and one weight
// block before: 100 x 14336 -> 4096 33.8 -> 23.4 | 46.0 -> 30.3; 64 x 14336 -> 4096 21.1 -> 17.0 | 28.1 -> 21.4; 100 x 2048 ->
// 2048 8.5 -> 4.9 | 10.2 -> 5.5; 128 x 8192 -> 28672 81 -> 77 | 119 -> 93; 128 x 4096 -> 24576 34.6 -> 33.0 | 50.4 -> 39.0). Up
// to 64 tokens two weight blocks pay from where the coarser grid takes no round more, one -> two (replayed graphs, four sets of operands): 64 x 8192 ->
// 28672, 3.5 blocks per compute unit, 46.0 -> 41.3 | 54.8 -> 45.0, 32 x 4096 -> 28672 16.7 -> 15.4 | 19.7 -> 17.5.
// Up to 16 tokens the line is the 32-row kernel's (NVFP4 16 x 8192 -> 28672 35.2 -> 33.7, INT4 44.1 -> 40.1); the 16-row kernel, which runs there,
// has half the activations to convert and little to share: 16 x 8192 -> 28672 28.1 -> 28.3 | 32.6 -> 31.3, 25088 27.0 -> 26.6 | 30.4 -> 29.9,
// 1 x 16384 -> 28672 51.5 -> 51.8 | 56.7 -> 56.2, and below the line, 16 x 8192 -> 20480, 21.0 -> 23.6 | 24.4 -> 28.8; but short K and many blocks
// are faster with one weight block on this side of it too: 1 x 192 -> 28672 3.1 -> 3.6 | 3.2 -> 3.7, 16 x 8192 -> 57344 50.0 -> 54.1 |
// 54.9 -> 58.3, 1 x 8192 -> 57344 46.2 -> 52.7 | 53.7 -> 57.4.
void few_token_blocks(int64_t M, int64_t N, int& rb, int& cbw) {
  const int64_t NB = (N + 31) / 32;
  const int64_t cus = device_cu_count(), tokens = (M + 31) / 32;
  rb = cbw = 2;
  if (M <= 32 || NB * tokens <= cus) {
    rb = 1;
    cbw = M <= 32 && NB > 3 * cus ? 2 : 1;
  } else if (M <= 64) {
    cbw = NB > 3 * cus ? 2 : 1;
  } else if (2 * NB <= cus) {
    cbw = 1;
  }
}

template <int FMT>
hipError_t launch_split_k(const void* Xq, const void* Xs, const float* tsx, const void* Wq, const void* Ws,
                          const float* tsw, int64_t M, int64_t N, int64_t K, int out_f32, int tiled, int rb, int cbw, void* Y,
                          int64_t ldy, hipStream_t stream) {
  const int NB = (int)((N + 31) / 32);
  const int groups = (NB + cbw - 1) / cbw;
  dim3 grid((unsigned)(groups < 4096 ? groups : 4096), (unsigned)((M + 32 * rb - 1) / (32 * rb))), block(kWaves * 64);
#define WUSH_W4S_LAUNCH(RB, CBW, F32, TILED)                                                                          \
  w4_skinny_kernel<RB, CBW, FMT, F32, TILED><<<grid, block, 0, stream>>>((const uint8_t*)Xq, (const uint8_t*)Xs, tsx, \
                                                                         (const uint8_t*)Wq, (const uint8_t*)Ws, tsw, \
                                                                         (int)M, (int)N, (int)K, Y, ldy)
#define WUSH_W4S_BY_OUT(RB, CBW)                                                                                      \
  {                                                                                                                   \
    if (tiled) { if (out_f32) WUSH_W4S_LAUNCH(RB, CBW, true, true); else WUSH_W4S_LAUNCH(RB, CBW, false, true); }     \
    else { if (out_f32) WUSH_W4S_LAUNCH(RB, CBW, true, false); else WUSH_W4S_LAUNCH(RB, CBW, false, false); }         \
  }
  if (M <= 16) {
    const int64_t per_wave = (K + 511) / 512;   // pairs of K steps
    const bool single = tiled ? per_wave <= 4 : per_wave <= 2;   // with two weight blocks of the tiled layout always
#define WUSH_W4S16(CBW, U, TILED) (out_f32 ? w4_skinny16_kernel<CBW, U, FMT, true, TILED> : w4_skinny16_kernel<CBW, U, FMT, false, TILED>)
    auto kernel = cbw == 2 ? (tiled ? WUSH_W4S16(2, 1, true) : single ? WUSH_W4S16(2, 1, false) : WUSH_W4S16(2, 2, false))
                           : (tiled ? (single ? WUSH_W4S16(1, 1, true) : WUSH_W4S16(1, 2, true))
                                    : (single ? WUSH_W4S16(1, 1, false) : WUSH_W4S16(1, 2, false)));
#undef WUSH_W4S16
    kernel<<<grid, block, 0, stream>>>((const uint8_t*)Xq, (const uint8_t*)Xs, tsx, (const uint8_t*)Wq, (const uint8_t*)Ws, tsw,
                                       (int)M, (int)N, (int)K, Y, ldy);
  } else if (rb == 1) {
    if (cbw == 2) WUSH_W4S_BY_OUT(1, 2) else WUSH_W4S_BY_OUT(1, 1)
  } else {
    if (cbw == 2) WUSH_W4S_BY_OUT(2, 2) else WUSH_W4S_BY_OUT(2, 1)
  }
#undef WUSH_W4S_BY_OUT
#undef WUSH_W4S_LAUNCH
  return hipGetLastError();
}

// The shared-X schedule takes 128 tokens and one weight block per wave: the only shape in which it
// beats the K split, and only on the layers that shared_x_pays() and w4_stream_plan() name.  With fewer tokens the K split's conversions are
// already cheap, with two weight blocks per wave too few workgroups are left, and with fewer output channels the whole-K
// walk of a wave leaves CUs idle.
template <int FMT>
hipError_t launch_shared_x(const void* Xq, const void* Xs, const float* tsx, const void* Wq, const void* Ws,
                           const float* tsw, int64_t M, int64_t N, int64_t K, int out_f32, int tiled, void* Y, int64_t ldy,
                           hipStream_t stream) {
  const int NB = (int)((N + 31) / 32);
  const int groups = (NB + kWaves - 1) / kWaves;
  dim3 grid((unsigned)(groups < 4096 ? groups : 4096), (unsigned)((M + 127) / 128)), block(kWaves * 64);
  auto kernel = out_f32 ? (tiled ? w4_shared_x_kernel<4, 1, FMT, true, true> : w4_shared_x_kernel<4, 1, FMT, true, false>)
                        : (tiled ? w4_shared_x_kernel<4, 1, FMT, false, true> : w4_shared_x_kernel<4, 1, FMT, false, false>);
  kernel<<<grid, block, 0, stream>>>((const uint8_t*)Xq, (const uint8_t*)Xs, tsx, (const uint8_t*)Wq, (const uint8_t*)Ws, tsw,
                                     (int)M, (int)N, (int)K, Y, ldy);
  return hipGetLastError();
}

// Whether the shared-X schedule is the faster one for 65..128 tokens, tiled operands.  Its time goes in rounds of two workgroups, eight blocks of 32
// channels, per CU, while the K split's finer grid grows with the channels; so it pays where a round is nearly full, for INT4, whose
// conversions cost more, from six blocks per CU, for NVFP4 from seven, but not where a second round has only begun.  Measured at
// 100 tokens from HBM, us, K split | shared X, by blocks per CU:
//   INT4  8192: 5 127 | 143, 6 150 | 148, 6.25 167 | 148, 7 179 | 154, 8 205 | 165, 9 234 | 228, 10 261 | 236, 12 302 | 254
//         4096: 5  64 |  78, 6  77 |  80, 6.25  84 |  80, 7  89 |  83, 8 101 |  87, 9 121 | 122, 10 131 | 124, 12 152 | 131
//   NVFP4 8192: 6 122 | 133, 6.5 139 | 137, 7 146 | 140, 8 171 | 147, 9 200 | 203, 10 220 | 211, 11 240 | 217
//         4096: 6  64 |  74, 6.5  73 |  75, 7  76 |  76, 8  87 |  79, 9  97 | 112, 10 109 | 115, 11 119 | 117
bool shared_x_pays(int fmt, int64_t N) {
  const int64_t NB = (N + 31) / 32, cus = device_cu_count();
  return fmt == kInt4 ? NB > 6 * cus && !(NB > 8 * cus && NB <= 9 * cus)
                      : NB >= 7 * cus && !(NB > 8 * cus && NB <= 10 * cus);
}

// Estimated duration, us, of `wgs` workgroups of KT K steps: `one` per step while every compute unit has one at most, otherwise
// `full` per step and round, and a fixed part per round (its first loads, sums and stores; more where the K range of a wave is too
// short to hide a load).
struct StreamCost {
  double one, full, fixed;
};
double stream_us(const StreamCost& c, int64_t wgs, int64_t KT, int cus) {
  const double x = (double)wgs / cus, step = (double)KT;
  if (x <= 1.0) return 4.0 + c.one * step + c.fixed;
  return 4.0 + (x <= 2.0 ? 2.0 : x + 0.25) * (c.full * step + c.fixed + (KT < 16 ? 0.7 : 0.0));
}

// Row and weight blocks per workgroup -- 1 x 1, 1 x 2, 2 x 1, 2 x 2 --, then the shared-X schedule; by layout and format.
// Fits to graph replays with every schedule forced, 1 to 2048 tokens on eleven layers from 704 -> 512 to 8192 -> 28672; a canonical
// operand costs more per step, its loads being 16-byte pieces of 32 rows.
constexpr StreamCost kStreamCost[2][2][5] = {
    {{{0.125, 0.140, 0.5}, {0.185, 0.237, 1.0}, {0.175, 0.204, 0.6}, {0.245, 0.314, 0.8}, {0.70, 0.63, 3.5}},     // canonical NVFP4
     {{0.125, 0.140, 0.5}, {0.185, 0.237, 1.0}, {0.175, 0.204, 0.6}, {0.245, 0.314, 0.8}, {0.70, 0.63, 3.5}}},    // and INT4
    {{{0.053, 0.052, 0.4}, {0.0755, 0.088, 0.9}, {0.0725, 0.079, 0.5}, {0.120, 0.139, 0.6}, {0.62, 0.51, 2.3}},   // tiled NVFP4
     {{0.075, 0.069, 0.4}, {0.109, 0.113, 0.9}, {0.107, 0.106, 0.5}, {0.154, 0.163, 0.6}, {0.66, 0.57, 2.3}}}};   // and INT4

}  // namespace

// A tiled layer of at most 128 tokens always streams, by the rules above.  Any other one takes the schedule with the smallest
// estimate, if that is below the estimate for the 256-row tiles (tile_us, which the caller has): those leave compute units idle until
// tokens / 256 x channels / 128 reaches their number (us, tiles | streaming: NVFP4 224 x 16384 -> 1024 182 | 20, 320 x 14336 ->
// 4096 160 | 54, 1024 x 4096 -> 4096 52 | 40, 2048 x 4096 -> 4096 61 | 71; canonical INT4 16 x 8192 -> 28672 134 | 60).
// With every schedule forced on eleven layers from 704 -> 512 to 8192 -> 28672, 17 to 4096 tokens, the choice is within 7 % of the fastest; the
// canonical INT4 costs, taken from NVFP4's, hold as well as those.  On 640 drawn layers of K from 64 on, 25 lose 8 % or more, 13 of them
// with K <= 192, where a wave's K range is a step or none.
// The costs are the 32-row kernel's also up to 16 tokens, where canonical operands take the 16-row one.  There the choice is the fastest or within 3 % of it
// on most of 300 drawn layers (geomean 1.026), but estimates are too high for short K, where streaming is the faster throughout: 1 x 64 -> 10240
// 5.0 (tiles) | 2.5, 4 x 192 -> 24576 7.5 | 3.0; beyond that the worst is the number of weight blocks, 12 x 1152 -> 39424 two 11.4, one 10.1,
// 4 x 22912 -> 8844 one 57, two 52.
W4StreamPlan w4_stream_plan(int fmt, int64_t M, int64_t N, int64_t K, int tiled, double tile_us) {
  const int forced = debug_option(kDbgW4Skinny);
  W4StreamPlan plan;
  if (forced == 0 || M > 4096) return plan;          // beyond it the tiles have enough rows; keeps blockIdx.y small
  if (forced >= 3 && forced <= 6) return {true, false, 1 + (forced - 3) / 2, 1 + (forced - 3) % 2};   // tests: the blocks of the K split
  if (tiled && M <= 128) {
    plan.streams = true;
    plan.shared_x = M > 64 && (forced == 2 || (forced != 1 && shared_x_pays(fmt, N)));
    few_token_blocks(M, N, plan.rb, plan.cbw);
    return plan;
  }
  if (forced < 0 && debug_option(kDbgW4Width) >= 0) return plan;   // tests: a width of the tiles
  const int cus = device_cu_count();
  const int64_t NB = (N + 31) / 32, T = (M + 31) / 32, KT = K / 64;
  const StreamCost* cost = kStreamCost[tiled ? 1 : 0][fmt == kInt4 ? 1 : 0];
  double best = forced >= 1 ? 1e30 : tile_us;
  for (int c = 0; c < 5; ++c) {
    const bool shared = c == 4;
    const int rb = shared ? 4 : 1 + c / 2, cbw = shared ? 4 : 1 + c % 2;   // shared X: one weight block for each of four waves
    if ((forced == 1 && shared) || (forced == 2 && !shared)) continue;
    // a second row block needs more than 32 tokens; canonical rows: so few tokens that the lanes of an activation load share
    // lines make the conversion cheap, and one weight block is the faster (16-row kernel, one | two: 1 x 8192 -> 28672 NVFP4 41.7 | 45.3, INT4 43.9 | 49.0,
    // 4 x 4096 -> 4096 7.8 | 11.9, 8.7 | 13.2; 16 tokens 8192 -> 28672 52.0 | 48.2, 52.8 | 51.2)
    if (!shared && ((rb == 2 && M <= 32) || (cbw == 2 && !tiled && M <= 8))) continue;
    const double us = stream_us(cost[c], ((NB + cbw - 1) / cbw) * ((T + rb - 1) / rb), KT, cus);
    if (us >= best) continue;
    best = us;
    plan = {true, shared, rb, cbw};
  }
  return plan;
}

namespace {

template <int FMT>
hipError_t launch(const W4StreamPlan& plan, const void* Xq, const void* Xs, const float* tsx, const void* Wq, const void* Ws,
                  const float* tsw, int64_t M, int64_t N, int64_t K, int out_f32, int tiled, void* Y, int64_t ldy, hipStream_t stream) {
  if (plan.shared_x) return launch_shared_x<FMT>(Xq, Xs, tsx, Wq, Ws, tsw, M, N, K, out_f32, tiled, Y, ldy, stream);
  return launch_split_k<FMT>(Xq, Xs, tsx, Wq, Ws, tsw, M, N, K, out_f32, tiled, plan.rb, plan.cbw, Y, ldy, stream);
}

}  // namespace

hipError_t launch_nvfp4_gemm_skinny(const W4StreamPlan& plan, const void* Xq, const void* Xs, const float* tsx, const void* Wq,
                                    const void* Ws, const float* tsw, int64_t M, int64_t N, int64_t K, int out_f32, int tiled,
                                    void* Y, int64_t ldy, hipStream_t stream) {
  return launch<kNvfp4>(plan, Xq, Xs, tsx, Wq, Ws, tsw, M, N, K, out_f32, tiled, Y, ldy, stream);
}

hipError_t launch_int4_gemm_skinny(const W4StreamPlan& plan, const void* Xq, const void* Xs, const void* Wq, const void* Ws,
                                   int64_t M, int64_t N, int64_t K, int out_f32, int tiled, void* Y, int64_t ldy,
                                   hipStream_t stream) {
  return launch<kInt4>(plan, Xq, Xs, nullptr, Wq, Ws, nullptr, M, N, K, out_f32, tiled, Y, ldy, stream);
}

}  // namespace wush
