// MXFP4 x MXFP4 GEMM, FP32 accumulation, on CDNA4 block-scaled MFMA
// (v_mfma_scale_f32_32x32x64_f8f6f4 with both operands E2M1 and one E8M0 scale
// per 32 elements): Y = deq(Xq,Xs) . deq(Wq,Ws)^T, the sum over blocks of the
// layer forward-pass equation ("FP4-MatMul" in section "GPU Kernel Support").
//
// Operand mapping of the instruction (verified on hardware): for a 32x64
// operand tile, lane l holds row l%32 and the 32 consecutive K elements of
// half l/32 -- 16 bytes of the canonical packed layout -- plus the one scale
// byte of exactly that group.  Accumulator r of lane l is output row
// 8*(r/4) + 4*(l/32) + r%4, column l%32.
#include "wush_device.hpp"
#include <math.h>

#include "wush_kernels.hpp"

namespace wush {

namespace {

__device__ __forceinline__ void store_out(void* Y, int64_t ldy, int row, int col, float v, int out_f32) {
  if (out_f32) reinterpret_cast<float*>(Y)[(int64_t)row * ldy + col] = v;
  else reinterpret_cast<uint16_t*>(Y)[(int64_t)row * ldy + col] = f32_to_bf16_bits(v);
}

// One wavefront per 32x32 output tile, operands straight from global memory.  Handles every
// shape (ragged M, N, odd K/32).  Runs where K is too short for a pipeline (short_k below), and, forced,
// as an independent implementation in the tests.
__global__ __launch_bounds__(256) void gemm_simple_kernel(
    const uint8_t* __restrict__ Xq, const uint8_t* __restrict__ Xs,
    const uint8_t* __restrict__ Wq, const uint8_t* __restrict__ Ws,
    int M, int N, int K, int out_f32, void* __restrict__ Y, int64_t ldy) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int tiles_n = (N + 31) / 32;
  const int64_t tile = (int64_t)blockIdx.x * 4 + wave;
  const int tm = (int)(tile / tiles_n), tn = (int)(tile % tiles_n);
  if (tm * 32 >= M) return;  // wave-uniform
  const int r = lane & 31, kh = lane >> 5;
  const int C = K / 32;
  const int arow = min(tm * 32 + r, M - 1);
  const int brow = min(tn * 32 + r, N - 1);
  const uint8_t* ap = Xq + (int64_t)arow * (K / 2);
  const uint8_t* bp = Wq + (int64_t)brow * (K / 2);
  const uint8_t* as = Xs + (int64_t)arow * C;
  const uint8_t* bs = Ws + (int64_t)brow * C;
  v16f acc = {0};
  for (int g = 0; g < C; g += 2) {
    const int gg = g + kh;
    v4i a = {0, 0, 0, 0}, b = {0, 0, 0, 0};
    int sa = 127, sb = 127;
    if (gg < C) {
      a = *reinterpret_cast<const v4i*>(ap + 16 * gg);
      b = *reinterpret_cast<const v4i*>(bp + 16 * gg);
      sa = as[gg];
      sb = bs[gg];
    }
    const v8i A = {a[0], a[1], a[2], a[3], 0, 0, 0, 0};
    const v8i B = {b[0], b[1], b[2], b[3], 0, 0, 0, 0};
    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A, B, acc, 4, 4, 0, sa, 0, sb);
  }
  const int col = tn * 32 + r;
  if (col < N) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = tm * 32 + 8 * (i >> 2) + 4 * kh + (i & 3);
      if (row < M) store_out(Y, ldy, row, col, acc[i], out_f32);
    }
  }
}

// Canonical layout: whether K is so short that the one-wave-per-tile kernel is the faster one.  The others spend a fixed part on their
// prologue and on turning the outputs in LDS, which one or two steps of K do not hide; what that costs depends on the outputs'
// width, on their rows' alignment and, once they no longer fit the L2s, on their number.  Ratio of times, one wave per tile : the other kernel
// (graph replays, 1 to 8192 tokens, 512 to 65536 channels), on either side of the lines:
//   Against the streaming kernel (its 16-row form up to 16 tokens): two tokens and fewer, K = 32 1.01 to 1.11, 64 0.95 to 1.08, 96 and 128 1.02 to 1.20,
//   with 2.2 to 2.8 us in all; K = 160 to 224 1.10 to 1.30, 288 to 480 1.4 to 1.6; more tokens 1.0 to 1.9 (16 x 480 -> 8192 4.3 us : 2.6).  (Against the 32-row
//   kernel, by which the line at two tokens was drawn: K <= 128 0.91 to 1.03.)
//   More blocks of channels than compute units, up to 16 tokens, against the 16-row kernel: K <= 128 1.0 to 1.1 up to four blocks per unit,
//   0.6 to 1.0 beyond; K = 160 to 224 1.05 to 1.2 up to four, 0.7 to 1.07 beyond; K = 288 to 480 1.1 to 1.5 (4 x 480 -> 16384 4.3 us : 3.0),
//   where the lines below, drawn against the tiles, still take this kernel for rows at multiples of 16 bytes.
//   Against the pipelined kernel ("aligned": rows at multiples of 16 bytes):
//   * BF16, aligned: up to 16 tokens, K <= 128 0.78 to 0.99.  More: K = 32 and 64 0.82 to 1.19; 96 and 128 0.89 to 1.15, from 2^24 outputs on
//     1.06 to 1.36 (2048 x 96 -> 8192 12.9 us : 10.1).  K = 160 to 224 0.85 to 1.62 (2048 x 192 -> 32768 54.7 : 43.7).
//   * FP32, aligned: K <= 128 0.58 to 1.08.  K = 160 to 224, from 2^24 outputs on 0.73 to 1.29 (2048 x 192 -> 32768 67 : 86), fewer 0.80 to 1.25.
//   * Other rows: K <= 64 0.58 to 1.23; 96 and 128 0.62 to 1.16, from 3 x 2^23 outputs on 1.01 to 1.30.  K = 160 to 224, FP32 0.64 to 1.17, from
//     2^24 on 0.92 to 1.36; BF16 0.65 to 1.26, from 2^23 on 0.97 to 1.74, K = 224 beyond 128 tokens 0.96 to 1.74.
//   * A partial second step of K: aligned, up to 16 tokens 0.79 to 1.20, more 0.93 to 2.4.  Other rows, up to 64 tokens and 2^22 outputs
//     0.62 to 1.18; more tokens, up to 2^21 outputs, BF16 K = 288 0.94 to 1.13, FP32 K = 288 and 352 0.84 to 1.07; beyond these 0.96 to 2.3
//     (1000 x 416 -> 3001 BF16 9.7 us : 6.6, FP32 10.1 : 7.9).
//   * Whole steps: 1.05 to 4.2 beyond 16 tokens, 0.73 to 1.55 up to there.
bool short_k(int64_t M, int64_t N, int64_t K, int out_f32, int vec_store) {
  if (canon_streams(M, N)) return M <= 2 && K <= 128;
  const int64_t outputs = M * N;
  if (outputs >= (int64_t)1 << 35) return false;   // its grid of 32 x 32 tiles
  const bool many = outputs >= (int64_t)1 << 24;
  if (K <= 128) {
    if (vec_store && !out_f32) return M <= 16 || K <= 64 || !many;
    return vec_store || K <= 64 || outputs < (int64_t)3 << 23;
  }
  if (K < 256) {
    if (vec_store) return out_f32 && many;
    return out_f32 ? !many : outputs < (int64_t)1 << 23 && (K < 224 || M <= 128);
  }
  if (K % 256 == 0 || K >= 512) return false;
  if (vec_store) return M <= 16;
  return M <= 64 ? outputs <= (int64_t)1 << 22 : outputs <= (int64_t)1 << 21 && K < (out_f32 ? 416 : 352);
}

}  // namespace

hipError_t launch_mxfp4_gemm(const void* Xq, const void* Xs, const void* Wq, const void* Ws,
                             int64_t M, int64_t N, int64_t K, int out_f32, int tiled, void* Y, int64_t ldy,
                             hipStream_t stream) {
  if (tiled) {
    // Small batches: the streaming kernel (one workgroup per 32 output channels, the whole K) or
    // the tiled kernel with one row of 128-row tiles.  Up to 32 tokens the streaming kernel always
    // wins or ties.  Beyond, whichever the timing models below put first; they are fits to
    // measurements on ten layer shapes (4096 x 4096 .. 8192 x 57344 and 28672 x 8192), of the streaming kernel before its
    // ring, which took 4 to 30 % off, in us:
    //   streaming, by the row blocks of 32 tokens a workgroup takes (skinny_row_blocks):
    //     1: 0.6 K/1024 + 1.8, 2: 0.75 K/1024 + 2.3, and at least MiB of weights / 5.5 + 3
    //     4: rounds of (N/32 workgroups over the CUs) x (1.05 K/1024 + 2.5)
    //   tiled                    : max(4.3 + 0.3 x K/256 x rounds of (N/128 tiles over the CUs),
    //                                  MiB of weights / 6.4 + 4)
    // (with the ring, replayed graphs, four sets of operands, 100 x 14336 -> 4096 10.4 against 21.6; 64 x 8192 -> 57344 59.7 against 46.8; 128 tokens
    //  83.9 against 47.8; 128 x 4096 -> 24576 16.8 against 11.7; 128 x 28672 -> 8192 41.3 against 69.6.  On 250 drawn layers of 33 to 128
    //  tokens the choice is 1.2 % off the faster in the mean; 12 lose 5 % or more, of them long K with one to two blocks of channels per compute
    //  unit, up to 64 tokens, 33 % (46 x 28672 -> 14569 54.7 streaming against 73.4) and K up to 768 with little more than one 10 to 17 %.)
    bool skinny = M <= 32;
    if (!skinny && M <= 128) {
      const double cus = (double)device_cu_count();
      const double weight_mib = (double)N * (double)K * (17.0 / 32.0) / 1048576.0;
      const double kk = (double)K / 1024.0;
      const int rb = skinny_row_blocks(M, N);
      const double skinny_us = rb == 4 ? ceil((double)((N + 31) / 32) / cus) * (1.05 * kk + 2.5)
                                       : fmax(rb == 1 ? 0.6 * kk + 1.8 : 0.75 * kk + 2.3, weight_mib / 5.5 + 3.0);
      const double tile_rounds = ceil((double)((N + 127) / 128) / cus);
      const double tiled_us = fmax(4.3 + 0.3 * (double)(K / 256) * tile_rounds, weight_mib / 6.4 + 4.0);
      skinny = skinny_us < tiled_us;
    }
    // Up to 1024 tokens the streaming kernel also takes the layers of so few output channels that it needs no more than one workgroup
    // per compute unit, where 128-row tiles leave most of them idle (us, tiles | streaming: 256 x 4096 -> 1024 7.8 | 3.5, 1024 x 4096 ->
    // 1024 8.5 | 7.0, 256 x 16384 -> 1024 22.0 | 7.7, 448 x 28672 -> 512 39 | 13, 256 x 14336 -> 4096 21.7 | 15.6, 256 x 4096 -> 4096
    // 8.7 | 7.1; with more workgroups 448 x 4096 -> 4096 8.9 | 10.6, 448 x 14336 -> 4096 22.3 | 28.6).  One or two row blocks per
    // workgroup take 0.3 to 0.9 of the tiles' time at any K from 256 to 28672; four 0.75 to 1.02 from K = 512, but 0.9 to 1.09 with the
    // one K tile of 256 (512 x 256 -> 1984 3.85 | 4.12; with the ring 3.67 | 3.46), and 1.3 to 1.6 where the grid's spare workgroups start a second round.
    if (M > 128 && M <= 1024 && debug_option(kDbgGemmTile) < 0) {
      const int rb = skinny_row_blocks(M, N);
      const int64_t groups = (M + 32 * rb - 1) / (32 * rb), blocks = rb < 4 ? (N + 31) / 32 : skinny_grid_width(N);
      skinny = groups * blocks <= device_cu_count() && (rb < 4 || K > 256);
    }
    if (M <= 1024 && debug_option(kDbgGemmSkinny) >= 0) skinny = debug_option(kDbgGemmSkinny) == 1;   // tests: force either kernel
    if (skinny) return launch_mxfp4_gemm_skinny(Xq, Xs, Wq, Ws, M, N, K, out_f32, Y, ldy, stream);
    return launch_mxfp4_gemm_frag(Xq, Xs, Wq, Ws, M, N, K, out_f32, Y, ldy, stream);
  }
  bool simple = short_k(M, N, K, out_f32, canon_vec_store(Y, ldy, out_f32));
  if (debug_option(kDbgGemmTile) >= 0) simple = false;                                       // tests: a tile shape of the other kernel
  if (const int forced = debug_option(kDbgGemmSimple); forced >= 0) simple = forced == 1;    // tests: either kernel
  if (!simple && (canon_streams(M, N) || canon_streams16(M, N, K)) && debug_option(kDbgGemmTile) < 0 && debug_option(kDbgGemmSkinny) != 0)
    return launch_mxfp4_gemm_canon_stream(Xq, Xs, Wq, Ws, M, N, K, out_f32, Y, ldy, stream);
  if (!simple) return launch_mxfp4_gemm_canon(Xq, Xs, Wq, Ws, M, N, K, out_f32, Y, ldy, stream);
  const int64_t tiles = ((M + 31) / 32) * ((N + 31) / 32);
  gemm_simple_kernel<<<dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, stream>>>(
      (const uint8_t*)Xq, (const uint8_t*)Xs, (const uint8_t*)Wq, (const uint8_t*)Ws,
      (int)M, (int)N, (int)K, out_f32, Y, ldy);
  return hipGetLastError();
}

}  // namespace wush
