// How the GEMM tile kernels write their outputs: every wavefront turns its accumulators in LDS of its own, 32 rows at a
// time, so that a store instruction covers whole runs of a row.
//
// The W fragment is the MFMA's first operand: lane (r, kh) = (lane % 32, lane / 32) of a 32 x 32 tile holds token row r, and
// its accumulator e is column 8 (e / 4) + 4 kh + e % 4 -- four consecutive columns per quad, one LDS write.  Read back as
// 16-byte chunks, a row segment of 32 CB columns goes out in 16-byte stores whatever its alignment: gfx950 takes a
// 16-byte store at any address, and rows that start at odd offsets (an N that is no multiple of 8) cost a cache line
// more per segment.  Stored element by element straight from the accumulators, every store instruction touched 64
// lines, for BF16 rows without 16-byte alignment and for every FP32 output.
#pragma once
#include "wush_device.hpp"

namespace wush {

template <bool OUT_F32, int CB>
struct RowStore {
  static constexpr int kElem = OUT_F32 ? 4 : 2;             // bytes of an output
  static constexpr int kPer = 16 / kElem;                   // outputs of a 16-byte chunk
  static constexpr int kChunks = 32 * CB / kPer;            // chunks of a row segment
  // Row pitch = segment + 16 B: the writes of a wavefront hit every bank equally often.
  static constexpr int kPitch = 16 * kChunks + 16, kBuf = 32 * kPitch;
  typedef int v4i_any __attribute__((ext_vector_type(4), aligned(2)));

  // MFMA tile j of the row block into the buffer
  static __device__ __forceinline__ void put(uint8_t* buf, const v16f& acc, int j, int lane) {
    const int r = lane & 31, kh = lane >> 5;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint8_t* at = buf + r * kPitch + kElem * (32 * j + 8 * q + 4 * kh);
      if constexpr (OUT_F32) {
        *reinterpret_cast<v4f*>(at) = (v4f){acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
      } else {
        typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
        typedef float v2f __attribute__((ext_vector_type(2)));
        v2u two;
        two[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){acc[4 * q], acc[4 * q + 1]}, v2bf));
        two[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){acc[4 * q + 2], acc[4 * q + 3]}, v2bf));
        *reinterpret_cast<v2u*>(at) = two;
      }
    }
  }

  // Whether the outputs go out as streaming stores (the same in every lane).  They are not read again by the kernel, and lines that leave the
  // L2 as they are written shorten the write-back at its end; but chunks that straddle cache lines are better put together in the L2.
  // Streaming against plain stores, whole call, both MXFP4 layouts, K = 256 .. 16384, rows of 1000 to 20008 outputs, 2 to 100 MiB of them:
  //   * rows at multiples of 64 bytes: no line is written in parts, streaming (plain, 4096 x 14336 -> 4096 118.7 -> 126.7 us).
  //   * long K: the products hide the stores, and the L2 is better left to the operands.  Rows at multiples of 16 bytes, K = 4096: -24 .. +10 %
  //     (2079 -> 10088 56.7 | 51.3 us, 4048 x 10496 -> 2416 63.1 | 58.7), K = 3072: -24 .. +11 %, K <= 1024: up to +119 %.  Other rows,
  //     K = 8192: -18 .. +10 %, K = 4096: -19 .. +12 %.
  //   * shorter K, FP32 outputs of 4 to 16 MiB: 2 MiB -3 .. +16 %, 4 MiB -8 .. +5, 8 MiB -10 .. 0, 12 MiB -11 .. +3, 16 MiB
  //     -14 .. +8, 20 MiB -11 .. +19, 28 MiB -21 .. +57 (777 x 1376 -> 3001 10.4 | 10.8 plain).  No such range for BF16: 6 MiB -8 .. +7, 8 MiB
  //     -9 .. +5, 12 MiB -11 .. +24, 28 MiB -12 .. +76.
  // NVFP4 and INT4 alike, with smaller differences: K = 4096 -7 .. +2 %, FP32 below it 12 MiB -13 .. -2, 24 MiB -13 .. +14.
  static __host__ __device__ __forceinline__ bool streams(const void* Y, int64_t ldy, int M, int N, int K) {
    const int64_t start = ldy * kElem | (int64_t)(uintptr_t)Y;   // alignment of every row
    const int64_t bytes = (int64_t)M * N * kElem;
    return (start & 63) == 0 || K >= ((start & 15) == 0 ? 4096 : 8192) || (OUT_F32 && bytes > (4 << 20) && bytes <= (16 << 20));
  }

  // The buffer's 32 rows, 32 CB columns to rows row0 ... and columns col0 ... of Y.
  static __device__ __forceinline__ void store(const uint8_t* buf, void* __restrict__ Y, int64_t ldy, int row0, int col0, int M,
                                               int N, int lane, bool stream) {
    const bool whole = row0 + 32 <= M && col0 + 32 * CB <= N;      // the same in every lane
    auto chunk_at = [&](int p, int& row, int& col) {               // 32 kChunks chunks, 64 per round
      const int idx = 64 * p + lane, row_l = idx / kChunks, chunk = idx % kChunks;
      row = row0 + row_l;
      col = col0 + kPer * chunk;
      return *reinterpret_cast<const v4i*>(buf + row_l * kPitch + 16 * chunk);
    };
    auto at = [&](int row, int col) { return static_cast<uint8_t*>(Y) + ((int64_t)row * ldy + col) * kElem; };
    int row, col;
    if (whole && stream) {
#pragma unroll
      for (int p = 0; p < kChunks / 2; ++p) {
        const v4i v = chunk_at(p, row, col);
        __builtin_nontemporal_store(v, reinterpret_cast<v4i_any*>(at(row, col)));
      }
    } else {
#pragma unroll
      for (int p = 0; p < kChunks / 2; ++p) {
        const v4i v = chunk_at(p, row, col);
        if (row >= M || col >= N) continue;
        uint8_t* y = at(row, col);
        if (col + kPer <= N) {
          *reinterpret_cast<v4i_any*>(y) = v;
        } else {                                            // the last columns of a row
#pragma unroll
          for (int e = 0; e < kPer - 1; ++e)
            if (col + e < N) {
              if constexpr (OUT_F32) reinterpret_cast<int*>(y)[e] = v[e];
              else reinterpret_cast<uint16_t*>(y)[e] = (uint16_t)((uint32_t)v[e >> 1] >> (16 * (e & 1)));
            }
        }
      }
    }
  }
};

}  // namespace wush
