// The conversion stage (Sec. IV-B, V-A, VI-B): line maxima and the fused
// encoder of both operands. Host side: operand descriptions and launch
// wrappers (convert.hip; the Karatsuba mode's encoder in karatsuba.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace ozfp4 {

// Chunks of k whose maxima a line's partial maxima hold, at most.
constexpr int kMaxChunks = 16;

// One operand as the conversion kernels see it: element (line, kk) at
// X[line * rs + kk * ks], rs == 1 (lines adjacent in memory) or ks == 1
// (lines contiguous). part holds the partial line maxima: bit patterns of
// the largest |x| as a double over k chunk c at part[c * pstride + line],
// nchunk chunks of `chunk` each. The encoder writes the line's maximum to
// amax (read by the reconstruction) and the limb planes.
struct ConvOperand {
  const void* X;
  int64_t rs, ks, lines, k;
  uint64_t* part;
  int64_t pstride, chunk;
  int nchunk;
  int cap;                 // capacity in bits
  uint64_t* amax;
  uint8_t* planes;
  int64_t plane_bytes;
  int64_t term_bytes;      // two-term split: from the first term's planes to the second's
  int64_t kblocks;         // fragments per 32-line block in the layout
  uint32_t blocks;         // 32-line blocks to encode
  uint32_t kfrags;         // fragments of each to encode
};

// Blocks of four fragments, one a wave: enough to fill the chip several
// times, each wave loops.
inline uint32_t encode_blocks(const ConvOperand& op) {
  const int64_t want = ((int64_t)op.blocks * op.kfrags + 3) / 4;
  return (uint32_t)(want < 256 * 16 ? want : 256 * 16);
}

// Fills chunk and nchunk of an operand whose X, rs, ks, lines and k are set.
void plan_line_max(ConvOperand* op);

// Partial line maxima of both operands (double, or float when f32), in one
// launch; *flag = 1 where a value is NaN or infinite.
hipError_t launch_line_max(hipStream_t stream, bool f32, const ConvOperand& a,
                           const ConvOperand& b, int* flag);

// The limb planes of both operands for the first L moduli of mc (`mod` is
// its host copy, `lut` its encoder table), FP64 or (f32) FP32 inputs;
// terms = 2 writes the second term's planes too (scaled by 2^d2).
hipError_t launch_encode(hipStream_t stream, bool f32, const ConvOperand& a, const ConvOperand& b,
                         int L, const ModConst& mod, const ModConst* mc, const uint16_t* lut,
                         int terms, int d2);

// out[line] = shift of the line (Sec. IV-B) from the partial maxima.
hipError_t launch_shifts(hipStream_t stream, const ConvOperand& op, int32_t* out);

}  // namespace ozfp4
