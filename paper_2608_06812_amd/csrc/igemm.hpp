// Host launch wrappers of the INT8 path's encoder and its GEMM for short
// products (igemm.hip). Arguments are checked by the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ozfp4 {

// One operand: element (line, kk) at X[line * rs + kk * ks], rs == 1 or
// ks == 1; its three limb planes (kblocks fragments per 32-line block), of
// which the first `blocks` line blocks and kfrags fragments are encoded.
struct S8Operand {
  const int8_t* X;
  int64_t rs, ks, lines, k;
  uint8_t* planes;
  int64_t plane_bytes, kblocks;
  uint32_t blocks, kfrags;
};

// The three greedy limb planes of both operands, in one launch (a profiled
// call passes one operand with blocks == 0).
hipError_t launch_encode_s8(hipStream_t stream, const S8Operand& a, const S8Operand& b,
                            const uint16_t* lut8);

// C = A B (m x n, wrapping int32) from the limb planes, k cut into nsplit
// ranges; with nsplit > 1 the ranges' sums go to `partial` (nsplit sets of
// m_pad x n_pad int32) and a second launch adds them into C.
struct ShortS8 {
  const uint8_t* pa;
  const uint8_t* pb;
  int32_t* C;
  int32_t* partial;
  int64_t plane_a, plane_b, kblocks;
  int64_t m, n, k, ldc, m_pad, n_pad;
  int nsplit;
};

hipError_t launch_gemm_s8_short(hipStream_t stream, const ShortS8& g);

}  // namespace ozfp4
