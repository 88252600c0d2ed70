// Host launch wrappers of the scheme-I kernels (ozaki1.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "convert.hpp"
#include "routes.hpp"

namespace ozfp4 {

// k_encode_ozi: nplanes (a multiple of 3) greedy limb planes of the lines of
// both operands; lut13 as HostTables::lut13, in device memory
hipError_t launch_encode_ozi(hipStream_t stream, const ConvOperand& a, const ConvOperand& b,
                             int nplanes, const uint32_t* lut13);

// k_gemm_ozi over every 128 x 128 tile of every block anti-diagonal; H holds
// 2 nblk - 1 planes of m_pad x n_pad int64 (column-major, ld m_pad)
hipError_t launch_gemm_ozi(hipStream_t stream, const uint8_t* PA, const uint8_t* PB, int64_t* H,
                           int64_t plane_a, int64_t plane_b, int64_t kblocks, int64_t m_pad,
                           int64_t n_pad, int nblk);

// the same over the 128 x 64 tiles that meet the m x n output, for k at most
// kOziShortK (ozaki1_short.hip)
hipError_t launch_gemm_ozi_short(hipStream_t stream, const uint8_t* PA, const uint8_t* PB,
                                 int64_t* H, int64_t plane_a, int64_t plane_b, int64_t kblocks,
                                 int64_t m, int64_t n, int64_t k, int64_t m_pad, int64_t n_pad,
                                 int nblk);

// k_ozi_reduce: C = RN(sum_h 2197^h H_h 2^-(s_i + t_j))
hipError_t launch_ozi_reduce(hipStream_t stream, const int64_t* H, int64_t ldh, int64_t hplane,
                             int nh, int64_t m, int64_t n, const uint64_t* amaxA,
                             const uint64_t* amaxB, int cap, double* C, int64_t ldc);

}  // namespace ozfp4
