// Host launch wrappers of the Karatsuba-mode kernels (karatsuba.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "convert.hpp"
#include "tables.hpp"

namespace ozfp4 {

// k_encode_dgemm<true, wide> on the given stream (same arguments as the kernel)
hipError_t launch_encode_kar(hipStream_t stream, const ConvOperand& a, const ConvOperand& b, int L,
                             const ModConst& mod, const ModConst* mc, const uint32_t* lut);

hipError_t launch_gemm_res_kar(unsigned grid, hipStream_t stream, const uint8_t* PA,
                               const uint8_t* PB, uint8_t* R, int64_t plane_a, int64_t plane_b,
                               int64_t kblocks, int64_t tiles_m, int64_t tiles_n, int64_t nblocks,
                               int64_t ldr, int64_t rplane, const ModConst* mc, int L);

}  // namespace ozfp4
