// Host launch wrappers of the FP32-emulation kernels (sgemm.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace ozfp4 {

// the CRT with nc 42-bit chunks and one rounding to binary32
hipError_t launch_crt_f32(hipStream_t stream, int nc, const uint8_t* R, int64_t ldr,
                          int64_t rplane, int64_t m, int64_t n, const uint64_t* amaxA,
                          const uint64_t* amaxB, int cA, int cB, const CrtConst* cc, float* C,
                          int64_t ldc);

}  // namespace ozfp4
