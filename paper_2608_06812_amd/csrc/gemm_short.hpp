// Host launch wrapper of the residue GEMM for short products
// (gemm_short.hip). Arguments are checked by the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace ozfp4 {

constexpr int kShortTile = 128;   // lines of A and of B per block

// For each of the first nmod two-limb moduli l of mc: the residues
// R[l * rplane + col * ldr + row] of the product of the limb planes 2l,
// 2l + 1 of pa and pb, for every 128 x 128 tile that meets the m x n output,
// over the k fragments that k touches. Planes as encoded (lines padded to
// 256, kblocks fragments per line block), ldr a multiple of 256.
hipError_t launch_gemm_short(hipStream_t stream, const uint8_t* pa, const uint8_t* pb, uint8_t* R,
                             int64_t ldr, int64_t rplane, int64_t plane_a, int64_t plane_b,
                             int64_t m, int64_t n, int64_t k, int64_t kblocks, int nmod,
                             const ModConst* mc);

}  // namespace ozfp4
