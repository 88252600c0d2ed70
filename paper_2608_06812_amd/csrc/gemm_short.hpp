// Host launch wrapper of the residue GEMM for short products
// (gemm_short.hip). Arguments are checked by the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tables.hpp"

namespace ozfp4 {

// The residues of nprod products of limb planes for the first nmod two-limb
// moduli l of mc, in one launch. Product q multiplies the planes 2l, 2l + 1
// at pa + (q / 2) term_a and pb + (q % 2) term_b (one product: q = 0; the
// two-term split: four) and writes R[q * rset + l * rplane + col * ldr + row]
// for every 128 x 128 tile that meets the m x n output, over the k fragments
// that k touches. Planes as encoded (lines padded to 256, kblocks fragments
// per line block), ldr a multiple of 256.
//
// nsplit > 1 cuts k into that many ranges, each a block of its own; the
// residues of ranges 1.. go to `partial` (nprod (nsplit - 1) sets of nmod
// residue planes) and a second launch adds them into R modulo m.
struct ShortGemm {
  const uint8_t* pa;
  const uint8_t* pb;
  uint8_t* R;
  uint8_t* partial;
  int64_t plane_a, plane_b, term_a, term_b;
  int64_t ldr, rplane, rset;
  int64_t m, n, k, kblocks;
  int nmod, nprod, nsplit;
  const ModConst* mc;
};

hipError_t launch_gemm_short(hipStream_t stream, const ShortGemm& g);

}  // namespace ozfp4
