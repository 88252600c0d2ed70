// LDS byte addresses of the scheme-II encoder's table entries, formed modulo
// 2^16. Integer arithmetic only, so the same text also compiles for the host,
// where a test checks every address of every modulus under UBSan.
#pragma once

#include <stdint.h>

#include "crt_round.hpp"

namespace ozfp4 {

// Alignment of the tables in LDS. A table starts at a multiple of 16 entries
// from the array's base, so the base has to be a multiple of 16 entries too
// for every m = odd 2^z, z <= 4, and entries of up to four bytes.
constexpr uint32_t kLutAlign = 64;

// q0 with -q0 e m = zero modulo 2^16, for tables of e-byte entries and
// m = odd 2^twos: zero, the address of the entry of remainder 0, has to be
// divisible by e 2^twos.
OZFP4_HD uint32_t entry_quotient_offset(uint32_t zero, uint32_t e, int twos, int odd_inv) {
  return ((0u - zero / e) >> twos) * (uint32_t)odd_inv & (0xffffu / e);
}

// -e m modulo 2^16
OZFP4_HD uint16_t entry_step(uint32_t e, int m) { return (uint16_t)(0u - e * (uint32_t)m); }

// q step + xl modulo 2^16: with q the quotient plus q0 and xl = e x, the
// address of the entry of the remainder. In 32 unsigned bits: two 16-bit
// factors would be promoted to int, which their product overflows.
OZFP4_HD uint16_t entry_sum(uint16_t q, uint16_t step, uint16_t xl) {
  return (uint16_t)((uint32_t)q * step + xl);
}

}  // namespace ozfp4
