// Host build of the encoder's table addresses (encode_address.hpp), for
// tests/test_encode_address_host.py: every quotient and remainder of every
// modulus of every list, both entry sizes, a group starting at any modulus,
// the tables' array at any base that its alignment allows.
// Prints the number of addresses checked; exit code 1 at a wrong one.
#include <cstdio>

#define OZFP4_HD inline
#include "encode_address.hpp"

using namespace ozfp4;

static long long g_checked = 0;

static bool check_list(const ModConst& mc, int L, uint32_t e, uint32_t base) {
  const int per_word = 4 / (int)e;
  for (int l0 = 0; l0 < L; ++l0) {
    const int word0 = mc.lut_off[l0] / per_word;
    for (int l = l0; l < L; ++l) {
      const int m = mc.m[l];
      const uint32_t zero = base + e * (uint32_t)(mc.lut_off[l] - word0 * per_word + m);
      const uint32_t q0 = entry_quotient_offset(zero, e, mc.twos[l], mc.odd_inv[l]);
      const uint16_t step = entry_step(e, m);
      // every 16-bit quotient at one remainder, every remainder at a few
      for (uint32_t q = 0; q < 65536; q += l0 == 0 ? 1 : 257) {
        for (int r = -m; r < 2 * m; r += (q & 4095) ? 3 * m - 1 : 1) {
          const uint16_t xl = (uint16_t)(e * (q * (uint32_t)m + (uint32_t)r));
          const uint16_t got = entry_sum((uint16_t)(q + q0), step, xl);
          ++g_checked;
          if (got != (uint16_t)(zero + e * (uint32_t)r)) {
            std::printf("modulus %d, entry %u, base %u, first %d: q %u r %d -> %u\n", m, e, base,
                        l0, q, r, got);
            return false;
          }
        }
      }
    }
  }
  return true;
}

int main() {
  static HostTables T;
  if (!build_tables(T)) return 2;
  for (uint32_t base : {0u, kLutAlign, 3 * kLutAlign, 16 * kLutAlign}) {
    if (!check_list(T.mod, kMaxModuli, 2, base) || !check_list(T.mod, kMaxModuli, 4, base)) return 1;
    for (int h = 1; h <= kMaxHeads; ++h)
      if (!check_list(T.lists[h].mod, kMaxModuli, 2, base)) return 1;
  }
  std::printf("%lld\n", g_checked);
  return 0;
}
