// Host build of the library's dispatch rules (routes.hpp), for
// tests/route_util.py. stdin lines and the line printed for each:
//   res m n k nmod nprod -> short | long, k ranges, moduli a block
//   s8 m n k             -> short | long, k ranges
//   ozi m n k nh         -> short | long
#include <cstdio>
#include <cstring>

#include "routes.hpp"

using namespace ozfp4;

int main() {
  char op[8];
  long long m, n, k;
  while (std::scanf("%7s %lld %lld %lld", op, &m, &n, &k) == 4) {
    if (!std::strcmp(op, "res")) {
      int nmod, nprod;
      if (std::scanf("%d %d", &nmod, &nprod) != 2) return 2;
      if (!use_short_gemm(m, n, k, nmod)) {
        std::printf("long 1 1\n");
        continue;
      }
      const int ns = short_gemm_split(m, n, k, nmod, nprod);
      const int64_t blocks = tiles(m, kShortTile) * tiles(n, kShortTile) * nprod * ns * nmod;
      std::printf("short %d %d\n", ns, moduli_per_block(blocks, stages_of(k), nmod));
    } else if (!std::strcmp(op, "s8")) {
      if (use_short_s8(m, n, k))
        std::printf("short %d\n", short_s8_split(m, n, k));
      else
        std::printf("long 1\n");
    } else if (!std::strcmp(op, "ozi")) {
      int nh;
      if (std::scanf("%d", &nh) != 1) return 2;
      std::printf("%s\n", use_short_ozi(m, n, k, nh) ? "short" : "long");
    } else {
      return 2;
    }
  }
  return 0;
}
