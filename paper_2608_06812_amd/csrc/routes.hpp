// Which GEMM a product takes, and how its work is cut: rules on sizes alone,
// plain C++, so that a host test can ask for the route of any size.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace ozfp4 {

constexpr int kLongTileM = 256, kLongTileN = 128;   // block tile of k_gemm_res
constexpr int kShortTile = 128;                     // of k_gemm_short, both sides
constexpr int kTileS8M = 128, kTileS8N = 128;       // of k_gemm_s8
constexpr int kL3TileM = 128, kL3TileN = 64;        // of the three-limb short GEMMs
constexpr int kStageShortK = 64;                    // k per stage of the short GEMMs
constexpr int kMaxRanges = 16;                      // k ranges of a product, at most
constexpr int64_t kS8ShortRange = 40960;            // longest k range of k_gemm_s8_short
constexpr int64_t kOziShortK = 8192;                // longest k of k_gemm_ozi_short

inline int64_t tiles(int64_t lines, int64_t tile) { return (lines + tile - 1) / tile; }
inline int stages_of(int64_t k) { return (int)tiles(k, kStageShortK); }

// Time in us of `blocks` blocks of a short GEMM cut into ns k ranges each:
// 512 run at a time, two a CU; a stage takes stage_two us there, stage_one
// where the last round leaves every block its own CU; 2.5 us around a block's
// stages.
inline double rounds_us(int64_t blocks, int nst, int ns, double stage_two, double stage_one) {
  const int64_t total = blocks * ns, rounds = total / 512, rest = total % 512;
  const double stages = (double)((nst + ns - 1) / ns);
  double t = (double)rounds * (stages * stage_two + 2.5);
  if (rest > 0) t += stages * (rest <= 256 ? stage_one : stage_two) + 2.5;
  return t;
}

// ------------------------------------------------------------ residue GEMM
// Which residue GEMM: the 256 x 128 tile's block has a CU to itself and pays
// about 7 us around its stages, the 128 x 128 tile (gemm_short.hip) overlaps
// them with a second block but moves a third more operand bytes. GEMM stage,
// us, 256 x 128 against 128 x 128, 18 moduli: 63 / 42 at 1024^3, 916 / 571 at
// 6000 x 6000 x 384, 2328 / 1966 at 6000 x 6000 x 2048, 1885 / 1759 at 4096^3,
// 29833 / 27431 at 16384 x 16384 x 4096, 13839 / 13820 and 13792 / 13427 at
// 8192^3, 6690 / 6699 at 4096 x 4096 x 16384, 107793 / 113244 at 16384^3: the
// line lies at k = 6144. Under four blocks per CU the smaller tile also
// leaves fewer CUs idle: 70 / 18 at 128 x 128 x 8192 (19 blocks), 519 / 465 at
// 1024 x 1024 x 16384 (576), 705 / 662 at 1536 x 1024 x 16384 (864), and at
// 1792 x 1024 (1008) as much at k = 16384 (765 / 765) and 2 % more at 65536
// (3079 / 3155). The blocks are one product's: the four of the two-term split
// run one after another in the larger tile (1086 / 913 at 1024 x 1024 x 8192,
// 608 blocks each; 1489 / 1372 at 1536 x 1024 x 8192, 912).
inline bool use_short_gemm(int64_t m, int64_t n, int64_t k, int nmod) {
  const int64_t blocks = tiles(m, kLongTileM) * tiles(n, kLongTileN) * nmod;
  return k <= 6144 || blocks < 1024;
}

// Estimated time of the residue GEMM's blocks cut into ns ranges each, with
// the second launch's 4.5 us and the partial residues' traffic. Measured (GEMM
// stage, one range / the ranges this chooses): 128 x 128 x 8192, 19 moduli,
// 39.7 / 17.8 us; 128 x 128 x 2048 15.9 / 13.5; 300 x 300 x 20000 116 / 90;
// 7 x 5 x 50000 203 / 46; 600 x 500 x 8000 82.4 / 81.7; 500 x 400 x 60000 561
// / 409 (502 with 256 x 128 tiles).
inline double short_gemm_us(int64_t blocks, int nst, int ns, double residues) {
  double t = rounds_us(blocks, nst, ns, 0.47, 0.27);
  if (ns > 1) t += 4.5 + 0.3 * ns + (double)(ns - 1) * residues * 2.0 / 4e6;
  return t;
}

// Ranges of k for a product that takes k_gemm_short (1: not split).
inline int short_gemm_split(int64_t m, int64_t n, int64_t k, int nmod, int nprod) {
  const int64_t blocks = tiles(m, kShortTile) * tiles(n, kShortTile) * nmod * nprod;
  const int nst = stages_of(k);
  if (blocks == 0 || blocks > 1024) return 1;   // two rounds and more: nothing to gain
  const double residues = (double)(m * n) * nmod * nprod;
  int best = 1;
  for (int ns = 2; ns <= kMaxRanges && nst / ns >= 8; ++ns)
    if (short_gemm_us(blocks, nst, ns, residues) < short_gemm_us(blocks, nst, best, residues))
      best = ns;
  return best;
}

// Moduli a block runs one after another. A block of a few stages spends most
// of its time before its first stage lands and in its epilogue; with several
// moduli the next one's copies run under both. GEMM stage, one modulus a
// block / as chosen: 568 / 514 us at 6000 x 6000 x 384, 342 / 287 at 6000 x
// 6000 x 100, 196 / 177 at 4096 x 4096 x 256; from k = 1024 on the longer
// control code costs more (478 / 491 at 4096 x 4096 x 1024), and below about
// seven rounds of blocks the lost balance does (72.5 / 77.7 for ten moduli at
// 3000 x 3000 x 300, in 5.6 rounds of two moduli).
inline int moduli_per_block(int64_t blocks, int nst, int nmod) {
  if (nst > 8) return 1;
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>(6, blocks / 3500));
  const int groups = (int)((nmod + most - 1) / most);
  return (nmod + groups - 1) / groups;
}

// ------------------------------------------------------------ INT8 GEMM
// Which INT8 GEMM: 128 x 128 tiles, one block a CU (k_gemm_s8), or 128 x 64
// tiles, two blocks a CU and half again as many operand bytes per MFMA
// (igemm.hip). GEMM, us, in that order: 17.5 / 14.2 at 1000^3, 79 / 73 at
// 6000 x 6000 x 384, 70 / 68 at 4096 x 4096 x 1024, 461 / 462 at 8192 x 8192
// x 2048, 220 / 227 at 4096^3, 1661 / 1721 at 8192^3: the line lies at k =
// 1024. Beyond it the smaller tile, with k ranges, wins where the larger
// leaves more than 15 % of its rounds' CUs idle (72 / 15 at 164 x 152 x 7877,
// 816 / 99 at 500 x 500 x 100000; 2048^3, one full round, 35.1 / 35.5).
inline bool use_short_s8(int64_t m, int64_t n, int64_t k) {
  if (k <= 1024) return true;
  if (tiles(k, kS8ShortRange) > kMaxRanges) return false;
  const int64_t blocks = tiles(m, kTileS8M) * tiles(n, kTileS8N);
  const int64_t slots = tiles(blocks, 256) * 256;
  return blocks * 100 < slots * 85;
}

// Estimated time of the INT8 GEMM's blocks cut into ns ranges. GEMM, one 128 x
// 128 block a tile before / the ranges this chooses: 164 x 152 x 7877 71 / 15
// us, 601 x 69 x 4441 45 / 14, 33 x 50 x 200001 1591 / 77.
inline double short_s8_us(int64_t blocks, int nst, int ns, double outputs) {
  double t = rounds_us(blocks, nst, ns, 0.52, 0.30);
  if (ns > 1) t += 4.5 + (double)ns * outputs * 8.0 / 4e6;
  return t;
}

// Ranges of k for a product that takes k_gemm_s8_short: at least the ones its
// exactness asks for.
inline int short_s8_split(int64_t m, int64_t n, int64_t k) {
  const int64_t blocks = tiles(m, kL3TileM) * tiles(n, kL3TileN);
  const int nst = stages_of(k), least = (int)tiles(k, kS8ShortRange);
  int best = least;
  if (blocks > 1024) return best;
  const double outputs = (double)(m * n);
  for (int ns = least + 1; ns <= kMaxRanges && nst / ns >= 8; ++ns)
    if (short_s8_us(blocks, nst, ns, outputs) < short_s8_us(blocks, nst, best, outputs)) best = ns;
  return best;
}

// ------------------------------------------------------------ scheme I
// Which scheme-I GEMM: 128 x 128 units, one a CU, or 128 x 64 units, two a CU
// (ozaki1_short.hip). GEMM, us, in that order, 15 limbs: 25.6 / 9.5 at 64^3,
// 108 / 102 at 1024^3, 224 / 211 at 2048 x 2048 x 512, 1465 / 1480 at 4096 x
// 4096 x 1024, 690 / 697 at 2048^3: short k, or under four units a CU (325 /
// 202 at 100 x 90 x 8000).
inline bool use_short_ozi(int64_t m, int64_t n, int64_t k, int nh) {
  const int64_t units = tiles(m, 128) * tiles(n, 128) * nh;
  return k <= 768 || (k <= kOziShortK && units < 1024);
}

}  // namespace ozfp4
