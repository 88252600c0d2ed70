// Device code shared by the translation units of the library: types,
// constants, the scale helpers, the residue-GEMM tile and its helpers.
// Templates and inline functions only, so every translation unit can include
// it.
//
// Data layout (HBM):
//   * limb planes: per operand, plane p holds one limb of one modulus for
//     every (line, k); it is a sequence of 1 KiB fragments of 32 lines x 64 k
//     in the exact register order of the A/B operand of
//     v_mfma_f32_32x32x64_f8f6f4 in FP4 mode (lane = line % 32 +
//     32 * (k / 32 % 2), 16 bytes per lane, two E2M1 codes per byte, low
//     nibble first). A wave therefore moves a fragment with one 16-byte
//     load per lane, coalesced in HBM and conflict-free in LDS. Fragments
//     of one 32-line block are contiguous along k.
//   * residues: one byte per (modulus, i, j), column-major per modulus with
//     the padded row count as leading dimension.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "crt_round.hpp"
#include "tables.hpp"

namespace ozfp4 {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kFragLines = 32;   // lines per fragment
constexpr int kFragK = 64;       // k per fragment
constexpr int kFragBytes = 1024;
constexpr int kTile = 256;       // line padding of every operand (multiple of both GEMM block tiles)
constexpr int kStageK = 128;     // k per pipeline stage (two fragments)
constexpr int kMinKPad = 384;    // k is padded to at least three stages

constexpr uint64_t kAbsMask = 0x7fffffffffffffffull;
constexpr uint64_t kNonFinite = 0x7ff0000000000000ull;

// One launch holds fewer than 2^32 work-items. Kernels with one thread per
// item take their first item as an argument and the host splits larger
// counts into launches of kLaunchThreads threads; grid-stride kernels take
// at most kLaunchThreads / 256 blocks of 256.
constexpr int64_t kLaunchThreads = int64_t(1) << 30;
inline unsigned stride_blocks(int64_t items, int64_t per) {
  const int64_t b = items / per + (items % per != 0);
  const int64_t cap = kLaunchThreads / 256;
  return (unsigned)(b < cap ? b : cap);
}

// ------------------------------------------------------------ Sec. IV-B
// floor(log2 |x|) from the bit pattern of the line maximum |x| (finite,
// nonzero), subnormals included; shift c - 1 - e, or 0 for a zero line.
__device__ __forceinline__ int line_shift(uint64_t amax_bits, int cap) {
  if (amax_bits == 0) return 0;
  int ex = (int)(amax_bits >> 52);
  int e;
  if (ex == 0) {
    uint64_t mant = amax_bits & 0x000fffffffffffffull;
    e = (63 - __clzll((long long)mant)) - 1074;
  } else {
    e = ex - 1023;
  }
  return cap - 1 - e;
}

// Maximum of a line over its nchunk partial maxima (line c * pstride + line).
__device__ __forceinline__ uint64_t partial_max(const uint64_t* __restrict__ part, int64_t pstride,
                                                int nchunk, int64_t line) {
  uint64_t v = 0;
  for (int c = 0; c < nchunk; c += 8) {   // eight loads in flight, the last chunk's repeated
    uint64_t w[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = part[min(c + e, nchunk - 1) * pstride + line];
#pragma unroll
    for (int e = 0; e < 8; ++e) v = max(v, w[e]);
  }
  return v;
}

constexpr int kEncWaves = 4;   // waves of an encoder block, one fragment each

// ------------------------------------------------------------ Sec. VI-D
// Block tile index -> (modulus, tile row, tile column). Consecutive block
// ids go to the 8 XCDs round-robin. When the tile count T of one modulus is
// a multiple of 8, XCD x takes tiles [x T/8, (x+1) T/8) of every modulus in
// turn: every XCD then carries the same mix of moduli, the blocks an XCD
// runs together share the A and B panels of one modulus in its L2, and all
// XCDs stream the same B panels at about the same time. Otherwise each XCD
// takes a contiguous range of the flattened (modulus, tile) order, and so it
// does below min_share tiles, where an eighth of the grid is too few tiles to
// share panels in an XCD's L2. Tiles are ordered in groups of kGroupM tile
// rows.
#ifndef OZFP4_GROUP_M
#define OZFP4_GROUP_M 4
#endif
constexpr int kGroupM = OZFP4_GROUP_M;
// A grid holds fewer than 2^32 work-items, so every count here is below 2^24
// and the divisions are 32-bit ones.
__device__ __forceinline__ void tile_coords(unsigned bid, int64_t nblocks, int64_t tiles_m,
                                            int64_t tiles_n, int* l, int64_t* tm, int64_t* tn,
                                            unsigned min_share = 8) {
  const unsigned xcd = bid & 7, local = bid >> 3;
  const unsigned T = (unsigned)(tiles_m * tiles_n);
  unsigned t;
  if ((T & 7) == 0 && T >= min_share) {
    const unsigned per = T >> 3;
    const unsigned li = local / per;
    *l = (int)li;
    t = xcd * per + (local - li * per);
  } else {
    const unsigned base = (unsigned)nblocks >> 3, rem = (unsigned)nblocks & 7;
    const unsigned logical = xcd * base + min(xcd, rem) + local;
    const unsigned li = logical / T;
    *l = (int)li;
    t = logical - li * T;
  }
  const unsigned span = kGroupM * (unsigned)tiles_n;
  const unsigned group = t / span;
  const unsigned first = group * kGroupM;
  const unsigned gm = min((unsigned)tiles_m - first, (unsigned)kGroupM);
  const unsigned in = t - group * span;
  const unsigned col = in / gm;
  *tm = first + (in - col * gm);
  *tn = col;
}

__device__ __forceinline__ v16f mfma_fp4(v4i a, v4i b, v16f c) {
  v8i a8 = {a.x, a.y, a.z, a.w, 0, 0, 0, 0};
  v8i b8 = {b.x, b.y, b.z, b.w, 0, 0, 0, 0};
  // cbsz = blgp = 4: both operands E2M1. Constant zero scale operands make
  // the compiler emit the unscaled v_mfma_f32_32x32x64_f8f6f4, which
  // multiplies by 2^0 (bitwise equal to the scaled form with E8M0 127) and
  // takes no scale register (0 to 1.2 % faster GEMMs at the same clock in
  // same-device comparisons).
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 4, 4, 0, 0, 0, 0);
}

// Raw 32-bit data format of untyped buffer loads: dword 3 of a buffer
// descriptor as the gfx9-family ISA defines it.
constexpr int kBufferWord3 = 0x00020000;

// Buffer-form LDS DMA: each lane copies 16 bytes from byte voffset + soffset
// of buffer `src` (a wave-uniform descriptor, held in SGPRs) to LDS at
// lds_base + 16 * lane (buffer_load_dwordx4 ... lds). A copy reads one
// 32-bit VGPR offset and one SGPR offset instead of a 64-bit address per
// lane. Completion is tracked by vmcnt.
__device__ __forceinline__ void dma16_buf(__amdgpu_buffer_rsrc_t src, uint32_t voffset,
                                          uint32_t soffset, uint8_t* lds_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      src, (__attribute__((address_space(3))) void*)lds_base, 16, voffset, soffset, 0, 0);
}

// s_waitcnt vmcnt(N) lgkmcnt(0) (expcnt untouched): this wave's vector
// loads except the newest N have landed, and its LDS reads are complete.
template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

__device__ __forceinline__ void block_sync() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Dgemm residue GEMM: planes 2l (c0) and 2l+1 (c1) of modulus l;
// accumulators acc0 = a0 b0, acc1 = a0 b1 + a1 b0, acc2 = a1 b1; epilogue
// r = (4 acc0 + 52 acc1 + 676 acc2) mod m, one byte per element.
//
// Block tile 256 (lines of A) x 128 (lines of B), k in stages of 128. Eight
// waves, two per SIMD, each 64 x 64 (2 x 2 MFMA tiles of 32 x 32, three
// accumulator sets = 192 registers, everything within 256 registers so two
// waves share a SIMD and cover each other's LDS and barrier waits). A stage
// is 48 fragments (A: 2 planes x 8 line blocks x 2 k fragments, then B:
// 2 planes x 4 line blocks x 2 k fragments), 48 KiB, copied into a 3-slot
// LDS ring by buffer-form LDS DMA (6 whole fragments per wave, each 1 KiB
// contiguous in HBM), two stages ahead of the one being multiplied.
constexpr int kTileM = 256;        // lines of A per block
constexpr int kTileN = 128;        // lines of B per block
constexpr int kRing = 3;           // LDS slots
constexpr int kWaves = 8;
constexpr int kStageFrags = 48;
constexpr int kStageBytes = kStageFrags * kFragBytes;
constexpr int kDmaPerWave = kStageFrags / kWaves;   // 6

// LDS offset of fragment (plane p, line block rb / cb, k fragment kbl)
__device__ __forceinline__ constexpr int fragA(int p, int rb, int kbl) { return ((p * 8 + rb) * 2 + kbl) * kFragBytes; }
__device__ __forceinline__ constexpr int fragB(int p, int cb, int kbl) { return (32 + (p * 4 + cb) * 2 + kbl) * kFragBytes; }

// Epilogue of a block tile: r = (W0 acc0 + W1 acc1 + W2 acc2) mod m for the
// wave's 64 x 64 outputs, one byte per element, four rows per 32-bit store.
// The accumulators hold exact multiples of 1/4 (Lemma 3), the FP64 sum is
// exact, and floor(d fl(1/m)) is within one of floor(d / m).
template <int W0, int W1, int W2>
__device__ __forceinline__ void store_residues(const v16f (&acc)[3][2][2], int l, int64_t tm,
                                               int64_t tn, int wm, int wn, int lane,
                                               uint8_t* __restrict__ R, int64_t ldr,
                                               int64_t rplane, const ModConst* __restrict__ mc) {
  const int m = mc->m[l];
  const double inv = mc->inv[l], md = mc->md[l];
  uint8_t* Rl = R + (int64_t)l * rplane;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t col = tn * kTileN + wn * 64 + j * 32 + (lane & 31);
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int64_t row = tm * kTileM + wm * 64 + i * 32 + g * 8 + (lane >> 5) * 4;
        uint32_t word = 0;
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
          const int v = g * 4 + v4;
          double d = (double)W0 * (double)acc[0][i][j][v] + (double)W1 * (double)acc[1][i][j][v] +
                     (double)W2 * (double)acc[2][i][j][v];
          double qd = __builtin_floor(d * inv);
          int r = (int)__builtin_fma(-qd, md, d);
          r += (r < 0) ? m : 0;
          r -= (r >= m) ? m : 0;
          word |= (uint32_t)r << (8 * v4);
        }
        *reinterpret_cast<uint32_t*>(Rl + col * ldr + row) = word;
      }
    }
}

// Residue composition in FP32. The accumulators hold exact multiples of 1/4
// and every limb of the two-limb splits is within +-8, so with
// t = acc0 + 13 acc1 + 169 acc2 (in units of 1/4, r = 4 t mod m):
//   kLevel 1, k <= 1337: |4 t| <= (64 + 13 * 128 + 169 * 64) k < 2^24, so t
//     is exact, and one reduction t - rint(t 4/m) m/4 (exact FMA) brings it
//     into (-m/4, m/4);
//   kLevel 2, k <= 17476: |4 (acc1 + 13 acc2)| <= 960 k < 2^24 is reduced
//     first, then 13 times that plus acc0;
//   kLevel 3, larger k: the FP64 composition.
// rint(t fl(4/m)) is within 2^24 / m * 2^-23 < 0.2 of t 4/m, so a reduced
// value is within 0.7 m/4, and adding m/4 to a negative one gives [0, m/4).
// Nine (twelve) full-rate operations an element in place of about twenty
// FP64 ones and conversions.
__device__ __forceinline__ int residue_level(int64_t k_pad) {
  return k_pad <= 1337 ? 1 : (k_pad <= 17476 ? 2 : 3);
}

__device__ __forceinline__ float reduce_quarter(float t, float inv4, float m4) {
  return __builtin_fmaf(-__builtin_rintf(t * inv4), m4, t);
}

// residue bytes of rows 8 g + 4 (lane / 32) .. + 3 of the 32 x 32 tile (i, j)
template <int kLevel, bool kSkipA1B1>
__device__ __forceinline__ uint32_t residue_word(const v16f (&acc)[3][2][2], int i, int j, int g,
                                                 int m, float inv4, float m4, double inv,
                                                 double md) {
  uint32_t word = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int v = g * 4 + e;
    if constexpr (kLevel < 3) {
      float t = acc[1][i][j][v];
      if constexpr (!kSkipA1B1) t = __builtin_fmaf(13.0f, acc[2][i][j][v], t);
      if constexpr (kLevel == 2) t = reduce_quarter(t, inv4, m4);
      t = __builtin_fmaf(13.0f, t, acc[0][i][j][v]);
      t = reduce_quarter(t, inv4, m4);
      // for t < 0 the bit pattern of t (as unsigned) exceeds that of
      // t + m/4, for t >= 0 it is the smaller one
      const uint32_t r = min((uint32_t)__float_as_uint(t), (uint32_t)__float_as_uint(t + m4));
      word = __builtin_amdgcn_cvt_pk_u8_f32(4.0f * __uint_as_float(r), e, word);
    } else {
      double d = __builtin_fma(52.0, (double)acc[1][i][j][v], 4.0 * (double)acc[0][i][j][v]);
      if constexpr (!kSkipA1B1) d = __builtin_fma(676.0, (double)acc[2][i][j][v], d);
      int r = (int)__builtin_fma(-__builtin_floor(d * inv), md, d);
      r += (r < 0) ? m : 0;
      r -= (r >= m) ? m : 0;
      word |= (uint32_t)r << (8 * e);
    }
  }
  return word;
}

// A wave's 64 x 64 residues, rows from row0, columns from col0. A swap of
// half-waves between the two row blocks leaves each lane 32 consecutive rows
// of one column, stored as two 16-byte words (instead of eight 4-byte ones,
// whose 8-byte segments cost L2 four times the write requests).
template <int kLevel, bool kSkipA1B1>
__device__ __forceinline__ void store_residues_wave(const v16f (&acc)[3][2][2], int m,
                                                    uint8_t* __restrict__ Rl, int64_t ldr,
                                                    int64_t row0, int64_t col0, int lane) {
  const float m4 = 0.25f * (float)m, inv4 = 4.0f / (float)m;
  const double md = (double)m, inv = 1.0 / md;
  uint8_t* dst = Rl + (col0 + (lane & 31)) * ldr + row0 + (lane >> 5) * 32;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    v4i w[2];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const uint32_t w0 = residue_word<kLevel, kSkipA1B1>(acc, 0, j, g, m, inv4, m4, inv, md);
      const uint32_t w1 = residue_word<kLevel, kSkipA1B1>(acc, 1, j, g, m, inv4, m4, inv, md);
      // lanes 0-31 keep w0 and get the upper lanes' w0 in place of w1;
      // lanes 32-63 keep w1 and get the lower lanes' w1 in place of w0
      const auto s = __builtin_amdgcn_permlane32_swap(w0, w1, false, false);
      w[g >> 1][2 * (g & 1)] = (int)s[0];
      w[g >> 1][2 * (g & 1) + 1] = (int)s[1];
    }
    v4i* p = reinterpret_cast<v4i*>(dst + (int64_t)j * 32 * ldr);
    p[0] = w[0];
    p[1] = w[1];
  }
}

// kMinLevel: the smallest level that is compiled in (a higher one than
// needed is exact too)
template <bool kSkipA1B1, int kMinLevel>
__device__ __forceinline__ void store_residues_by_k(const v16f (&acc)[3][2][2], int64_t k_pad,
                                                    int m, uint8_t* __restrict__ Rl, int64_t ldr,
                                                    int64_t row0, int64_t col0, int lane) {
  const int level = residue_level(k_pad);
  if (kMinLevel == 1 && level == 1)
    store_residues_wave<1, kSkipA1B1>(acc, m, Rl, ldr, row0, col0, lane);
  else if (level <= 2)
    store_residues_wave<2, kSkipA1B1>(acc, m, Rl, ldr, row0, col0, lane);
  else
    store_residues_wave<3, kSkipA1B1>(acc, m, Rl, ldr, row0, col0, lane);
}

// The blocks that one XCD runs together share their operand panels in its L2,
// which holds about 16 stages of them, so they have to stay in step over
// their 100 and more stages. With the FP64 epilogue (about 9 us of VALU and
// of narrow stores through the shared L2) they did; with the FP32 one they
// drift apart: L2 hit rate 84 -> 40 %, GEMM 108.4 -> 114.9 ms at 16384^3 with
// 18 moduli. So a block whose first copies are issued waits until the other
// blocks of its group have come as far: the arrivals on an XCD (block id mod
// 8) are counted in arrive[xcd], `slots` of them (the XCD's CUs, one block
// each) form a group, the last group takes what is left. The wait ends after
// 24 polls in any case (about 20 us; a group stays short where another stream
// holds CUs). With it: 107.0 ms at 16384^3, 13.57 ms against 13.77 at 8192^3.
// The Karatsuba GEMM goes without: its blocks differ in length by modulus and
// were not in step with the FP64 epilogue either (16384^3, FP64 / FP32: L2 hit
// rate 63 / 61 %, FETCH_SIZE 2.10e8 / 2.06e8 KiB, 118.0 / 117.1 ms).
constexpr int kLockstepPolls = 24;
__device__ __forceinline__ void xcd_lockstep(unsigned* arrive, unsigned nblocks, unsigned slots) {
  if (threadIdx.x != 0) return;
  const unsigned xcd = blockIdx.x & 7;
  const unsigned total = (nblocks >> 3) + (xcd < (nblocks & 7) ? 1u : 0u);
  unsigned* count = arrive + xcd;
  const unsigned mine =
      __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const unsigned target = min((mine / slots + 1) * slots, total);
  for (int poll = 0; poll < kLockstepPolls; ++poll) {
    if (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target) break;
    __builtin_amdgcn_s_sleep(4);
  }
}

// One block tile of modulus l. kSkipA1B1: m = 169 = 13^2, where 169 a1 b1 is
// 0 mod m (Sec. V-A), so the a1 b1 products are not issued (acc2 stays 0).
// arrive: the lockstep counters (null: no lockstep).
template <bool kSkipA1B1>
__device__ __forceinline__ void gemm_res_tile(
    uint8_t* lds, int l, int64_t tm, int64_t tn, const uint8_t* __restrict__ PA,
    const uint8_t* __restrict__ PB, uint8_t* __restrict__ R, int64_t plane_a, int64_t plane_b,
    int64_t kblocks, int64_t ldr, int64_t rplane, const ModConst* __restrict__ mc,
    unsigned* arrive, unsigned nblocks, unsigned slots) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int rbw = 2 * wm, cbw = 2 * wn;   // this wave's first A / B line block

  // fragment f = wave * 6 + j of a stage (LDS offset f KiB): a buffer
  // descriptor per fragment, based at that fragment of stage 0 (uniform);
  // stage st adds st * 2 KiB as the SGPR offset
  const int nst = (int)(kblocks / 2);
  __amdgpu_buffer_rsrc_t src[kDmaPerWave];
#pragma unroll
  for (int j = 0; j < kDmaPerWave; ++j) {
    const int f = wave * kDmaPerWave + j;
    const uint8_t* base;
    if (f < 32) {
      const int kbl = f & 1, rb = (f >> 1) & 7, p = f >> 4;
      base = PA + (int64_t)(2 * l + p) * plane_a + ((tm * 8 + rb) * kblocks + kbl) * kFragBytes;
    } else {
      const int g = f - 32, kbl = g & 1, cb = (g >> 1) & 3, p = g >> 3;
      base = PB + (int64_t)(2 * l + p) * plane_b + ((tn * 4 + cb) * kblocks + kbl) * kFragBytes;
    }
    src[j] = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, nst * 2 * kFragBytes,
                                               kBufferWord3);
  }
  const int lane16 = lane * 16;
  auto dma = [&](int st, int j) {
    dma16_buf(src[j], (uint32_t)lane16, (uint32_t)(st * 2 * kFragBytes),
              lds + (st % kRing) * kStageBytes + (wave * kDmaPerWave + j) * kFragBytes);
  };

  v16f acc[3][2][2];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][i][j][v] = 0.0f;

  // Schedule. The operand registers of a k fragment (a_p, b_p: two
  // fragments each for planes p = 0, 1) are refilled from LDS for the next
  // k fragment as soon as their last product group has been issued, so
  // every LDS read has at least one product group (four MFMAs of this wave,
  // eight of its SIMD) to land in, and the two waves of a SIMD no longer
  // wait for their reads together at the start of each k fragment. With product group g_pq = the four
  // MFMAs a_p b_q, k fragment 0 of a stage issues g00 g01 g11 g10 and
  // k fragment 1 issues g01 g00 g10 g11: each fragment's last groups free
  // the registers that the next fragment's first groups need last.
  // Modulus 169 has no g11 and issues g10 g00 g01 in both fragments.
  //
  // Stage s + 2 is copied during stage s into the slot of stage s - 1,
  // which every wave finished reading before the previous barrier; the six
  // copies per wave are spread over the product groups before the
  // handover. The
  // handover (this wave's copies of stage s + 1 landed and its reads of
  // stage s done, then a barrier) comes after the first two groups of
  // k fragment 1 (first one for 169), so the matrix pipe still has eight
  // MFMAs of the wave queued while the waves synchronise; the reads of
  // stage s + 1 start right after it.
  v4i a[2][2], b[2][2];   // [plane][i] of A, [plane][j] of B
  auto readA = [&](const uint8_t* sb, int kbl, int p) {
#pragma unroll
    for (int i = 0; i < 2; ++i) a[p][i] = *reinterpret_cast<const v4i*>(sb + fragA(p, rbw + i, kbl) + lane16);
  };
  auto readB = [&](const uint8_t* sb, int kbl, int p) {
#pragma unroll
    for (int j = 0; j < 2; ++j) b[p][j] = *reinterpret_cast<const v4i*>(sb + fragB(p, cbw + j, kbl) + lane16);
  };
  // g_pq into acc[p + q]: a0 b0 -> acc0, a0 b1 and a1 b0 -> acc1, a1 b1 -> acc2
  auto group = [&](int p, int q) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[p + q][i][j] = mfma_fp4(a[p][i], b[q][j], acc[p + q][i][j]);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  auto handover = [&](bool copy) {
    if (copy)
      wait_vm_lgkm0<kDmaPerWave>();   // stage s + 1 landed; reads of stage s done
    else
      wait_vm_lgkm0<0>();
    block_sync();
  };

  // copy: issue the copies of stage s + 2; next: stage s + 1 exists
  auto stage = [&](int s, bool copy, bool next) {
    const uint8_t* sb = lds + (s % kRing) * kStageBytes;
    const uint8_t* nb = lds + ((s + 1) % kRing) * kStageBytes;
    auto cp = [&](int j) {
      if (copy) dma(s + 2, j);
    };
    if constexpr (!kSkipA1B1) {
      group(0, 0); cp(0); fence();
      group(0, 1); readA(sb, 1, 0); cp(1); fence();
      group(1, 1); readB(sb, 1, 1); cp(2); fence();
      group(1, 0); readA(sb, 1, 1); readB(sb, 1, 0); cp(3); fence();
      group(0, 1); cp(4); fence();
      group(0, 0); cp(5); fence();
      if (next) {
        handover(copy);
        readA(nb, 0, 0); fence();
        group(1, 0); readB(nb, 0, 0); fence();
        group(1, 1); readA(nb, 0, 1); readB(nb, 0, 1); fence();
      } else {
        group(1, 0); group(1, 1); fence();
      }
    } else {
      group(1, 0); readA(sb, 1, 1); cp(0); cp(1); fence();
      group(0, 0); readB(sb, 1, 0); cp(2); cp(3); fence();
      group(0, 1); readA(sb, 1, 0); readB(sb, 1, 1); cp(4); fence();
      group(1, 0); cp(5); fence();
      if (next) {
        handover(copy);
        readA(nb, 0, 1); fence();
        group(0, 0); readB(nb, 0, 0); fence();
        group(0, 1); readA(nb, 0, 0); readB(nb, 0, 1); fence();
      } else {
        group(0, 0); group(0, 1); fence();
      }
    }
  };

#pragma unroll
  for (int j = 0; j < kDmaPerWave; ++j) dma(0, j);
#pragma unroll
  for (int j = 0; j < kDmaPerWave; ++j) dma(1, j);   // nst >= 2 by padding
  if (arrive) xcd_lockstep(arrive, nblocks, slots);
  wait_vm_lgkm0<kDmaPerWave>();   // stage 0 landed
  block_sync();
  // k fragment 0 of stage 0, in the order in which a stage reads the next
  // stage's (so the waits at the top of the loop are the same on entry)
  if constexpr (!kSkipA1B1) {
    readA(lds, 0, 0);
    readB(lds, 0, 0);
    readA(lds, 0, 1);
    readB(lds, 0, 1);
  } else {
    readA(lds, 0, 1);
    readB(lds, 0, 0);
    readA(lds, 0, 0);
    readB(lds, 0, 1);
  }
  fence();

  int s = 0;
  for (; s + 2 < nst; ++s) stage(s, true, true);   // steady state: stage s + 2 exists
  stage(s, false, true);
  stage(s + 1, false, false);

  store_residues_by_k<kSkipA1B1, 2>(acc, kblocks * kFragK, mc->m[l], R + (int64_t)l * rplane, ldr,
                                    tm * kTileM + wm * 64, tn * kTileN + wn * 64, lane);
}

}  // namespace ozfp4
