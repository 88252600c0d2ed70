// The residue GEMM for short products: few stages or few tiles. A
// translation unit of its own, so nothing here can change how the compiler
// schedules the default kernels.
#include "device_common.hpp"
#include "gemm_short.hpp"
#include "routes.hpp"

namespace ozfp4 {

namespace {

// Block tile 128 x 128 of one modulus, four waves (one per SIMD) of 64 x 64
// with the default tile's three accumulator sets, k in stages of one 64-wide
// fragment: 16 fragments (A: 2 planes x 4 line blocks, then B the same), 16
// KiB, in a 4-slot LDS ring of 64 KiB. Two such blocks fit a CU (registers
// and LDS), and they are independent: one block's first copies, epilogue and
// stores run under the other's MFMAs. A 256 x 128 block of the default
// kernel has its CU to itself, so a block pays those in full: about 7 us,
// against 0.43 us of MFMA time per k = 64. The price is a third more operand
// bytes per MFMA (256 against 192), which is why long products stay there.
static_assert(kStageShortK == kFragK, "routes and kernel disagree");
constexpr int kShortWaves = 4;
constexpr int kShortRing = 4;
constexpr int kShortFrags = 16;
constexpr int kShortStage = kShortFrags * kFragBytes;
constexpr int kShortDma = kShortFrags / kShortWaves;   // 4

// Up to 64 tiles an XCD takes whole moduli: eight XCDs with eight tiles or
// fewer of each modulus fetch every panel into most L2s. GEMM, us, tiles of a
// modulus shared by the XCDs / whole moduli, 18 moduli, k = 4096: 59.6 / 46.5
// for 16 tiles (512 x 512), 81.1 / 72.4 for 32, 107.5 / 97.8 for 48, 124.1 /
// 122.8 for 64 (1024 x 1024; 43.4 / 39.9 at k = 1024), 148.2 / 147.7 for 80,
// and the other way from 128 on (227.0 / 229.0; 192: 339.8 / 342.9; 256, at
// k = 2048: 231.8 / 234.5).
constexpr unsigned kShortMinShare = 72;

// LDS offset of fragment (plane p, line block rb / cb)
__device__ __forceinline__ constexpr int fragAs(int p, int rb) { return (p * 4 + rb) * kFragBytes; }
__device__ __forceinline__ constexpr int fragBs(int p, int cb) { return (8 + p * 4 + cb) * kFragBytes; }

// The run of one block: one modulus, or (kGrouped) the stages of several
// moduli one after another as one sequence of N = moduli * nst stages through
// the ring, so that the copies of a modulus's first stages are in flight
// during the last stages and the epilogue of the one before it.
struct ShortRun {
  uint8_t* lds;
  __amdgpu_buffer_rsrc_t src;   // this wave's operand plane of the modulus being copied
  const uint8_t* base;
  int64_t plane2;               // bytes from a modulus's planes to the next one's
  uint32_t row;                 // bytes from a line block to the next
  int nst, st0;                 // stages a modulus, the first one's index
  int copied_st;                // kGrouped: next stage to copy
  int total;                    // N
  int wave, lane16, rbw, cbw;
};

__device__ __forceinline__ void short_source(ShortRun& r) {
  r.src = __builtin_amdgcn_make_buffer_rsrc((void*)r.base, (short)0, (int)(4 * r.row), kBufferWord3);
}

template <bool kGrouped>
__device__ __forceinline__ void short_copy(const ShortRun& r, int S, int j) {
  const int st = r.st0 + (kGrouped ? r.copied_st : S);
  dma16_buf(r.src, (uint32_t)r.lane16, (uint32_t)j * r.row + (uint32_t)st * kFragBytes,
            r.lds + (S % kShortRing) * kShortStage + (r.wave * kShortDma + j) * kFragBytes);
}

// After the four copies of a stage: on to the next one.
template <bool kGrouped>
__device__ __forceinline__ void short_advance(ShortRun& r) {
  if (kGrouped && ++r.copied_st == r.nst) {
    r.copied_st = 0;
    r.base += r.plane2;
    short_source(r);
  }
}

// At most `stages` newer stages' copies of this wave in flight. The count
// leaves out the epilogue's stores: they can only make the wait longer.
__device__ __forceinline__ void short_wait(int stages) {
  if (stages >= 3)
    wait_vm_lgkm0<3 * kShortDma>();
  else if (stages == 2)
    wait_vm_lgkm0<2 * kShortDma>();
  else if (stages == 1)
    wait_vm_lgkm0<kShortDma>();
  else
    wait_vm_lgkm0<0>();
}

// Stages S0 .. S0 + nst - 1 of the sequence: one modulus, into acc.
template <bool kSkipA1B1, bool kGrouped>
__device__ __forceinline__ void gemm_short_modulus(ShortRun& r, int S0, v16f (&acc)[3][2][2]) {
  v4i a[2][2], b[2][2];   // [plane][i] of A, [plane][j] of B
  auto readA = [&](const uint8_t* sb, int p) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      a[p][i] = *reinterpret_cast<const v4i*>(sb + fragAs(p, r.rbw + i) + r.lane16);
  };
  auto readB = [&](const uint8_t* sb, int p) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
      b[p][j] = *reinterpret_cast<const v4i*>(sb + fragBs(p, r.cbw + j) + r.lane16);
  };
  auto group = [&](int p, int q) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[p + q][i][j] = mfma_fp4(a[p][i], b[q][j], acc[p + q][i][j]);
  };
  // the first group into an accumulator set starts from the constant zero
  auto first = [&](int p, int q) {
    const v16f zero = {0.0f};
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[p + q][i][j] = mfma_fp4(a[p][i], b[q][j], zero);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

  // Stage s of the modulus multiplies the operands in registers and reads
  // those of stage s + 1 as registers free up (the product groups' order
  // alternates as in the default tile). The handover after the first group
  // (the next stage landed, with the copies of the newer stages still in
  // flight; the reads of this stage done; a barrier) also frees this stage's
  // slot, which takes the stage four on. `next`: the modulus has a stage
  // s + 1; `after`: stages of the whole run after this one.
  auto stage = [&](auto odd, auto fresh, int S, bool next, int after) {
    constexpr bool kOdd = decltype(odd)::value, kFresh = decltype(fresh)::value;
    const uint8_t* nb = r.lds + ((S + 1) % kShortRing) * kShortStage;
    const bool copy = after >= kShortRing;
    auto handover = [&] {
      if (next || (kGrouped && copy)) {   // one modulus: a copy implies a next stage
        short_wait(min(after - 1, 2));
        block_sync();
      }
    };
    auto cp = [&](int j) {
      if (copy) short_copy<kGrouped>(r, S + kShortRing, j);
    };
    auto head = [&](int p, int q) {
      if constexpr (kFresh) first(p, q); else group(p, q);
    };
    if constexpr (!kSkipA1B1) {
      if constexpr (!kOdd) {
        head(0, 0); fence();
        handover();
        head(0, 1); cp(0); fence();
        if (next) readA(nb, 0);
        head(1, 1); cp(1); fence();
        if (next) readB(nb, 1);
        group(1, 0); cp(2); cp(3); fence();
        if (next) { readA(nb, 1); readB(nb, 0); }
      } else {
        group(0, 1); fence();
        handover();
        group(0, 0); cp(0); fence();
        if (next) readA(nb, 0);
        group(1, 0); cp(1); fence();
        if (next) readB(nb, 0);
        group(1, 1); cp(2); cp(3); fence();
        if (next) { readA(nb, 1); readB(nb, 1); }
      }
    } else {
      head(1, 0); fence();
      handover();
      if (next) readA(nb, 1);
      head(0, 0); cp(0); cp(1); fence();
      if (next) readB(nb, 0);
      group(0, 1); cp(2); cp(3); fence();
      if (next) { readA(nb, 0); readB(nb, 1); }
    }
    fence();
    if (copy) short_advance<kGrouped>(r);
  };
  typedef std::integral_constant<bool, false> No;
  typedef std::integral_constant<bool, true> Yes;

  // the first stage's operands in the order in which a stage reads the next
  // one's
  const uint8_t* sb = r.lds + (S0 % kShortRing) * kShortStage;
  short_wait(min(r.total - 1 - S0, kShortRing - 1));
  block_sync();
  if constexpr (!kSkipA1B1) {
    readA(sb, 0);
    readB(sb, 0);
    readA(sb, 1);
    readB(sb, 1);
  } else {
    readA(sb, 1);
    readB(sb, 0);
    readA(sb, 0);
    readB(sb, 1);
  }
  fence();

  const int last = S0 + r.nst - 1, end = r.total - 1;
  stage(No{}, Yes{}, S0, r.nst > 1, end - S0);
  int S = S0 + 1;
  // both stages have a copy and a next stage
  for (; (!kGrouped || S + 1 < last) && S + 1 + kShortRing <= end; S += 2) {
    stage(Yes{}, No{}, S, true, kShortRing);
    stage(No{}, No{}, S + 1, true, kShortRing);
  }
  for (; S <= last; S += 2) {
    stage(Yes{}, No{}, S, S < last, end - S);
    if (S < last) stage(No{}, No{}, S + 1, S + 1 < last, end - S - 1);
  }
}

// Block order: sets (product, k range) times groups of `group` moduli take
// the place of moduli in the tile mapping.
template <bool kGrouped>
__global__ __launch_bounds__(kShortWaves * 64, 2) void k_gemm_short(ShortGemm g, int nst_all,
                                                                    int group, int64_t tiles_m,
                                                                    int64_t tiles_n,
                                                                    int64_t nblocks) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kShortRing * kShortStage];
  int u;
  int64_t tm, tn;
  tile_coords(blockIdx.x, nblocks, tiles_m, tiles_n, &u, &tm, &tn, kShortMinShare);
  const int ngroups = kGrouped ? (g.nmod + group - 1) / group : g.nmod;
  const int set = u / ngroups, l0 = (u - set * ngroups) * (kGrouped ? group : 1);
  const int l1 = kGrouped ? min(g.nmod, l0 + group) : l0 + 1;
  const int q = set / g.nsplit, part = set - q * g.nsplit;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // Wave w copies operand w / 2, plane w % 2: its four line blocks j. The
  // line blocks are kblocks KiB apart; stage s is st0 + s KiB into each. One
  // descriptor covers all (4 kblocks KiB, below 2^31 for k <= 2^24).
  ShortRun r;
  r.lds = lds;
  r.st0 = nst_all * part / g.nsplit;
  r.nst = nst_all * (part + 1) / g.nsplit - r.st0;
  r.total = r.nst * (l1 - l0);
  r.copied_st = 0;
  r.row = (uint32_t)(g.kblocks * kFragBytes);
  r.plane2 = 2 * (wave < 2 ? g.plane_a : g.plane_b);
  r.base = wave < 2 ? g.pa + (q >> 1) * g.term_a + (int64_t)(2 * l0 + wave) * g.plane_a +
                          tm * 4 * g.kblocks * kFragBytes
                    : g.pb + (q & 1) * g.term_b + (int64_t)(2 * l0 + wave - 2) * g.plane_b +
                          tn * 4 * g.kblocks * kFragBytes;
  r.wave = wave;
  r.lane16 = lane * 16;
  r.rbw = 2 * wm;
  r.cbw = 2 * wn;   // this wave's first A / B line block
  short_source(r);
  const int first = min(r.total, kShortRing);
  for (int S = 0; S < first; ++S) {
#pragma unroll
    for (int j = 0; j < kShortDma; ++j) short_copy<kGrouped>(r, S, j);
    short_advance<kGrouped>(r);
  }
  uint8_t* Rset = part == 0 ? g.R + q * g.rset
                            : g.partial + (int64_t)(q * (g.nsplit - 1) + part - 1) * g.nmod * g.rplane;
  v16f acc[3][2][2];
  int S0 = 0;
  for (int l = l0; l < l1; ++l, S0 += r.nst) {
    const int m = g.mc->m[l];
    uint8_t* Rl = Rset + l * g.rplane;
    if (m == 169) {
      gemm_short_modulus<true, kGrouped>(r, S0, acc);
      store_residues_by_k<true, 1>(acc, (int64_t)r.nst * kFragK, m, Rl, g.ldr,
                                   tm * kShortTile + wm * 64, tn * kShortTile + wn * 64, lane);
    } else {
      gemm_short_modulus<false, kGrouped>(r, S0, acc);
      store_residues_by_k<false, 1>(acc, (int64_t)r.nst * kFragK, m, Rl, g.ldr,
                                    tm * kShortTile + wm * 64, tn * kShortTile + wn * 64, lane);
    }
  }
}

// R += the partial residues, modulo m: one thread per four rows of a column
// of one residue plane (blockIdx.y = product and modulus).
__global__ __launch_bounds__(256) void k_add_partials(ShortGemm g, uint32_t rows4,
                                                      uint32_t threads) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t >= threads) return;
  const int q = (int)blockIdx.y / g.nmod, l = (int)blockIdx.y - q * g.nmod;
  const uint32_t col = t / rows4;
  const int64_t off = l * g.rplane + (int64_t)col * g.ldr + (int64_t)(t - col * rows4) * 4;
  uint32_t* r = reinterpret_cast<uint32_t*>(g.R + q * g.rset + off);
  const uint8_t* x = g.partial + (int64_t)q * (g.nsplit - 1) * g.nmod * g.rplane + off;
  uint32_t lo = *r & 0x00ff00ffu, hi = (*r >> 8) & 0x00ff00ffu;   // sums <= 16 * 168
  for (int part = 1; part < g.nsplit; ++part) {
    const uint32_t w = *reinterpret_cast<const uint32_t*>(x);
    lo += w & 0x00ff00ffu;
    hi += (w >> 8) & 0x00ff00ffu;
    x += g.nmod * g.rplane;
  }
  const uint32_t m = (uint32_t)g.mc->m[l];
  *r = ((lo & 0xffffu) % m) | (((hi & 0xffffu) % m) << 8) | (((lo >> 16) % m) << 16) |
       (((hi >> 16) % m) << 24);
}

}  // namespace

hipError_t launch_gemm_short(hipStream_t stream, const ShortGemm& g) {
  const int64_t tiles_m = (g.m + kShortTile - 1) / kShortTile;
  const int64_t tiles_n = (g.n + kShortTile - 1) / kShortTile;
  const int64_t sets = tiles_m * tiles_n * g.nprod * g.nsplit;
  const int nst = stages_of(g.k), group = moduli_per_block(sets * g.nmod, nst, g.nmod);
  const int64_t nblocks = sets * ((g.nmod + group - 1) / group);
  auto kernel = group > 1 ? k_gemm_short<true> : k_gemm_short<false>;
  hipLaunchKernelGGL(kernel, dim3((unsigned)nblocks), dim3(kShortWaves * 64), 0, stream, g, nst,
                     group, tiles_m, tiles_n, nblocks);
  if (g.nsplit > 1) {
    const uint32_t rows4 = (uint32_t)((g.m + 3) / 4), threads = rows4 * (uint32_t)g.n;
    hipLaunchKernelGGL(k_add_partials, dim3((threads + 255) / 256, g.nmod * g.nprod), dim3(256), 0,
                       stream, g, rows4, threads);
  }
  return hipGetLastError();
}

}  // namespace ozfp4
