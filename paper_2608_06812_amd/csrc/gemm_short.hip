// The residue GEMM for short products: few stages or few tiles. A
// translation unit of its own, so nothing here can change how the compiler
// schedules the default kernels.
#include <algorithm>

#include "device_common.hpp"
#include "gemm_short.hpp"

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
constexpr int kShortWaves = 4;
constexpr int kShortRing = 4;
constexpr int kShortFrags = 16;
constexpr int kShortStage = kShortFrags * kFragBytes;
constexpr int kShortDma = kShortFrags / kShortWaves;   // 4

// Up to 64 tiles an XCD takes whole moduli: eight XCDs with eight tiles or
// fewer of each modulus fetch every panel into most L2s (512 x 512 x 4096:
// 58 us at 5.1 TB/s from beyond L2, 46 us with whole moduli; 1024^3 41.9 and
// 39.5); at 256 tiles the shared order is ahead again (2048^3 228 and 231).
constexpr unsigned kShortMinShare = 72;

// LDS offset of fragment (plane p, line block rb / cb)
__device__ __forceinline__ constexpr int fragAs(int p, int rb) { return (p * 4 + rb) * kFragBytes; }
__device__ __forceinline__ constexpr int fragBs(int p, int cb) { return (8 + p * 4 + cb) * kFragBytes; }

template <bool kSkipA1B1>
__device__ __forceinline__ void gemm_short_tile(
    uint8_t* lds, int l, int64_t tm, int64_t tn, const uint8_t* __restrict__ PA,
    const uint8_t* __restrict__ PB, uint8_t* __restrict__ Rl, int64_t plane_a, int64_t plane_b,
    int64_t kblocks, int st0, int nst, int64_t ldr, int m) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int rbw = 2 * wm, cbw = 2 * wn;   // this wave's first A / B line block

  // Wave w copies operand w / 2, plane w % 2: its four line blocks j. The
  // line blocks are kblocks KiB apart; stage s is st0 + s KiB into each. One
  // descriptor covers all (4 kblocks KiB, below 2^31 for k <= 2^24).
  const uint8_t* base = wave < 2 ? PA + (int64_t)(2 * l + wave) * plane_a + tm * 4 * kblocks * kFragBytes
                                 : PB + (int64_t)(2 * l + wave - 2) * plane_b + tn * 4 * kblocks * kFragBytes;
  const uint32_t row = (uint32_t)(kblocks * kFragBytes);
  const __amdgpu_buffer_rsrc_t src =
      __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(4 * row), kBufferWord3);
  const int lane16 = lane * 16;
  auto dma = [&](int st, int j) {
    dma16_buf(src, (uint32_t)lane16, (uint32_t)j * row + (uint32_t)(st0 + st) * kFragBytes,
              lds + (st % kShortRing) * kShortStage + (wave * kShortDma + j) * kFragBytes);
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

  v4i a[2][2], b[2][2];   // [plane][i] of A, [plane][j] of B
  auto readA = [&](const uint8_t* sb, int p) {
#pragma unroll
    for (int i = 0; i < 2; ++i) a[p][i] = *reinterpret_cast<const v4i*>(sb + fragAs(p, rbw + i) + lane16);
  };
  auto readB = [&](const uint8_t* sb, int p) {
#pragma unroll
    for (int j = 0; j < 2; ++j) b[p][j] = *reinterpret_cast<const v4i*>(sb + fragBs(p, cbw + j) + lane16);
  };
  auto group = [&](int p, int q) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[p + q][i][j] = mfma_fp4(a[p][i], b[q][j], acc[p + q][i][j]);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

  // Stage s multiplies the operands in registers and reads those of stage
  // s + 1 as registers free up (the product groups' order alternates as in
  // the default tile). The handover after the first group (stage s + 1
  // landed, with the copies of the newer stages still in flight; the reads
  // of stage s done; a barrier) also frees the slot of stage s, which takes
  // stage s + 4. `after` is the number of stages after s.
  auto stage = [&](auto odd, int s, int after) {
    constexpr bool kOdd = decltype(odd)::value;
    const uint8_t* nb = lds + ((s + 1) % kShortRing) * kShortStage;
    const bool next = after > 0, copy = after >= kShortRing;
    auto handover = [&] {
      if (after >= 3)
        wait_vm_lgkm0<2 * kShortDma>();
      else if (after == 2)
        wait_vm_lgkm0<kShortDma>();
      else
        wait_vm_lgkm0<0>();
      block_sync();
    };
    auto cp = [&](int j) {
      if (copy) dma(s + kShortRing, j);
    };
    if constexpr (!kSkipA1B1) {
      if constexpr (!kOdd) {
        group(0, 0); fence();
        if (next) handover();
        group(0, 1); cp(0); fence();
        if (next) readA(nb, 0);
        group(1, 1); cp(1); fence();
        if (next) readB(nb, 1);
        group(1, 0); cp(2); cp(3); fence();
        if (next) { readA(nb, 1); readB(nb, 0); }
        fence();
      } else {
        group(0, 1); fence();
        if (next) handover();
        group(0, 0); cp(0); fence();
        if (next) readA(nb, 0);
        group(1, 0); cp(1); fence();
        if (next) readB(nb, 0);
        group(1, 1); cp(2); cp(3); fence();
        if (next) { readA(nb, 1); readB(nb, 1); }
        fence();
      }
    } else {
      group(1, 0); fence();
      if (next) handover();
      if (next) readA(nb, 1);
      group(0, 0); cp(0); cp(1); fence();
      if (next) readB(nb, 0);
      group(0, 1); cp(2); cp(3); fence();
      if (next) { readA(nb, 0); readB(nb, 1); }
      fence();
    }
  };
  typedef std::integral_constant<bool, false> Even;
  typedef std::integral_constant<bool, true> Odd;

  // the first stages' copies, then stage 0's operands in the order in which
  // a stage reads the next one's
  const int first = nst < kShortRing ? nst : kShortRing;
  for (int st = 0; st < first; ++st) {
#pragma unroll
    for (int j = 0; j < kShortDma; ++j) dma(st, j);
  }
  if (first == 4)
    wait_vm_lgkm0<3 * kShortDma>();
  else if (first == 3)
    wait_vm_lgkm0<2 * kShortDma>();
  else if (first == 2)
    wait_vm_lgkm0<kShortDma>();
  else
    wait_vm_lgkm0<0>();
  block_sync();
  if constexpr (!kSkipA1B1) {
    readA(lds, 0);
    readB(lds, 0);
    readA(lds, 1);
    readB(lds, 1);
  } else {
    readA(lds, 1);
    readB(lds, 0);
    readA(lds, 0);
    readB(lds, 1);
  }
  fence();

  int s = 0;
  for (; s + kShortRing + 1 < nst; s += 2) {   // both stages have a copy to issue
    stage(Even{}, s, kShortRing);
    stage(Odd{}, s + 1, kShortRing);
  }
  for (; s < nst; s += 2) {
    stage(Even{}, s, nst - 1 - s);
    if (s + 1 < nst) stage(Odd{}, s + 1, nst - 2 - s);
  }

  store_residues_by_k<kSkipA1B1, 1>(acc, (int64_t)nst * kFragK, m, Rl, ldr,
                                    tm * kShortTile + wm * 64, tn * kShortTile + wn * 64, lane);
}

// Block order: sets (product, k range) take the place of moduli in the tile
// mapping, each with its nmod moduli.
__global__ __launch_bounds__(kShortWaves * 64, 2) void k_gemm_short(ShortGemm g, int nst,
                                                                    int64_t tiles_m,
                                                                    int64_t tiles_n,
                                                                    int64_t nblocks) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kShortRing * kShortStage];
  int u;
  int64_t tm, tn;
  tile_coords(blockIdx.x, nblocks, tiles_m, tiles_n, &u, &tm, &tn, kShortMinShare);
  const int set = u / g.nmod, l = u - set * g.nmod;
  const int q = set / g.nsplit, part = set - q * g.nsplit;
  const int st0 = nst * part / g.nsplit, st1 = nst * (part + 1) / g.nsplit;
  const uint8_t* pa = g.pa + (q >> 1) * g.term_a;
  const uint8_t* pb = g.pb + (q & 1) * g.term_b;
  uint8_t* Rl = (part == 0 ? g.R + q * g.rset
                           : g.partial + (int64_t)(q * (g.nsplit - 1) + part - 1) * g.nmod * g.rplane) +
                l * g.rplane;
  const int m = g.mc->m[l];
  if (m == 169)
    gemm_short_tile<true>(lds, l, tm, tn, pa, pb, Rl, g.plane_a, g.plane_b, g.kblocks, st0,
                          st1 - st0, g.ldr, m);
  else
    gemm_short_tile<false>(lds, l, tm, tn, pa, pb, Rl, g.plane_a, g.plane_b, g.kblocks, st0,
                           st1 - st0, g.ldr, m);
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

int stages_of(int64_t k) { return (int)((k + kFragK - 1) / kFragK); }

}  // namespace

// Estimated time in us of the blocks cut into ns ranges each. 512 blocks run
// at a time, two a CU; a stage takes 0.47 us there, 0.27 us where the last
// round leaves every block its own CU; 2.5 us around a block's stages; the
// second launch 4.5 us and the partial residues' traffic. Measured (GEMM
// stage, one range / the ranges this chooses): 128 x 128 x 8192, 19 moduli,
// 38.5 / 18.2 us; 128 x 128 x 2048 15.4 / 13.3; 300 x 300 x 20000 112 / 87;
// 7 x 5 x 50000 202 / 55; 500 x 400 x 60000 615 / 311 (513 with 256 x 128
// tiles); no case of 64 .. 1024 a side slower.
static double short_gemm_us(int64_t blocks, int nst, int ns, double residues) {
  const int64_t total = blocks * ns, rounds = total / 512, rest = total % 512;
  const double stages = (double)((nst + ns - 1) / ns);
  double t = (double)rounds * (stages * 0.47 + 2.5);
  if (rest > 0) t += stages * (rest <= 256 ? 0.27 : 0.47) + 2.5;
  if (ns > 1) t += 4.5 + 0.3 * ns + (double)(ns - 1) * residues * 2.0 / 4e6;
  return t;
}

int short_gemm_split(int64_t m, int64_t n, int64_t k, int nmod, int nprod) {
  const int64_t blocks = ((m + kShortTile - 1) / kShortTile) * ((n + kShortTile - 1) / kShortTile) *
                         nmod * nprod;
  const int nst = stages_of(k);
  if (blocks == 0 || blocks > 1024) return 1;   // two rounds and more: nothing to gain
  const double residues = (double)(m * n) * nmod * nprod;
  int best = 1;
  for (int ns = 2; ns <= 16 && nst / ns >= 8; ++ns)
    if (short_gemm_us(blocks, nst, ns, residues) < short_gemm_us(blocks, nst, best, residues))
      best = ns;
  return best;
}

hipError_t launch_gemm_short(hipStream_t stream, const ShortGemm& g) {
  const int64_t tiles_m = (g.m + kShortTile - 1) / kShortTile;
  const int64_t tiles_n = (g.n + kShortTile - 1) / kShortTile;
  const int64_t nblocks = tiles_m * tiles_n * g.nmod * g.nprod * g.nsplit;
  hipLaunchKernelGGL(k_gemm_short, dim3((unsigned)nblocks), dim3(kShortWaves * 64), 0, stream, g,
                     stages_of(g.k), tiles_m, tiles_n, nblocks);
  if (g.nsplit > 1) {
    const uint32_t rows4 = (uint32_t)((g.m + 3) / 4), threads = rows4 * (uint32_t)g.n;
    hipLaunchKernelGGL(k_add_partials, dim3((threads + 255) / 256, g.nmod * g.nprod), dim3(256), 0,
                       stream, g, rows4, threads);
  }
  return hipGetLastError();
}

}  // namespace ozfp4
