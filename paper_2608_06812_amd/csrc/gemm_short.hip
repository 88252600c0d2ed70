// The residue GEMM for short products: few stages or few tiles. A
// translation unit of its own, so nothing here can change how the compiler
// schedules the default kernels.
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

// LDS offset of fragment (plane p, line block rb / cb)
__device__ __forceinline__ constexpr int fragAs(int p, int rb) { return (p * 4 + rb) * kFragBytes; }
__device__ __forceinline__ constexpr int fragBs(int p, int cb) { return (8 + p * 4 + cb) * kFragBytes; }

template <bool kSkipA1B1>
__device__ __forceinline__ void gemm_short_tile(
    uint8_t* lds, int l, int64_t tm, int64_t tn, const uint8_t* __restrict__ PA,
    const uint8_t* __restrict__ PB, uint8_t* __restrict__ R, int64_t plane_a, int64_t plane_b,
    int64_t kblocks, int nst, int64_t ldr, int64_t rplane, const ModConst* __restrict__ mc) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int rbw = 2 * wm, cbw = 2 * wn;   // this wave's first A / B line block

  // Wave w copies operand w / 2, plane w % 2: its four line blocks j. The
  // line blocks are kblocks KiB apart; stage s is at s KiB in each. One
  // descriptor covers all (4 kblocks KiB, below 2^31 for k <= 2^24).
  const uint8_t* base = wave < 2 ? PA + (int64_t)(2 * l + wave) * plane_a + tm * 4 * kblocks * kFragBytes
                                 : PB + (int64_t)(2 * l + wave - 2) * plane_b + tn * 4 * kblocks * kFragBytes;
  const uint32_t row = (uint32_t)(kblocks * kFragBytes);
  const __amdgpu_buffer_rsrc_t src =
      __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(4 * row), kBufferWord3);
  const int lane16 = lane * 16;
  auto dma = [&](int st, int j) {
    dma16_buf(src, (uint32_t)lane16, (uint32_t)j * row + (uint32_t)st * kFragBytes,
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

  store_residues_by_k<kSkipA1B1, 1>(acc, (int64_t)nst * kFragK, mc->m[l], R + (int64_t)l * rplane,
                                    ldr, tm * kShortTile + wm * 64, tn * kShortTile + wn * 64, lane);
}

__global__ __launch_bounds__(kShortWaves * 64, 2) void k_gemm_short(
    const uint8_t* __restrict__ PA, const uint8_t* __restrict__ PB, uint8_t* __restrict__ R,
    int64_t plane_a, int64_t plane_b, int64_t kblocks, int nst, int64_t tiles_m, int64_t tiles_n,
    int64_t nblocks, int64_t ldr, int64_t rplane, const ModConst* __restrict__ mc) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kShortRing * kShortStage];
  int l;
  int64_t tm, tn;
  tile_coords(blockIdx.x, nblocks, tiles_m, tiles_n, &l, &tm, &tn);
  if (mc->m[l] == 169)
    gemm_short_tile<true>(lds, l, tm, tn, PA, PB, R, plane_a, plane_b, kblocks, nst, ldr, rplane, mc);
  else
    gemm_short_tile<false>(lds, l, tm, tn, PA, PB, R, plane_a, plane_b, kblocks, nst, ldr, rplane, mc);
}

}  // namespace

hipError_t launch_gemm_short(hipStream_t stream, const uint8_t* pa, const uint8_t* pb, uint8_t* R,
                             int64_t ldr, int64_t rplane, int64_t plane_a, int64_t plane_b,
                             int64_t m, int64_t n, int64_t k, int64_t kblocks, int nmod,
                             const ModConst* mc) {
  const int64_t tiles_m = (m + kShortTile - 1) / kShortTile, tiles_n = (n + kShortTile - 1) / kShortTile;
  const int64_t nblocks = tiles_m * tiles_n * nmod;
  const int nst = (int)((k + kFragK - 1) / kFragK);
  hipLaunchKernelGGL(k_gemm_short, dim3((unsigned)nblocks), dim3(kShortWaves * 64), 0, stream, pa,
                     pb, R, plane_a, plane_b, kblocks, nst, tiles_m, tiles_n, nblocks, ldr, rplane,
                     mc);
  return hipGetLastError();
}

}  // namespace ozfp4
