// Main loop of the short GEMMs over three limbs per operand: the INT8 GEMM's
// (Sec. III, igemm.hip) and scheme I's (Sec. IV, ozaki1_short.hip).
//
// Block tile 128 x 64, four waves (one per SIMD) of 64 x 32 with five
// accumulator sets (limb sums 0..4), k in stages of one 64-wide fragment: 18
// fragments (A: 3 planes x 4 line blocks, then B: 3 planes x 2), 18 KiB, in
// a 4-slot LDS ring of 72 KiB. Two such blocks fit a CU, and one's first
// copies, epilogue and stores run under the other's MFMAs; the 128 x 128
// block of the long GEMMs has its CU to itself. The price is half as many
// operand bytes per MFMA again (256 against 171).
//
// Fragment f of a stage is copied by wave f % 4 as its copy f / 4, so waves 0
// and 1 issue five copies a stage and waves 2 and 3 four.
#pragma once

#include "device_common.hpp"
#include "routes.hpp"

namespace ozfp4 {

constexpr int kL3Waves = 4;
constexpr int kL3Ring = 4;
constexpr int kL3Frags = 18;
constexpr int kL3Stage = kL3Frags * kFragBytes;
constexpr int kL3Dma = 5;

__device__ __forceinline__ constexpr int fragAl3(int p, int rb) { return (p * 4 + rb) * kFragBytes; }
__device__ __forceinline__ constexpr int fragBl3(int p, int cb) { return (12 + p * 2 + cb) * kFragBytes; }

// Adds the products of `total` (>= 1) stages into acc. copy(j) issues this
// wave's copy j of the next stage to be copied into its slot, advance() goes
// on to the following stage; both are called in stage order.
template <class Copy, class Advance>
__device__ __forceinline__ void limb3_short_run(const uint8_t* lds, int total, int wave, int lane16,
                                                Copy&& copy_frag, Advance&& advance,
                                                v16f (&acc)[5][2]) {
  const int rbw = 2 * (wave >> 1), wn = wave & 1;   // first A line block; B line block
  const bool five = wave < 2;
  // at most `stages` (0..3) newer stages' copies of this wave in flight
  auto wait = [&](int stages) {
    if (stages >= 3) {
      if (five) wait_vm_lgkm0<15>(); else wait_vm_lgkm0<12>();
    } else if (stages == 2) {
      if (five) wait_vm_lgkm0<10>(); else wait_vm_lgkm0<8>();
    } else if (stages == 1) {
      if (five) wait_vm_lgkm0<5>(); else wait_vm_lgkm0<4>();
    } else {
      wait_vm_lgkm0<0>();
    }
  };

  v4i a[3][2], b[3];
  auto group = [&](int p, int q) {
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[p + q][i] = mfma_fp4(a[p][i], b[q], acc[p + q][i]);
  };
  auto readA = [&](const uint8_t* sb, int p) {
#pragma unroll
    for (int i = 0; i < 2; ++i) a[p][i] = *reinterpret_cast<const v4i*>(sb + fragAl3(p, rbw + i) + lane16);
  };
  auto readB = [&](const uint8_t* sb, int p) {
    b[p] = *reinterpret_cast<const v4i*>(sb + fragBl3(p, wn) + lane16);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

  // Stage s multiplies the operands in registers, and as a register's last
  // group has been issued refills it for stage s + 1 (every read has at least
  // two groups, four MFMAs of the wave, to land in). The handover after the
  // first group makes stage s + 1 visible and frees the slot of stage s,
  // which takes stage s + 4. `after`: stages after s.
  auto stage = [&](int s, int after) {
    const uint8_t* nb = lds + ((s + 1) % kL3Ring) * kL3Stage;
    const bool next = after > 0, copy = after >= kL3Ring;
    auto cp = [&](int j) {
      if (copy) copy_frag(j);
    };
    group(0, 0); fence();
    if (next) {
      wait(min(after - 1, 2));
      block_sync();
    }
    group(0, 1); cp(0); fence();
    group(0, 2); fence(); if (next) readA(nb, 0); fence();
    group(1, 0); cp(1); fence();
    group(2, 0); fence(); if (next) readB(nb, 0); fence();
    group(1, 1); cp(2); fence();
    group(1, 2); fence(); if (next) readA(nb, 1); fence();
    group(2, 1); cp(3); fence(); if (next) readB(nb, 1); fence();
    group(2, 2); if (copy && five) copy_frag(4); fence();
    if (next) { readA(nb, 2); readB(nb, 2); }
    fence();
    if (copy) advance();
  };

  const int first = min(total, kL3Ring);
  for (int st = 0; st < first; ++st) {
#pragma unroll
    for (int j = 0; j < 4; ++j) copy_frag(j);
    if (five) copy_frag(4);
    advance();
  }
  wait(first - 1);
  block_sync();
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    readA(lds, p);
    readB(lds, p);
  }
  fence();
  int s = 0;
  for (; s + kL3Ring < total; ++s) stage(s, kL3Ring);
  for (; s < total; ++s) stage(s, total - 1 - s);
}

}  // namespace ozfp4
