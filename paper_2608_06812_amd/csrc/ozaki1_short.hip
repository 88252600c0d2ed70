// Scheme I's limb-product GEMM for short products (Sec. IV, Lemma 2). A
// translation unit of its own, so nothing here can change how the compiler
// schedules the long one.
//
// A work unit is one 128 x 64 output tile of one block anti-diagonal h, as in
// the long GEMM: it runs every block pair (I, J = h - I) in turn through the
// same five accumulators, here as one sequence of npairs * nst stages of the
// main loop of limb3_short.hpp. Exactness: at most 15 products of magnitude
// <= 64 (doubled limbs) a k, so |4 acc| <= 960 k < 2^23 for k <= 8192: the
// accumulators and the 24-bit multiplies are exact.
#include "device_common.hpp"
#include "limb3_short.hpp"
#include "ozaki1.hpp"

namespace ozfp4 {

namespace {

typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(kL3Waves * 64, 2) void k_gemm_ozi_short(
    const uint8_t* __restrict__ PA, const uint8_t* __restrict__ PB, int64_t* __restrict__ H,
    int64_t plane_a, int64_t plane_b, int64_t kblocks, int nst, int64_t tiles_m, int64_t tiles_n,
    int64_t ldh, int64_t hplane, int nblk) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kL3Ring * kL3Stage];
  // The anti-diagonals differ in work, so every XCD takes an eighth of the
  // tiles of each in turn (a grid of tiles that 8 does not divide has blocks
  // without a tile: contiguous ranges would give XCD 0 the longest units,
  // 156 us instead of 110 at 1500 x 700 x 1500, 12 limbs).
  const unsigned T = (unsigned)(tiles_m * tiles_n), per = (T + 7) >> 3;
  const unsigned local = blockIdx.x >> 3, l = local / per;
  const unsigned t = (blockIdx.x & 7) * per + (local - l * per);
  if (t >= T) return;
  const unsigned span = kGroupM * (unsigned)tiles_n, tg = t / span;
  const unsigned gm = min((unsigned)tiles_m - tg * kGroupM, (unsigned)kGroupM);
  const unsigned in = t - tg * span;
  const int64_t tn = in / gm, tm = tg * kGroupM + in % gm;
  // the middle ones, which carry the most pairs, come first
  const int dist = (int)(l + 1) >> 1;
  const int h = (l & 1) ? nblk - 1 - dist : nblk - 1 + dist;
  const int I0 = h - nblk + 1 > 0 ? h - nblk + 1 : 0;
  const int I1 = h < nblk - 1 ? h : nblk - 1;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // fragment f = wave + 4 j of a stage (waves 2 and 3: j < 4); a pair further
  // on, A's block is the next one and B's the one before
  const uint8_t* base[kL3Dma];
  int64_t step[kL3Dma];
  __amdgpu_buffer_rsrc_t src[kL3Dma];
  auto source = [&](int j) {
    src[j] = __builtin_amdgcn_make_buffer_rsrc((void*)base[j], (short)0, nst * kFragBytes, kBufferWord3);
  };
#pragma unroll
  for (int j = 0; j < kL3Dma; ++j) {
    const int f = min(wave + 4 * j, kL3Frags - 1);
    if (f < 12) {
      base[j] = PA + (int64_t)(3 * I0 + (f >> 2)) * plane_a + (tm * 4 + (f & 3)) * kblocks * kFragBytes;
      step[j] = 3 * plane_a;
    } else {
      base[j] = PB + (int64_t)(3 * (h - I0) + ((f - 12) >> 1)) * plane_b +
                (tn * 2 + (f & 1)) * kblocks * kFragBytes;
      step[j] = -3 * plane_b;
    }
    source(j);
  }
  const int lane16 = lane * 16;
  int copied = 0, copied_st = 0;   // next stage to copy: of the run, of its pair
  auto copy = [&](int j) {
    dma16_buf(src[j], (uint32_t)lane16, (uint32_t)(copied_st * kFragBytes),
              lds + (copied % kL3Ring) * kL3Stage + (wave + 4 * j) * kFragBytes);
  };
  auto advance = [&] {
    ++copied;
    if (++copied_st == nst) {
      copied_st = 0;
#pragma unroll
      for (int j = 0; j < kL3Dma; ++j) {
        base[j] += step[j];
        source(j);
      }
    }
  };
  v16f acc[5][2];
#pragma unroll
  for (int e = 0; e < 5; ++e)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[e][i][v] = 0.0f;
  limb3_short_run(lds, (I1 - I0 + 1) * nst, wave, lane16, copy, advance, acc);

  // H_h = sum_g 13^g 4 acc_g: the first two terms in 32 bits (the first three
  // would fit too, below 183 * 2^23 < 2^31), the others in 64; the tile lies
  // inside the padded planes
  int64_t* dst0 = H + (int64_t)h * hplane + (tn * kL3TileN + wn * 32 + (lane & 31)) * ldh +
                  tm * kL3TileM + wm * 64 + (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      int64_t val[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = 4 * q + e;
        // |4 acc0 + 13 * 4 acc1| < 14 * 2^23 fits 32 bits
        const int low = (int)(4.0f * acc[0][i][v]) + __mul24((int)(4.0f * acc[1][i][v]), 13);
        val[e] = (int64_t)low + (int64_t)(int)(4.0f * acc[2][i][v]) * 169 +
                 (int64_t)(int)(4.0f * acc[3][i][v]) * 2197 +
                 (int64_t)(int)(4.0f * acc[4][i][v]) * 28561;
      }
      i64x2* dst = reinterpret_cast<i64x2*>(dst0 + i * 32 + q * 8);
      dst[0] = i64x2{val[0], val[1]};
      dst[1] = i64x2{val[2], val[3]};
    }
}

}  // namespace

hipError_t launch_gemm_ozi_short(hipStream_t stream, const uint8_t* PA, const uint8_t* PB,
                                 int64_t* H, int64_t plane_a, int64_t plane_b, int64_t kblocks,
                                 int64_t m, int64_t n, int64_t k, int64_t m_pad, int64_t n_pad,
                                 int nblk) {
  const int64_t tiles_m = (m + kL3TileM - 1) / kL3TileM, tiles_n = (n + kL3TileN - 1) / kL3TileN;
  const int64_t nblocks = (tiles_m * tiles_n + 7) / 8 * 8 * (2 * nblk - 1);
  const int nst = (int)((k + kFragK - 1) / kFragK);
  hipLaunchKernelGGL(k_gemm_ozi_short, dim3((unsigned)nblocks), dim3(kL3Waves * 64), 0, stream, PA,
                     PB, H, plane_a, plane_b, kblocks, nst, tiles_m, tiles_n, m_pad, m_pad * n_pad,
                     nblk);
  return hipGetLastError();
}

}  // namespace ozfp4
