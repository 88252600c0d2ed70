// The INT8 path (Sec. III): encoder of both operands and the GEMM for short
// products. A translation unit of its own, so nothing here can change how
// the compiler schedules the other GEMMs.
#include <algorithm>

#include "device_common.hpp"
#include "igemm.hpp"
#include "limb3_short.hpp"
#include "routes.hpp"

namespace ozfp4 {

namespace {

// ------------------------------------------------------------ encoder
// Three greedy limbs per value from a 256-entry table in LDS (codes of c0,
// c1, c2 in the low nibbles of bytes 0, 1, 2, so that a pair of values is
// E0 | E1 << 4 and byte permutes gather a plane's word), one wave per
// fragment, four fragments of adjacent line blocks per block.
//
// Bound by HBM (1 B read and 1.5 B written a value). Lines along k are read
// as two 16-byte words a lane. Adjacent lines are read as 32-bit words of
// four lines (128 lines, 128 bytes, a row of k), transposed 4 x 4 in
// registers and handed to the lane that owns the line through LDS; 8192 x
// 8192 takes 45 us (A) and 45 us (B); byte loads of either form took 119 and
// 161 us.
constexpr int kS8Waves = 4;
constexpr int kS8Lines = kS8Waves * kFragLines;   // lines of a block
constexpr int kS8Row = kFragK + 16;               // LDS bytes of a line, 16-byte aligned

__device__ __forceinline__ uint32_t pair_codes(const uint32_t* lut, uint32_t w, int sh) {
  return lut[(w >> sh) & 0xffu] | (lut[(w >> (sh + 8)) & 0xffu] << 4);
}

__global__ __launch_bounds__(256) void k_encode_s8(S8Operand a, S8Operand b, uint32_t blocks_a,
                                                   const uint16_t* __restrict__ lut8) {
  __shared__ uint32_t s_lut[256];
  __shared__ __attribute__((aligned(16))) uint8_t s_x[kS8Lines * kS8Row];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  {
    const uint32_t e = lut8[tid ^ 128];   // table index: the byte itself
    s_lut[tid] = (e & 0xfu) | ((e >> 4) & 0xfu) << 8 | ((e >> 8) & 0xfu) << 16;
  }
  const bool is_b = blockIdx.x >= blocks_a;
  const uint32_t first = is_b ? blockIdx.x - blocks_a : blockIdx.x;
  const uint32_t step = is_b ? gridDim.x - blocks_a : blocks_a;
  const S8Operand& op = is_b ? b : a;
  const int64_t lines = op.lines, k = op.k;
  const uint32_t groups = (op.blocks + kS8Waves - 1) / kS8Waves;   // of four line blocks
  const uint32_t units = groups * op.kfrags;
  __syncthreads();
  for (uint32_t u = first; u < units; u += step) {
    const uint32_t group = u / op.kfrags, kb = u - group * op.kfrags;
    const int64_t line0 = (int64_t)group * kS8Lines, k0 = (int64_t)kb * kFragK;
    const int64_t line = line0 + wave * kFragLines + (lane & 31);
    const int64_t kbase = k0 + (lane >> 5) * 32;
    uint32_t x[8];   // this lane's 32 values, four a word, zero beyond the operand
    if (op.ks == 1) {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = 0;
      if (line < lines) {
        const int8_t* src = op.X + line * op.rs + kbase;
        if (kbase + 32 <= k) {
          __builtin_memcpy(x, src, 32);
        } else {
          for (int e = 0; e < 32; ++e)
            if (kbase + e < k) x[e >> 2] |= (uint32_t)(uint8_t)src[e] << (8 * (e & 3));
        }
      }
    } else {
      // patch (4 lines x 4 k): thread = line group + 32 * k group, two each
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int lg = tid & 31, kg = (tid >> 5) + 8 * h;
        const int64_t l = line0 + 4 * lg;
        uint32_t r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t kk = k0 + 4 * kg + e;
          r[e] = 0;
          if (kk < k && l < lines) {
            const int8_t* src = op.X + l + kk * op.ks;
            if (l + 4 <= lines) {
              __builtin_memcpy(&r[e], src, 4);
            } else {
              for (int q = 0; q < 4; ++q)
                if (l + q < lines) r[e] |= (uint32_t)(uint8_t)src[q] << (8 * q);
            }
          }
        }
        // word q of the transpose: line l + q, k 4 kg .. + 3
        const uint32_t lo01 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u);
        const uint32_t lo23 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u);
        const uint32_t hi01 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
        const uint32_t hi23 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
        uint8_t* dst = s_x + (4 * lg) * kS8Row + 4 * kg;
        *reinterpret_cast<uint32_t*>(dst) = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
        *reinterpret_cast<uint32_t*>(dst + kS8Row) = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
        *reinterpret_cast<uint32_t*>(dst + 2 * kS8Row) = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
        *reinterpret_cast<uint32_t*>(dst + 3 * kS8Row) = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
      }
      __syncthreads();
      const uint8_t* src = s_x + (wave * kFragLines + (lane & 31)) * kS8Row + (lane >> 5) * 32;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const v4i v = *reinterpret_cast<const v4i*>(src + 16 * e);
#pragma unroll
        for (int q = 0; q < 4; ++q) x[4 * e + q] = (uint32_t)v[q];
      }
      __syncthreads();   // the rows are rewritten by the next unit
    }
    const uint32_t rb = group * kS8Waves + wave;
    if (rb >= op.blocks) continue;
    uint32_t w[3][4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint32_t p[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) p[h] = pair_codes(s_lut, x[2 * g + (h >> 1)], 16 * (h & 1));
      const uint32_t t01 = __builtin_amdgcn_perm(p[1], p[0], 0x05010400u);
      const uint32_t t23 = __builtin_amdgcn_perm(p[3], p[2], 0x05010400u);
      w[0][g] = __builtin_amdgcn_perm(t23, t01, 0x05040100u);
      w[1][g] = __builtin_amdgcn_perm(t23, t01, 0x07060302u);
      const uint32_t s01 = __builtin_amdgcn_perm(p[1], p[0], 0x00000602u);
      const uint32_t s23 = __builtin_amdgcn_perm(p[3], p[2], 0x00000602u);
      w[2][g] = __builtin_amdgcn_perm(s23, s01, 0x05040100u);
    }
    uint8_t* out = op.planes + ((int64_t)rb * op.kblocks + kb) * kFragBytes + lane * 16;
#pragma unroll
    for (int p = 0; p < 3; ++p)
      *reinterpret_cast<v4i*>(out + (int64_t)p * op.plane_bytes) =
          v4i{(int)w[p][0], (int)w[p][1], (int)w[p][2], (int)w[p][3]};
  }
}

// ------------------------------------------------------------ short GEMM
// The main loop of limb3_short.hpp over one k range of one 128 x 64 tile.
__global__ __launch_bounds__(kL3Waves * 64, 2) void k_gemm_s8_short(ShortS8 g, int nst_all,
                                                                     int64_t tiles_m,
                                                                     int64_t tiles_n,
                                                                     int64_t nblocks) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kL3Ring * kL3Stage];
  int part;
  int64_t tm, tn;
  tile_coords(blockIdx.x, nblocks, tiles_m, tiles_n, &part, &tm, &tn, 72);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int st0 = (int)((int64_t)nst_all * part / g.nsplit);
  const int nst = (int)((int64_t)nst_all * (part + 1) / g.nsplit) - st0;

  // fragment f = wave + 4 j of a stage (waves 2 and 3: j < 4)
  __amdgpu_buffer_rsrc_t src[kL3Dma];
#pragma unroll
  for (int j = 0; j < kL3Dma; ++j) {
    const int f = min(wave + 4 * j, kL3Frags - 1);
    const uint8_t* base;
    if (f < 12)
      base = g.pa + (int64_t)(f >> 2) * g.plane_a +
             ((tm * 4 + (f & 3)) * g.kblocks + st0) * kFragBytes;
    else
      base = g.pb + (int64_t)((f - 12) >> 1) * g.plane_b +
             ((tn * 2 + (f & 1)) * g.kblocks + st0) * kFragBytes;
    src[j] = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, nst * kFragBytes, kBufferWord3);
  }
  const int lane16 = lane * 16;
  int copied = 0;   // next stage to copy
  auto copy = [&](int j) {
    dma16_buf(src[j], (uint32_t)lane16, (uint32_t)(copied * kFragBytes),
              lds + (copied % kL3Ring) * kL3Stage + (wave + 4 * j) * kFragBytes);
  };
  v16f acc[5][2];
#pragma unroll
  for (int e = 0; e < 5; ++e)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[e][i][v] = 0.0f;
  limb3_short_run(lds, nst, wave, lane16, copy, [&] { ++copied; }, acc);

  // sum_g 13^g 4 acc_g: |4 acc_g| <= 192 k < 2^23 for k <= 40960, so the
  // 24-bit multiplies are exact; the sum wraps modulo 2^32
  const bool direct = g.nsplit == 1;
  int32_t* C = direct ? g.C : g.partial + (int64_t)part * g.m_pad * g.n_pad;
  const int64_t ldc = direct ? g.ldc : g.m_pad, m = direct ? g.m : g.m_pad, n = direct ? g.n : g.n_pad;
  const int64_t col = tn * kL3TileN + wn * 32 + (lane & 31);
  const int64_t row0 = tm * kL3TileM + wm * 64 + (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v4i out;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = 4 * q + e;
        uint32_t x = (uint32_t)(int)(4.0f * acc[0][i][v]);
        x += (uint32_t)__mul24((int)(4.0f * acc[1][i][v]), 13);
        x += (uint32_t)__mul24((int)(4.0f * acc[2][i][v]), 169);
        x += (uint32_t)__mul24((int)(4.0f * acc[3][i][v]), 2197);
        x += (uint32_t)__mul24((int)(4.0f * acc[4][i][v]), 28561);
        out[e] = (int)x;
      }
      const int64_t r = row0 + i * 32 + q * 8;
      int32_t* dst = C + r + col * ldc;
      if (col < n && r + 3 < m && ((uintptr_t)dst & 15) == 0) {
        *reinterpret_cast<v4i*>(dst) = out;
      } else if (col < n) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (r + e < m) dst[e] = out[e];
      }
    }
}

// C = sum of the ranges' partial sums, modulo 2^32
__global__ __launch_bounds__(256) void k_add_partials_s8(ShortS8 g, uint32_t threads) {
  const uint32_t t = blockIdx.x * 256 + threadIdx.x;
  if (t >= threads) return;
  const uint32_t col = t / (uint32_t)g.m, row = t - col * (uint32_t)g.m;
  const int32_t* x = g.partial + (int64_t)col * g.m_pad + row;
  uint32_t sum = 0;
#pragma unroll 4
  for (int part = 0; part < g.nsplit; ++part) sum += (uint32_t)x[(int64_t)part * g.m_pad * g.n_pad];
  g.C[(int64_t)col * g.ldc + row] = (int32_t)sum;
}

}  // namespace

hipError_t launch_encode_s8(hipStream_t stream, const S8Operand& a, const S8Operand& b,
                            const uint16_t* lut8) {
  auto blocks = [](const S8Operand& op) {
    const int64_t units = (int64_t)((op.blocks + kS8Waves - 1) / kS8Waves) * op.kfrags;
    return (uint32_t)std::min<int64_t>(units, 256 * 8);
  };
  const uint32_t ba = blocks(a), bb = blocks(b);
  hipLaunchKernelGGL(k_encode_s8, dim3(ba + bb), dim3(256), 0, stream, a, b, ba, lut8);
  return hipGetLastError();
}

hipError_t launch_gemm_s8_short(hipStream_t stream, const ShortS8& g) {
  const int64_t tiles_m = (g.m + kL3TileM - 1) / kL3TileM;
  const int64_t tiles_n = (g.n + kL3TileN - 1) / kL3TileN;
  const int64_t nblocks = tiles_m * tiles_n * g.nsplit;
  hipLaunchKernelGGL(k_gemm_s8_short, dim3((unsigned)nblocks), dim3(kL3Waves * 64), 0, stream, g,
                     stages_of(g.k), tiles_m, tiles_n, nblocks);
  if (g.nsplit > 1) {
    const uint32_t threads = (uint32_t)(g.m * g.n);
    hipLaunchKernelGGL(k_add_partials_s8, dim3((threads + 255) / 256), dim3(256), 0, stream, g, threads);
  }
  return hipGetLastError();
}

}  // namespace ozfp4
