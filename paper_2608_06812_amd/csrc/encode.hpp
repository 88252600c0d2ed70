// The fused encoder of scheme II (device template) and its launch.
#pragma once

#include <algorithm>

#include "convert.hpp"
#include "device_common.hpp"
#include "encode_address.hpp"

namespace ozfp4 {

// ------------------------------------------------------------ Sec. V-A / VI-B
// Fused integer conversion, residues for every modulus, two-limb split and
// E2M1 packing, for FP64 (or FP32, taken exactly as FP64) inputs. One wave per
// fragment (32 lines x 64 k); lane (line % 32, k half) converts its 32 values
// once, then for each modulus reduces them, looks the codes up in an LDS table
// and stores 16 bytes to each plane of that modulus: c0 (plane 2l), c1 (plane
// 2l + 1) and, in the Karatsuba mode (kKar) for a Karatsuba modulus, c0 + c1
// (plane 2L + ksum).
//   x = round_half_even(X * 2^s), |x| <= 2^53, is exact in FP64. For each m,
//   q = rint(x fl(1/m)) is within 0.7 of x / m, so r = x - q m lies in
//   (-m, m) and indexes a table over [-m, 2m) that maps every estimate to the
//   codes of its class (E bytes an entry: 2, or 4 in the Karatsuba mode).
//   Only the LDS byte address of the entry, E r + zero below 2^16, is formed,
//   and modulo 2^16: one FMA adds x fl(1/m) to 1.5 * 2^52 + q0, whose low
//   bits then hold q + q0, and one 16-bit multiply-add gives
//   E x - (q + q0) E m with E x modulo 2^16 kept from the conversion; q0 is
//   chosen so that -q0 E m is the address `zero` of remainder 0. (An even
//   m = odd 2^z needs zero / E divisible by 2^z: the tables' array is aligned
//   to 16 entries, tables start at multiples of 16 entries within it, and
//   m <= 169 has z <= 4.)
//   Two VALU operations a value and modulus before the lookup, in place of
//   four in FP64: both operands at 2048^3 67 -> 61 us (18 moduli), 1500 x 3001
//   44.6 -> 38.2 us, FP32 2048^3 48 -> 43 us. Large operands are bound by
//   their plane writes (26 B a value at 18 moduli, 4.2-4.9 TB/s).
//   kWide (capacity above 53 bits): x = A 2^s is an exact double below
//   2^63; a floor step first brings x down to an exact d with |d| < 2^15 (the
//   quotient is within 2^8 of floor(x / m), and the FMA's result is
//   representable, so exact), and the step above then runs on d.
//   Second term (the two-term split, blockIdx.z == 1): the value encoded is
//   x2 = round_half_even((A 2^s - x) 2^d2), |x2| <= 2^(d2 - 1); A 2^s - x
//   is exact (the fraction of A 2^s), and so is its product by 2^d2.
//
// One launch covers both operands (blocks below blocks_a encode a, the rest
// b), blockIdx.y the moduli per_group * y .. + per_group - 1.
template <typename T>
__device__ __forceinline__ uint32_t lut_lookup(uint32_t addr) {
  return *reinterpret_cast<__attribute__((address_space(3))) const T*>((size_t)addr);
}

// The integer x modulo 2^32, |x| <= 2^53.
__device__ __forceinline__ uint32_t low_word(double x) {
  const double lo = __builtin_fma(-0x1p32, __builtin_rint(x * 0x1p-32), x);   // |lo| <= 2^31
  return (uint32_t)__double_as_longlong(lo + 0x1.8p52);
}

template <bool kWide>
__device__ __forceinline__ uint32_t entry_address(double x, uint16_t xl, double inv, double md,
                                                  double magic, uint16_t step, uint32_t e) {
  if constexpr (kWide) {
    x = __builtin_fma(-__builtin_floor(x * inv), md, x);
    xl = (uint16_t)(e * (uint32_t)__double_as_longlong(x + 0x1.8p52));
  }
  const uint16_t q = (uint16_t)__double_as_longlong(__builtin_fma(x, inv, magic));
  return entry_sum(q, step, xl);
}

template <bool kKar, bool kWide, typename TIn, int kTerms>
__global__ __launch_bounds__(256) void k_encode_dgemm(
    ConvOperand a, ConvOperand b, uint32_t blocks_a, int L, int per_group,
    const ModConst* __restrict__ mc, const void* __restrict__ lut, int d2) {
  typedef typename std::conditional<kKar, uint32_t, uint16_t>::type Entry;
  constexpr uint32_t kE = (uint32_t)sizeof(Entry);
  extern __shared__ __attribute__((aligned(kLutAlign))) uint8_t s_raw[];
  const bool is_b = blockIdx.x >= blocks_a;
  const uint32_t block = is_b ? blockIdx.x - blocks_a : blockIdx.x;
  const uint32_t nblocks = is_b ? gridDim.x - blocks_a : blocks_a;
  const ConvOperand& op = is_b ? b : a;
  const int64_t rs = op.rs, ks = op.ks, lines = op.lines, k = op.k, kblocks = op.kblocks;
  const int64_t plane_bytes = op.plane_bytes;
  const TIn* X = reinterpret_cast<const TIn*>(op.X);
  const int l0 = (int)blockIdx.y * per_group, l1 = min(L, l0 + per_group);
  const bool second = kTerms == 2 && blockIdx.z != 0;
  uint8_t* planes = op.planes + (second ? op.term_bytes : 0);
  // this group's table, copied in 32-bit words from the word that holds its
  // first entry
  constexpr int kPerWord = 4 / (int)sizeof(Entry);
  const int word0 = mc->lut_off[l0] / kPerWord;
  const int words = (mc->lut_off[l1 - 1] + 3 * mc->m[l1 - 1] + kPerWord - 1) / kPerWord - word0;
  uint32_t* s_lut = reinterpret_cast<uint32_t*>(s_raw);
  const uint32_t* g_lut = reinterpret_cast<const uint32_t*>(lut) + word0;
  for (int i = threadIdx.x; i < words; i += 256) s_lut[i] = g_lut[i];
  __syncthreads();
  const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t*)s_raw;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const uint32_t kfrags = op.kfrags, nfrag = op.blocks * kfrags;
  for (uint32_t f = block * kEncWaves + wave; f < nfrag; f += nblocks * kEncWaves) {
    const uint32_t rb = f / kfrags, kb = f - rb * kfrags;
    const int64_t line = (int64_t)rb * kFragLines + (lane & 31);
    const int64_t kbase = (int64_t)kb * kFragK + (lane >> 5) * 32;
    const bool live = line < lines;
    int s = 0;
    if (live) {
      const uint64_t mx = partial_max(op.part, op.pstride, op.nchunk, line);
      s = line_shift(mx, op.cap);
      if (kb == 0 && lane < 32 && blockIdx.y == 0 && !second) op.amax[line] = mx;
    }
    double xe[32];
    const TIn* src = X + (live ? line : 0) * rs + kbase * ks;
    if (live && kbase + 32 <= k && ks == 1 && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
      // the lane's 32 values are contiguous (lines along k, as B's
      // columns): 16-byte loads
      constexpr int kPer = 16 / (int)sizeof(TIn);
      typedef TIn Vec __attribute__((ext_vector_type(kPer)));
      const Vec* v = reinterpret_cast<const Vec*>(src);
#pragma unroll
      for (int e = 0; e < 32 / kPer; ++e) {
        const Vec x = v[e];
#pragma unroll
        for (int q = 0; q < kPer; ++q) xe[e * kPer + q] = (double)x[q];
      }
    } else if (live && kbase + 32 <= k) {
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        xe[e] = (double)*src;
        src += ks;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        xe[e] = (live && kbase + e < k) ? (double)*src : 0.0;
        src += ks;
      }
    }
    uint16_t xl[32];   // E x modulo 2^16
#pragma unroll
    for (int e = 0; e < 32; ++e) {
      const double T = __builtin_ldexp(xe[e], s);
      double t = __builtin_rint(T);
      if constexpr (kTerms == 2) {
        if (second) t = __builtin_rint(__builtin_ldexp(T - t, d2));
      }
      // finite inputs give |t| <= 2^53 (2^63 when wide); NaN/Inf (reported
      // by the scale stage) must not drive the table address out of range
      t = (__builtin_fabs(t) <= (kWide ? 0x1p63 : 0x1p53)) ? t : 0.0;
      xe[e] = t;
      if constexpr (!kWide) xl[e] = (uint16_t)(kE * low_word(t));
    }
    uint8_t* out = planes + ((int64_t)rb * kblocks + kb) * kFragBytes + lane * 16;
    for (int l = l0; l < l1; ++l) {
      const int m = mc->m[l];
      const double inv = mc->inv[l], md = mc->md[l];
      // LDS address of the table entry of remainder 0, and the offset q0 of
      // the quotients with q0 E m = -address modulo 2^16
      const uint32_t zero = lds_base + kE * (uint32_t)(mc->lut_off[l] - word0 * kPerWord + m);
      const uint32_t q0 = entry_quotient_offset(zero, kE, mc->twos[l], mc->odd_inv[l]);
      const double magic = 0x1.8p52 + (double)q0;
      const uint16_t step = entry_step(kE, m);
      uint32_t w0[4], w1[4], w2[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint32_t p[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const int e = g * 8 + h * 2;
          const uint32_t E0 = lut_lookup<Entry>(
              entry_address<kWide>(xe[e], kWide ? 0 : xl[e], inv, md, magic, step, kE));
          const uint32_t E1 = lut_lookup<Entry>(
              entry_address<kWide>(xe[e + 1], kWide ? 0 : xl[e + 1], inv, md, magic, step, kE));
          // byte 0: plane-0 byte, byte 1: plane-1 byte (byte 2: sum plane)
          p[h] = E0 | (E1 << 4);
        }
        if constexpr (!kKar) {
          const uint32_t u = p[0] | (p[1] << 16), v = p[2] | (p[3] << 16);
          w0[g] = __builtin_amdgcn_perm(v, u, 0x06040200u);
          w1[g] = __builtin_amdgcn_perm(v, u, 0x07050301u);
        } else {
          const uint32_t t01 = __builtin_amdgcn_perm(p[1], p[0], 0x05010400u);
          const uint32_t t23 = __builtin_amdgcn_perm(p[3], p[2], 0x05010400u);
          w0[g] = __builtin_amdgcn_perm(t23, t01, 0x05040100u);
          w1[g] = __builtin_amdgcn_perm(t23, t01, 0x07060302u);
          const uint32_t s01 = __builtin_amdgcn_perm(p[1], p[0], 0x00000602u);
          const uint32_t s23 = __builtin_amdgcn_perm(p[3], p[2], 0x00000602u);
          w2[g] = __builtin_amdgcn_perm(s23, s01, 0x05040100u);
        }
      }
      const v4i p0 = {(int)w0[0], (int)w0[1], (int)w0[2], (int)w0[3]};
      const v4i p1 = {(int)w1[0], (int)w1[1], (int)w1[2], (int)w1[3]};
      *reinterpret_cast<v4i*>(out + (int64_t)(2 * l) * plane_bytes) = p0;
      *reinterpret_cast<v4i*>(out + (int64_t)(2 * l + 1) * plane_bytes) = p1;
      if constexpr (kKar) {
        const int ksum = mc->ksum[l];
        if (ksum >= 0) {
          const v4i p2 = {(int)w2[0], (int)w2[1], (int)w2[2], (int)w2[3]};
          *reinterpret_cast<v4i*>(out + (int64_t)(2 * L + ksum) * plane_bytes) = p2;
        }
      }
    }
  }
}

// Moduli that one wave encodes its fragment for. A wave takes about 0.5 us a
// modulus, so small operands give each fragment to several waves (which
// convert its values again, from L2) as long as that makes no more than 4096
// waves, four a SIMD: both operands 41 -> 9 us at 64^3, 53 -> 36 us at
// 1024^3 (18 moduli); with 8192 waves 42 us at 1024^3, with 2048 as with 4096.
constexpr int64_t kEncodeWaves = 4096;
inline int moduli_per_group(const ConvOperand& a, const ConvOperand& b, int L, int terms) {
  const int64_t frags = ((int64_t)a.blocks * a.kfrags + (int64_t)b.blocks * b.kfrags) * terms;
  const int64_t share = kEncodeWaves / std::max<int64_t>(1, frags);
  const int64_t groups = std::min<int64_t>(L, std::max<int64_t>(1, share));
  return (int)((L + groups - 1) / groups);
}

// Launches the encoder over both operands. `mod` is the host copy of mc;
// kTerms: 2 for the two-term split.
template <bool kKar, bool kWide, typename TIn, int kTerms = 1>
hipError_t launch_encode_kernel(hipStream_t stream, const ConvOperand& a, const ConvOperand& b,
                                int L, const ModConst& mod, const ModConst* mc, const void* lut,
                                int d2) {
  const uint32_t ba = encode_blocks(a), bb = encode_blocks(b);
  const int per_group = moduli_per_group(a, b, L, kTerms);
  const int groups = (L + per_group - 1) / per_group;
  const size_t entry = kKar ? sizeof(uint32_t) : sizeof(uint16_t);
  size_t lds = 0;
  for (int g = 0; g < groups; ++g) {
    const int l0 = g * per_group, l1 = std::min(L, l0 + per_group) - 1;
    lds = std::max(lds, entry * (size_t)(mod.lut_off[l1] + 3 * mod.m[l1] - mod.lut_off[l0]) + 8);
  }
  hipLaunchKernelGGL((k_encode_dgemm<kKar, kWide, TIn, kTerms>), dim3(ba + bb, groups, kTerms),
                     dim3(256), lds, stream, a, b, ba, L, per_group, mc, lut, d2);
  return hipGetLastError();
}

}  // namespace ozfp4
