// Line maxima of both operands (Sec. IV-B) and the encoder instances of the
// FP64 and FP32 paths. A translation unit of its own,
// so nothing here can change how the compiler schedules the GEMMs.
#include "convert.hpp"
#include "device_common.hpp"
#include "encode.hpp"

#include <algorithm>

namespace ozfp4 {

namespace {

// |x| as an unsigned word whose order is the numeric one (NaN and infinity
// above every finite value), and that word's value as a double's bits.
__device__ __forceinline__ uint64_t abs_word(double x) {
  return (uint64_t)__double_as_longlong(x) & kAbsMask;
}
__device__ __forceinline__ uint32_t abs_word(float x) { return __float_as_uint(x) & 0x7fffffffu; }
__device__ __forceinline__ uint64_t double_bits(uint64_t w) { return w; }
__device__ __forceinline__ uint64_t double_bits(uint32_t w) {
  return (uint64_t)__double_as_longlong((double)__uint_as_float(w));
}

// Lines of a block where they are adjacent in memory: a power of two, so
// that a wave reads whole 128-byte segments of wide operands and a narrow
// one still keeps its lanes busy (the other lanes take other k).
__host__ __device__ inline int adjacent_lines(int64_t lines) {
  return lines > 16 ? 64 : (lines > 4 ? 16 : 4);
}

// Partial maxima of one (line group, chunk). Bound by HBM at large sizes;
// at small ones by the latency of a thread's serial loads, so chunks are cut
// to put up to 1024 blocks an operand on the chip and every thread keeps eight
// (four) loads in flight: 12.6 -> 3 us for 256 x 256 (the maxima of both
// operands), 26 -> 4 us for 1024 x 1024.
// Each (line, chunk) has one writer, so no zero fill and no atomics.
template <typename T>
__device__ __forceinline__ void line_max_block(const ConvOperand& op, uint32_t block, int* flag) {
  const T* X = reinterpret_cast<const T*>(op.X);
  typedef decltype(abs_word(T())) Word;
  __shared__ Word s_max[256];
  const int tid = threadIdx.x;
  const uint32_t nchunk = (uint32_t)op.nchunk;
  const uint32_t group = block / nchunk, c = block - group * nchunk;
  const int64_t k0 = (int64_t)c * op.chunk, k1 = min(op.k, k0 + op.chunk);
  Word mx = 0;
  if (op.ks == 1) {   // contiguous lines: one wave each, four a block
    const int64_t line = (int64_t)group * 4 + (tid >> 6);
    const int lane = tid & 63;
    if (line >= op.lines) return;
    const T* p = X + line * op.rs;
    int64_t kk = k0 + lane;
    for (; kk + 192 < k1; kk += 256) {
      const Word a = abs_word(p[kk]), b = abs_word(p[kk + 64]);
      const Word d = abs_word(p[kk + 128]), e = abs_word(p[kk + 192]);
      mx = max(mx, max(max(a, b), max(d, e)));
    }
    for (; kk < k1; kk += 64) mx = max(mx, abs_word(p[kk]));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = max(mx, (Word)__shfl_xor(mx, off, 64));
    if (lane == 0) {
      const uint64_t v = double_bits(mx);
      if (v >= kNonFinite) *flag = 1;
      op.part[c * op.pstride + line] = v;
    }
    return;
  }
  // adjacent lines: `span` lines a block, 256 / span k phases
  const int span = adjacent_lines(op.lines);
  const int lane_line = tid & (span - 1), phases = 256 / span;
  const int64_t line = (int64_t)group * span + lane_line;
  if (line < op.lines) {
    const T* p = X + line;
    const int64_t step = (int64_t)phases * op.ks;
    int64_t kk = k0 + tid / span;
    const T* q = p + kk * op.ks;
    for (; kk + 7 * phases < k1; kk += 8 * phases) {
      Word w[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = abs_word(q[e * step]);
      q += 8 * step;
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = max(mx, w[e]);
    }
    for (; kk < k1; kk += phases) {
      mx = max(mx, abs_word(*q));
      q += step;
    }
  }
  s_max[tid] = mx;
  __syncthreads();
  if (tid < span && line < op.lines) {
    for (int ph = 1; ph < phases; ++ph) mx = max(mx, s_max[ph * span + tid]);
    const uint64_t v = double_bits(mx);
    if (v >= kNonFinite) *flag = 1;
    op.part[c * op.pstride + line] = v;
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_line_max(ConvOperand a, ConvOperand b, uint32_t blocks_a,
                                                  uint32_t first, int* __restrict__ flag) {
  const uint32_t block = first + blockIdx.x;
  if (block < blocks_a)
    line_max_block<T>(a, block, flag);
  else
    line_max_block<T>(b, block - blocks_a, flag);
}

__global__ void k_shifts(const uint64_t* __restrict__ part, int64_t pstride, int nchunk,
                         int64_t lines, int cap, int32_t* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < lines) out[i] = line_shift(partial_max(part, pstride, nchunk, i), cap);
}

int64_t line_groups(const ConvOperand& op) {
  const int per = op.ks == 1 ? 4 : adjacent_lines(op.lines);
  return (op.lines + per - 1) / per;
}

}  // namespace

void plan_line_max(ConvOperand* op) {
  const int64_t groups = line_groups(*op);
  // at least 256 k a wave (contiguous) or eight k a thread (adjacent)
  const int64_t unit = op->ks == 1 ? 256 : 8 * (256 / adjacent_lines(op->lines));
  const int64_t most = std::max<int64_t>(1, std::min<int64_t>(kMaxChunks, 1024 / groups));
  const int64_t want = (op->k + most - 1) / most;
  op->chunk = (want + unit - 1) / unit * unit;
  op->nchunk = (int)((op->k + op->chunk - 1) / op->chunk);
}

hipError_t launch_line_max(hipStream_t stream, bool f32, const ConvOperand& a,
                           const ConvOperand& b, int* flag) {
  const int64_t blocks_a = line_groups(a) * a.nchunk, total = blocks_a + line_groups(b) * b.nchunk;
  constexpr int64_t kBlocks = kLaunchThreads / 256;
  for (int64_t first = 0; first < total; first += kBlocks) {
    const unsigned grid = (unsigned)std::min(total - first, kBlocks);
    if (f32)
      hipLaunchKernelGGL(k_line_max<float>, dim3(grid), dim3(256), 0, stream, a, b,
                         (uint32_t)blocks_a, (uint32_t)first, flag);
    else
      hipLaunchKernelGGL(k_line_max<double>, dim3(grid), dim3(256), 0, stream, a, b,
                         (uint32_t)blocks_a, (uint32_t)first, flag);
  }
  return hipGetLastError();
}

hipError_t launch_encode(hipStream_t stream, bool f32, const ConvOperand& a, const ConvOperand& b,
                         int L, const ModConst& mod, const ModConst* mc, const uint16_t* lut,
                         int terms, int d2) {
  if (f32) return launch_encode_kernel<false, false, float>(stream, a, b, L, mod, mc, lut, 0);
  // the two-term split keeps to 53 bits
  if (terms == 2)
    return launch_encode_kernel<false, false, double, 2>(stream, a, b, L, mod, mc, lut, d2);
  // c_A >= c_B, so the wide encoder is exact for both where A needs it
  if (a.cap > 53) return launch_encode_kernel<false, true, double>(stream, a, b, L, mod, mc, lut, 0);
  return launch_encode_kernel<false, false, double>(stream, a, b, L, mod, mc, lut, 0);
}

hipError_t launch_shifts(hipStream_t stream, const ConvOperand& op, int32_t* out) {
  hipLaunchKernelGGL(k_shifts, dim3((unsigned)((op.lines + 255) / 256)), dim3(256), 0, stream,
                     op.part, op.pstride, op.nchunk, op.lines, op.cap, out);
  return hipGetLastError();
}

}  // namespace ozfp4
