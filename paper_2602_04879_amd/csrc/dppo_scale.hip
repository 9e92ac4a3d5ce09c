// The gradient times the incoming gradient of the scalar loss, which an autograd engine hands over as
// a device scalar: the factor is read by the kernel, so nothing waits for it on the host, and a
// factor of one (loss.backward()) ends every workgroup at once.
//
// Bound by HBM: one read and one write of the bf16 gradient, in place (V = 50257, 6000 tokens: 1.2 GB).
// As tensor operations (widen, multiply, narrow) the same was 20 bytes per entry and two fp32 copies
// of the gradient, behind a synchronisation that looked at the factor.
#include "dppo_common.hpp"
#include "dppo_launch.hpp"

namespace dppo {
namespace {

constexpr int kThreads = 256;
constexpr int kUnroll = 4;                            // 16-byte blocks in flight per thread
constexpr int kPiece = kThreads * kUnroll;            // blocks of one workgroup's piece of a row

__device__ __forceinline__ uint32_t scale2(uint32_t w, float f) {
  return pack_bf16x2(__uint_as_float(w << 16) * f, __uint_as_float(w & 0xffff0000u) * f);
}

// x[r, 0..cols) *= *factor, rounded to bf16 once.  Rows of any pitch and 2-byte alignment: a row is
// handled in the aligned 16-byte blocks that hold it, an incomplete first or last block entry by entry.
__global__ __launch_bounds__(kThreads) void dppo_scale_rows_kernel(uint16_t* x, int64_t rows, int64_t cols, int64_t ld, const float* factor) {
  const float f = *factor;
  if (f == 1.f) return;
  const int64_t pieces = (cols / 8 + 2 + kPiece - 1) / kPiece;        // of one row, whatever its alignment
  for (int64_t item = blockIdx.x; item < rows * pieces; item += gridDim.x) {
    const int64_t r = item / pieces;
    uint16_t* row = x + r * ld;
    const int h = static_cast<int>((reinterpret_cast<uintptr_t>(row) & 15u) >> 1);    // entries of the first block in front of the row
    const int64_t b0 = (item - r * pieces) * kPiece + threadIdx.x;
    const int64_t whole = (h + cols) >> 3;                                            // blocks that end inside the row
    u32x4 v[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t b = b0 + u * kThreads;
      if (b < whole && (b > 0 || h == 0)) v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row - h) + b);
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t b = b0 + u * kThreads;
      if (b < whole && (b > 0 || h == 0)) {
        const u32x4 o = {scale2(v[u].x, f), scale2(v[u].y, f), scale2(v[u].z, f), scale2(v[u].w, f)};
        __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(row - h) + b);
      } else {
        for (int64_t e = max(8 * b - h, int64_t(0)); e < min(8 * b - h + 8, cols); ++e)
          row[e] = float_to_bf16_bits(bf16_bits_to_float(row[e]) * f);
      }
    }
  }
}

// dst[i] = bf16(src[i] * *factor) for an fp32 source (the weight gradient): the conversion autograd
// needs anyway, with the factor in it.  src and dst 16-byte aligned; eight 16-byte loads in flight per
// thread, neighbouring lanes at neighbouring addresses.
constexpr int kQuads = 8;
__global__ __launch_bounds__(kThreads) void dppo_scale_to_bf16_kernel(uint16_t* __restrict__ dst, const float* __restrict__ src, int64_t n,
                                                                      const float* factor) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const float f = *factor;
  const int64_t quads = n >> 2, i = static_cast<int64_t>(blockIdx.x) * (kQuads * kThreads) + threadIdx.x;
  const f32x4* s = reinterpret_cast<const f32x4*>(src);
  u32x2* d = reinterpret_cast<u32x2*>(dst);
  f32x4 a[kQuads];
#pragma unroll
  for (int u = 0; u < kQuads; ++u)
    if (i + u * kThreads < quads) a[u] = __builtin_nontemporal_load(s + i + u * kThreads);
#pragma unroll
  for (int u = 0; u < kQuads; ++u)
    if (i + u * kThreads < quads)
      __builtin_nontemporal_store(u32x2{pack_bf16x2(a[u][0] * f, a[u][1] * f), pack_bf16x2(a[u][2] * f, a[u][3] * f)}, d + i + u * kThreads);
  if (blockIdx.x == 0 && 4 * quads + threadIdx.x < n) dst[4 * quads + threadIdx.x] = float_to_bf16_bits(src[4 * quads + threadIdx.x] * f);
}

}  // namespace

hipError_t launch_scale_rows(uint16_t* x, int64_t rows, int64_t cols, int64_t ld, const float* factor, int cus, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (ld == cols) { cols *= rows; rows = 1; ld = cols; }              // packed rows: one long one
  const int64_t items = rows * ((cols / 8 + 2 + kPiece - 1) / kPiece);
  const int64_t grid = items < 8 * static_cast<int64_t>(cus) ? items : 8 * static_cast<int64_t>(cus);
  hipLaunchKernelGGL(dppo_scale_rows_kernel, dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, s, x, rows, cols, ld, factor);
  return hipGetLastError();
}

hipError_t launch_scale_to_bf16(uint16_t* dst, const float* src, int64_t n, const float* factor, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t grid = (n / 4 + kQuads * kThreads - 1) / (kQuads * kThreads) + (n < 4 ? 1 : 0);
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(dppo_scale_to_bf16_kernel, dim3(static_cast<unsigned>(grid)), dim3(kThreads), 0, s, dst, src, n, factor);
  return hipGetLastError();
}

}  // namespace dppo
