// Small helpers of the adapter (LoRA) variant: packing the caller's rank-r adapter matrices into
// zero-padded bf16 operands the GEMM accepts (rank padded to 64; the three q/k/v adapters stacked
// into one [3*64, d] A matrix and one block-diagonal [(Hq+2Hkv)*hd, 3*64] B matrix), scaling the
// low-rank activations, and cutting the adapter gradients back out of the padded products.
#include "kernels.h"

#include <algorithm>

namespace {

// Grid (elements, destination).
struct PackDsts { PackDst d[4]; };
template <bool BF16>
__global__ __launch_bounds__(256) void lora_pack_kernel(const PackDsts all) {
  const PackDst &D = all.d[blockIdx.y];
  const size_t n = (size_t)D.rows * D.cols, stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    const int r = (int)(i / D.cols), c = (int)(i % D.cols);
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (k < D.n_src) {
        const int rr = r - D.src[k].r0, cc = c - D.src[k].c0;
        if (rr >= 0 && rr < D.src[k].rows && cc >= 0 && cc < D.src[k].cols) v = ld_io<BF16>(D.src[k].p, (size_t)rr * D.src[k].cols + cc);
      }
    bf16_t h, l;
    split_bf(v * D.scale, h, l);
    D.hi[i] = h;
    if (D.lo) D.lo[i] = l;
  }
}

__device__ __forceinline__ float ld_parts(const Parts &s, size_t i) {
  float v = s.p[i];
  for (int k = 1; k < s.n; ++k) v += s.p[(size_t)k * s.stride + i];
  return v;
}

__global__ __launch_bounds__(256) void scale_split_kernel(const Parts src, size_t n, float scale,
                                                          bf16_t *__restrict__ hi, bf16_t *__restrict__ lo) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    bf16_t h, l;
    split_bf(ld_parts(src, i) * scale, h, l);
    hi[i] = h;
    if (lo) lo[i] = l;
  }
}

// dst[rows, cols] (+)= src[(r0 + i) * src_ld + c0 + j]
__global__ __launch_bounds__(256) void extract_kernel(const Parts src, int src_ld, int r0, int c0, int rows, int cols,
                                                      float scale, float *__restrict__ dst, int accumulate) {
  const size_t n = (size_t)rows * cols, stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    const int r = (int)(i / cols), c = (int)(i % cols);
    const float v = scale * ld_parts(src, (size_t)(r0 + r) * src_ld + c0 + c);
    dst[i] = accumulate ? dst[i] + v : v;
  }
}

unsigned grid_for(size_t n) { return (unsigned)((n + 255) / 256 < 2048 ? (n + 255) / 256 : 2048); }

}  // namespace

hipError_t launch_lora_pack(const PackDst *dst, int n_dst, bool src_bf16, hipStream_t st) {
  if (n_dst < 1 || n_dst > 4) return hipErrorInvalidValue;
  PackDsts all = {};
  size_t most = 0;
  for (int i = 0; i < n_dst; ++i) {
    const PackDst &D = all.d[i] = dst[i];
    if (D.n_src < 1 || D.n_src > 3 || D.rows <= 0 || D.cols <= 0) return hipErrorInvalidValue;
    for (int k = 0; k < D.n_src; ++k) {
      const PackSrc &s = D.src[k];
      if (!s.p || s.rows <= 0 || s.cols <= 0 || s.r0 < 0 || s.c0 < 0 || s.r0 + s.rows > D.rows || s.c0 + s.cols > D.cols) return hipErrorInvalidValue;
    }
    most = std::max(most, (size_t)D.rows * D.cols);
  }
  const dim3 grid(grid_for(most), (unsigned)n_dst);
  if (src_bf16) hipLaunchKernelGGL(lora_pack_kernel<true>, grid, dim3(256), 0, st, all);
  else hipLaunchKernelGGL(lora_pack_kernel<false>, grid, dim3(256), 0, st, all);
  return hipGetLastError();
}

hipError_t launch_scale_split(const Parts &src, size_t n, float scale, bf16_t *hi, bf16_t *lo, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(scale_split_kernel, dim3(grid_for(n)), dim3(256), 0, st, src, n, scale, hi, lo);
  return hipGetLastError();
}

hipError_t launch_extract(const Parts &src, int src_ld, int r0, int c0, int rows, int cols, float scale, float *dst, int accumulate, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(extract_kernel, dim3(grid_for((size_t)rows * cols)), dim3(256), 0, st, src, src_ld, r0, c0, rows, cols, scale, dst, accumulate);
  return hipGetLastError();
}
