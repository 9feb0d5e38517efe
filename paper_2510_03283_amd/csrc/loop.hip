// The two small pieces that close the loop around an iteration: the greedy next token of
// inference rows from their logits (what the serving loop samples and checks for end of sequence)
// and the AdamW update that turns an iteration's gradients into the next iteration's weights.
#include "kernels.h"

namespace {

// One block per row: arg max over V fp32 logits, lowest index on ties.
__global__ __launch_bounds__(256) void argmax_rows_kernel(const float *__restrict__ logits, int V, int32_t *__restrict__ out) {
  const float *row = logits + (size_t)blockIdx.x * V;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int j = threadIdx.x; j < V; j += 256) {
    const float v = row[j];
    if (v > best || (v == best && j < bi)) { best = v; bi = j; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
  }
  __shared__ float sv[4];
  __shared__ int si[4];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sv[w] = best; si[w] = bi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; ++k)
      if (sv[k] > best || (sv[k] == best && si[k] < bi)) { best = sv[k]; bi = si[k]; }
    out[blockIdx.x] = bi == 0x7fffffff ? 0 : bi;       // a row of NaNs / -inf yields 0
  }
}

// AdamW, decoupled weight decay; c1 = 1/(1-b1^t), c2 = 1/(1-b2^t) come from the host in fp64 -> fp32.
struct AdamW {
  float lr, b1, b2, eps, wd, c1, c2;
  __device__ __forceinline__ float step(float g, float &m, float &v, float p) const {
    m = b1 * m + (1.f - b1) * g;
    v = b2 * v + (1.f - b2) * g * g;
    return p - lr * ((m * c1) / (sqrtf(v * c2) + eps) + wd * p);
  }
};

// HBM-bound: 26 - 30 bytes per element.  A block owns ADAM_U x 4 KB adjacent bytes of every fp32 stream and a thread asks for
// all its operands before the first is used; the last n % 4 elements are done one by one by the first threads.  (A loop over 8192
// blocks, one group of four per turn: 966 us for 131 M elements with an fp32 master copy, 263 us for 45 M; now 668 and 231 us,
// 5.9 TB/s.)
constexpr int ADAM_U = 2;
typedef float f32x4_s __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_s __attribute__((ext_vector_type(2)));

template <bool NT, typename T>
__device__ __forceinline__ T ld_stream(const T *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename T>
__device__ __forceinline__ void st_stream(T v, T *p) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

template <bool PBF16, bool NT>
__global__ __launch_bounds__(256) void adamw_kernel(void *__restrict__ param, float *__restrict__ master, const float *__restrict__ grad,
                                                    float *__restrict__ m, float *__restrict__ v, size_t n, const AdamW a) {
  const size_t n4 = n / 4, stride = (size_t)gridDim.x * 256 * ADAM_U;
  for (size_t base = (size_t)blockIdx.x * 256 * ADAM_U + threadIdx.x; base < n4; base += stride) {
    f32x4_s g[ADAM_U], mi[ADAM_U], vi[ADAM_U], p[ADAM_U];
#pragma unroll
    for (int u = 0; u < ADAM_U; ++u) {
      const size_t i = base + u * 256;
      if (i >= n4) continue;
      g[u] = ld_stream<NT>((const f32x4_s *)grad + i);
      mi[u] = ld_stream<NT>((const f32x4_s *)m + i);
      vi[u] = ld_stream<NT>((const f32x4_s *)v + i);
      if (master) p[u] = ld_stream<NT>((const f32x4_s *)master + i);
      else if constexpr (PBF16) {
        const u32x2_s r = ld_stream<NT>((const u32x2_s *)param + i);
        p[u] = f32x4_s{__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u), __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u)};
      } else p[u] = ld_stream<NT>((const f32x4_s *)param + i);
    }
#pragma unroll
    for (int u = 0; u < ADAM_U; ++u) {
      const size_t i = base + u * 256;
      if (i >= n4) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float mj = mi[u][j], vj = vi[u][j];
        p[u][j] = a.step(g[u][j], mj, vj, p[u][j]);
        mi[u][j] = mj;
        vi[u][j] = vj;
      }
      st_stream<NT>(mi[u], (f32x4_s *)m + i);
      st_stream<NT>(vi[u], (f32x4_s *)v + i);
      if (master) st_stream<NT>(p[u], (f32x4_s *)master + i);
      if constexpr (PBF16) st_stream<NT>(u32x2_s{pack2(f2bf(p[u].x), f2bf(p[u].y)), pack2(f2bf(p[u].z), f2bf(p[u].w))}, (u32x2_s *)param + i);
      else st_stream<NT>(p[u], (f32x4_s *)param + i);
    }
  }
  const size_t i = n4 * 4 + (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) {
    float mi = m[i], vi = v[i];
    const float p = a.step(grad[i], mi, vi, master ? master[i] : ld_io<PBF16>(param, i));
    m[i] = mi;
    v[i] = vi;
    if (master) master[i] = p;
    st_io<PBF16>(param, i, p);
  }
}

}  // namespace

hipError_t launch_argmax_rows(const float *logits, int rows, int V, int32_t *out, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(argmax_rows_kernel, dim3(rows), dim3(256), 0, st, logits, V, out);
  return hipGetLastError();
}

hipError_t launch_adamw(void *param, bool param_bf16, float *master, const float *grad, float *m, float *v, size_t n, float lr,
                        float b1, float b2, float eps, float wd, float c1, float c2, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const size_t want = (n / 4 + 256 * ADAM_U - 1) / (256 * ADAM_U) + 1;
  const unsigned blocks = (unsigned)(want < (1u << 20) ? want : (1u << 20));
  const AdamW a{lr, b1, b2, eps, wd, c1, c2};
  const uintptr_t al = (uintptr_t)param | (uintptr_t)master | (uintptr_t)grad | (uintptr_t)m | (uintptr_t)v;
  if (al & 15) return hipErrorInvalidValue;       // 16-byte accesses
  // Streams of more than four times the 256 MB last-level cache are read and written past it: 131 M elements 734 -> 668 us, 45 M
  // 247 -> 231; 17 M elements are better off cached where the step is repeated (67 against 85 us).
  const bool nt = n * 28 > ((size_t)1 << 30);
  auto *k = param_bf16 ? (nt ? adamw_kernel<true, true> : adamw_kernel<true, false>) : (nt ? adamw_kernel<false, true> : adamw_kernel<false, false>);
  hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, st, param, master, grad, m, v, n, a);
  return hipGetLastError();
}
