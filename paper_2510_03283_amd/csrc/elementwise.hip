// HBM-bound row kernels: RMSNorm, rotary embedding, SwiGLU, operand splitting (fwd and bwd).
#include "kernels.h"

#include <type_traits>

namespace {

template <bool BF16>
__device__ __forceinline__ void ld4(const void *p, size_t i, float v[4]) {
  if constexpr (BF16) {
    const uint2 u = *(const uint2 *)((const bf16_t *)p + i);
    v[0] = __uint_as_float(u.x << 16); v[1] = __uint_as_float(u.x & 0xffff0000u);
    v[2] = __uint_as_float(u.y << 16); v[3] = __uint_as_float(u.y & 0xffff0000u);
  } else {
    const float4 f = *(const float4 *)((const float *)p + i);
    v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
  }
}

__device__ __forceinline__ void st4_split(bf16_t *hi, bf16_t *lo, size_t i, const float v[4]) {
  bf16_t h[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) split_bf(v[j], h[j], l[j]);
  *(uint2 *)(hi + i) = make_uint2(pack2(h[0], h[1]), pack2(h[2], h[3]));
  if (lo) *(uint2 *)(lo + i) = make_uint2(pack2(l[0], l[1]), pack2(l[2], l[3]));
}

__device__ __forceinline__ float4 ld4_parts(const Parts &s, size_t i) {
  float4 v = *(const float4 *)(s.p + i);
  for (int k = 1; k < s.n; ++k) {
    const float4 w = *(const float4 *)(s.p + (size_t)k * s.stride + i);
    v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
  }
  return v;
}

// ------------------------------------------------------------------ RMSNorm forward
// NV float4 chunks of a row per thread (d <= 1024 NV), zeros past its end.  No branch around a load: a thread past the end reads
// the last chunk again, and the loads go out one behind the other.
template <bool BF, int NV>
__device__ __forceinline__ void row_ld_as(const void *p, size_t at, int d, float (&v)[NV][4]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) ld4<BF>(p, at + min(4 * (int)threadIdx.x + 1024 * i, d - 4), v[i]);
#pragma unroll
  for (int i = 0; i < NV; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) v[i][j] = 4 * (int)threadIdx.x + 1024 * i < d ? v[i][j] : 0.f;
}
template <int NV>
__device__ __forceinline__ void row_ld(const void *p, int bf16, size_t at, int d, float (&v)[NV][4]) {
  if (bf16) row_ld_as<true, NV>(p, at, d, v);
  else row_ld_as<false, NV>(p, at, d, v);
}

// One block per row; NV float4 chunks per thread stay in registers between the reduction and the output.  With few rows
// the time is the chain of load latencies, so all chunks of an operand are asked for together, and the gain before the row.
// (Chunk by chunk, each asked for when the one before it had arrived, and the gain behind the reduction: a decode pass of the
// edge layer, 32 rows of 2048, 113.0 us, now 111.3; its prefill of 2329 rows 364 and 358.)
template <int NV, bool GBF>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(const NormRows g0, const NormRows g1, const void *gain, int d, float eps) {
  __shared__ float red[4];
  const bool second = (int)blockIdx.x >= g0.rows;
  const NormRows &G = second ? g1 : g0;
  const int r = second ? (int)blockIdx.x - g0.rows : (int)blockIdx.x;
  const size_t xin = (size_t)(G.row_idx ? G.row_idx[r] : r) * d, xo = (size_t)r * d;
  std::conditional_t<GBF, uint2, float4> graw[NV];      // unpacked where it is used: nothing waits for it before
#pragma unroll
  for (int i = 0; i < NV; ++i) graw[i] = *(const decltype(&graw[0]))((const char *)gain + min(4 * (int)threadIdx.x + 1024 * i, d - 4) * (GBF ? 2 : 4));
  float v[NV][4];
  float ss = 0.f;
  row_ld<NV>(G.x, G.x_bf16, xin, d, v);
  if (G.parts.p) {
    float s[NV][4], t[NV][4];
    row_ld<NV>(G.parts.p, 0, xo, d, s);
    for (int p = 1; p < G.parts.n; ++p) {
      row_ld<NV>(G.parts.p + (size_t)p * G.parts.stride, 0, xo, d, t);
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) s[i][j] += t[i][j];
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = 4 * threadIdx.x + 1024 * i;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[i][j] = s[i][j] + v[i][j];
      if (k < d) *(float4 *)(G.v_out + xo + k) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
    }
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) ss += v[i][0] * v[i][0] + v[i][1] * v[i][1] + v[i][2] * v[i][2] + v[i][3] * v[i][3];
  ss = block_sum<256>(ss, red);
  const float rs = 1.0f / sqrtf(ss / (float)d + eps);
  if (G.rstd && threadIdx.x == 0) G.rstd[r] = rs;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int k = 4 * threadIdx.x + 1024 * i;
    if (k < d) {
      float gg[4];
      ld4<GBF>(&graw[i], 0, gg);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[i][j] = v[i][j] * rs * gg[j];
      st4_split(G.hi, G.lo, G.frag ? frag_index(r, k, d) : xo + k, v[i]);
    }
  }
}

// ------------------------------------------------------------------ RMSNorm backward
constexpr int RB_MAXV = 8;   // d <= 8192
// One block per partial row of dg; a block walks rows r = blockIdx.x, + gridDim.x, ...  NV = float4
// chunks per thread (d <= 1024 NV): the row of dy and of x stays in registers between the reduction
// and the output pass, and g is read once per block.
template <bool XBF, bool GBF, int NV>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(const Parts dy, const void *x, const int32_t *row_idx,
                                                          const void *g, const float *rstd, const float *resid,
                                                          int rows, int d, float *dx_out, bf16_t *dx_bf,
                                                          float *dg_partial, int dense_out) {
  __shared__ float red[4];
  float dgacc[NV][4], gg[NV][4];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int k = 4 * threadIdx.x + 1024 * i;
#pragma unroll
    for (int j = 0; j < 4; ++j) dgacc[i][j] = gg[i][j] = 0.f;
    if (k < d) ld4<GBF>(g, k, gg[i]);
  }
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    const size_t xr = (size_t)(row_idx ? row_idx[r] : r) * d, yr = (size_t)r * d;
    float dv[NV][4], xv[NV][4], rr[NV][4];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = 4 * threadIdx.x + 1024 * i;
#pragma unroll
      for (int j = 0; j < 4; ++j) dv[i][j] = xv[i][j] = rr[i][j] = 0.f;
      if (k < d) {
        const float4 t = ld4_parts(dy, yr + k);
        dv[i][0] = t.x; dv[i][1] = t.y; dv[i][2] = t.z; dv[i][3] = t.w;
        ld4<XBF>(x, xr + k, xv[i]);
        if (resid) ld4<false>(resid, yr + k, rr[i]);
      }
    }
    const float rs = rstd[r];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s += dv[i][j] * gg[i][j] * xv[i][j];
        dgacc[i][j] += dv[i][j] * xv[i][j] * rs;
      }
    s = block_sum<256>(s, red);
    const float c = rs * rs * rs * s / (float)d;
    const size_t orow = dense_out ? yr : xr;      // dense: output row r (may be dy itself), else the gathered row
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = 4 * threadIdx.x + 1024 * i;
      if (k < d) {
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = rr[i][j] + rs * dv[i][j] * gg[i][j] - xv[i][j] * c;
        *(float4 *)(dx_out + orow + k) = make_float4(o[0], o[1], o[2], o[3]);
        if (dx_bf) *(uint2 *)(dx_bf + orow + k) = make_uint2(pack2(f2bf(o[0]), f2bf(o[1])), pack2(f2bf(o[2]), f2bf(o[3])));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int k = 4 * threadIdx.x + 1024 * i;
    if (k < d) *(float4 *)(dg_partial + (size_t)blockIdx.x * d + k) = make_float4(dgacc[i][0], dgacc[i][1], dgacc[i][2], dgacc[i][3]);
  }
}

// Column sums of the partial rows in two launches: slice y of COLSUM_SLICES sums the rows y, y + S,
// y + 2S, ... of 256 adjacent columns (1 KB contiguous per row, eight loads in flight per thread) into
// row y of a scratch buffer; the second launch (n_slices rows, slices == 1) adds those rows in a fixed
// order: deterministic.  (A block that walks many rows of a narrow column strip puts all its loads, a
// power-of-two stride apart, on the same memory channel.)
__global__ __launch_bounds__(256) void colsum_kernel(const float *part, int n_part, int d, int slices, float *out, int accumulate) {
  const int j = blockIdx.x * 256 + threadIdx.x, y = blockIdx.y;
  if (j >= d) return;
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int i = y;
  for (; i + 7 * slices < n_part; i += 8 * slices) {
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] += part[(size_t)(i + slices * u) * d + j];
  }
  for (; i < n_part; i += slices) a[0] += part[(size_t)i * d + j];
  const float t = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  float *o = out + (size_t)y * d + j;
  *o = accumulate ? *o + t : t;
}

// ------------------------------------------------------------------ rotary embedding
// One block per row.  A thread takes four neighbouring elements i .. i + 3 of a head and their partners i + hd/2 ..;
// the row's (cos, sin) table is formed once in LDS.
template <bool CBF>
__global__ __launch_bounds__(256) void rope_split_kernel(const RopeRows g0, const RopeRows g1, const double *inv_freq, int Hq, int Hkv, int hd,
                                                         void *cache_k, void *cache_v, long long num_slots, int block_size) {
  __shared__ float2 cs[64];
  const bool second = (int)blockIdx.x >= g0.rows;
  const RopeRows &G = second ? g1 : g0;
  const int r = second ? (int)blockIdx.x - g0.rows : (int)blockIdx.x, half = hd >> 1;
  if ((int)threadIdx.x < half) cs[threadIdx.x] = rope_angle((double)G.positions[r] * inv_freq[threadIdx.x]);
  __syncthreads();
  const int qd = Hq * hd, kd = Hkv * hd, nq = qd + 2 * kd;
  const size_t in = (size_t)r * nq;
  long long slot = -1;
  if (G.slot_mapping) {
    slot = G.slot_mapping[r];
    if (slot >= num_slots) slot = -1;
  }
  const long long cbase = slot >= 0 ? (slot / block_size) * (long long)Hkv * block_size * hd + (slot % block_size) * (long long)hd : 0;
  // four elements e .. e + 3 of kv head kh to the cache
  auto to_cache = [&](void *cache, int kh, int e, const float *v, uint2 w) {
    const long long c = cbase + (long long)kh * block_size * hd + e;
    if constexpr (CBF) *(uint2 *)((bf16_t *)cache + c) = w;
    else *(float4 *)((float *)cache + c) = make_float4(v[0], v[1], v[2], v[3]);
  };
  auto put = [&](bf16_t *hi, bf16_t *lo, size_t o, const float *v) -> uint2 {
    uint32_t h0, l0, h1, l1;
    split_pk_bf16(v[0], v[1], h0, l0);
    split_pk_bf16(v[2], v[3], h1, l1);
    *(uint2 *)(hi + o) = make_uint2(h0, h1);
    if (lo) *(uint2 *)(lo + o) = make_uint2(l0, l1);
    return make_uint2(h0, h1);
  };
  const int qpr = half >> 2;                             // quads of pairs per head
  for (int idx = threadIdx.x; idx < (Hq + Hkv) * qpr; idx += 256) {
    const int head = idx / qpr, i = (idx - head * qpr) * 4;
    const float4 a = ld4_parts(G.qkv, in + head * hd + i), b = ld4_parts(G.qkv, in + head * hd + i + half);
    const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
    float ra[4], rb[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float2 t = cs[i + e];
      ra[e] = av[e] * t.x - bv[e] * t.y;
      rb[e] = bv[e] * t.x + av[e] * t.y;
    }
    if (head < Hq) {
      const size_t o = (size_t)r * qd + head * hd + i;
      put(G.q_hi, G.q_lo, o, ra);
      put(G.q_hi, G.q_lo, o + half, rb);
    } else {
      const int kh = head - Hq;
      const size_t o = (size_t)r * kd + kh * hd + i;
      const uint2 wa = put(G.k_hi, G.k_lo, o, ra), wb = put(G.k_hi, G.k_lo, o + half, rb);
      if (slot >= 0) {
        to_cache(cache_k, kh, i, ra, wa);
        to_cache(cache_k, kh, i + half, rb, wb);
      }
    }
  }
  for (int idx = 4 * threadIdx.x; idx < kd; idx += 1024) {
    const float4 v4 = ld4_parts(G.qkv, in + qd + kd + idx);
    const float v[4] = {v4.x, v4.y, v4.z, v4.w};
    const uint2 w = put(G.v_hi, G.v_lo, (size_t)r * kd + idx, v);
    if (slot >= 0) to_cache(cache_v, idx / hd, idx % hd, v, w);
  }
}

__global__ __launch_bounds__(64) void rope_table_kernel(const int32_t *__restrict__ positions, const double *__restrict__ inv_freq,
                                                        int half, float2 *__restrict__ cs) {
  const int r = blockIdx.x, i = threadIdx.x;
  if (i >= half) return;
  cs[(size_t)r * half + i] = rope_angle((double)positions[r] * inv_freq[i]);
}

// ------------------------------------------------------------------ SwiGLU
// 8 hidden units per thread (16-byte accesses); F % 8 == 0.
__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const bf16_t *__restrict__ dhm, const Parts parts, const bf16_t *__restrict__ gu, int F,
                                                         bf16_t *__restrict__ dgu) {
  const int r = blockIdx.x;
  const int k = 8 * (blockIdx.y * 256 + threadIdx.x);
  if (k >= F) return;
  const uint4 gq = *(const uint4 *)(gu + (size_t)r * 2 * F + k), uq = *(const uint4 *)(gu + (size_t)r * 2 * F + F + k);
  float dv[8];
  if (dhm) {
    const uint4 dq = *(const uint4 *)(dhm + (size_t)r * F + k);
    const uint32_t dw[4] = {dq.x, dq.y, dq.z, dq.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) { dv[2 * j] = __uint_as_float(dw[j] << 16); dv[2 * j + 1] = __uint_as_float(dw[j] & 0xffff0000u); }
  } else {
    const float4 a = ld4_parts(parts, (size_t)r * F + k), b = ld4_parts(parts, (size_t)r * F + k + 4);
    dv[0] = a.x; dv[1] = a.y; dv[2] = a.z; dv[3] = a.w; dv[4] = b.x; dv[5] = b.y; dv[6] = b.z; dv[7] = b.w;
  }
  const uint32_t gw[4] = {gq.x, gq.y, gq.z, gq.w}, uw[4] = {uq.x, uq.y, uq.z, uq.w};
  uint32_t og[4], ou[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float dg[2], du[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float g = e ? __uint_as_float(gw[j] & 0xffff0000u) : __uint_as_float(gw[j] << 16);
      const float u = e ? __uint_as_float(uw[j] & 0xffff0000u) : __uint_as_float(uw[j] << 16);
      const float dh = dv[2 * j + e];
      const float sg = 1.0f / (1.0f + expf(-g));
      du[e] = dh * g * sg;
      dg[e] = dh * u * sg * (1.0f + g * (1.0f - sg));
    }
    og[j] = cvt_pk_bf16(dg[0], dg[1]);
    ou[j] = cvt_pk_bf16(du[0], du[1]);
  }
  *(uint4 *)(dgu + (size_t)r * 2 * F + k) = make_uint4(og[0], og[1], og[2], og[3]);
  *(uint4 *)(dgu + (size_t)r * 2 * F + F + k) = make_uint4(ou[0], ou[1], ou[2], ou[3]);
}

// HBM-bound: four elements per thread (16-byte loads, 8-byte stores) where the pointers allow it (n4 = n / 4, else 0), the
// rest one by one.  65536 x 4096 to one bf16 term: 412 us with one element per turn (3.9 TB/s), 330 us now (4.9 TB/s).
// One launch for all ranges of a call (a model in fp32 has seven weight matrices to split in front of every forward and
// backward: 2.3 us each, and as much again between two launches).  A range takes the blocks first .. first + count - 1 of the grid.
struct SplitJob { SplitRange r; size_t n4; unsigned first, count; };
struct SplitJobs { SplitJob j[MAX_SPLIT_RANGES]; };
__global__ __launch_bounds__(256) void split_f32_kernel(const SplitJobs jobs, int n_jobs) {
  int k = 0;
  while (k + 1 < n_jobs && blockIdx.x >= jobs.j[k + 1].first) ++k;
  const float *__restrict__ src = jobs.j[k].r.src;
  bf16_t *__restrict__ hi = jobs.j[k].r.hi, *__restrict__ lo = jobs.j[k].r.lo;
  const size_t n = jobs.j[k].r.n, n4 = jobs.j[k].n4, stride = (size_t)jobs.j[k].count * 256, t = (size_t)(blockIdx.x - jobs.j[k].first) * 256 + threadIdx.x;
  for (size_t i = t; i < n4; i += stride) {
    float v[4];
    ld4<false>(src, 4 * i, v);
    st4_split(hi, lo, 4 * i, v);
  }
  for (size_t i = 4 * n4 + t; i < n; i += stride) {
    bf16_t h, l;
    split_bf(src[i], h, l);
    hi[i] = h;
    if (lo) lo[i] = l;
  }
}

// G and U of four hidden units per thread.
__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const SwigluRows g0, const SwigluRows g1, int F) {
  const bool second = (int)blockIdx.x >= g0.rows;
  const SwigluRows &G = second ? g1 : g0;
  const size_t r = second ? blockIdx.x - g0.rows : blockIdx.x;
  const int k = 4 * (blockIdx.y * 256 + threadIdx.x);
  if (k >= F) return;
  const float4 g4 = ld4_parts(G.gu_in, r * 2 * F + k), u4 = ld4_parts(G.gu_in, r * 2 * F + F + k);
  const float g[4] = {g4.x, g4.y, g4.z, g4.w}, u[4] = {u4.x, u4.y, u4.z, u4.w};
  float h[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) h[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
  st4_split(G.hi, G.lo, r * F + k, h);
  if (G.gu) {
    *(uint2 *)(G.gu + r * 2 * F + k) = make_uint2(cvt_pk_bf16(g[0], g[1]), cvt_pk_bf16(g[2], g[3]));
    *(uint2 *)(G.gu + r * 2 * F + F + k) = make_uint2(cvt_pk_bf16(u[0], u[1]), cvt_pk_bf16(u[2], u[3]));
  }
}

template <bool OBF>
__global__ __launch_bounds__(256) void sum_parts_kernel(const SumRange s0, const SumRange s1, const SumRange s2) {
  const size_t n = s0.n + s1.n + s2.n, stride = (size_t)gridDim.x * 1024;
  for (size_t t = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4; t < n; t += stride) {      // all lengths multiples of 4
    const int w = t < s0.n ? 0 : (t < s0.n + s1.n ? 1 : 2);
    const SumRange &S = w == 0 ? s0 : (w == 1 ? s1 : s2);
    const size_t i = t - (w == 0 ? 0 : (w == 1 ? s0.n : s0.n + s1.n));
    float4 a = ld4_parts(S.parts, i);
    if (S.resid) {
      const float4 b = *(const float4 *)(S.resid + i);
      a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
    }
    if constexpr (OBF) *(uint2 *)((bf16_t *)S.out + i) = make_uint2(cvt_pk_bf16(a.x, a.y), cvt_pk_bf16(a.z, a.w));
    else *(float4 *)((float *)S.out + i) = a;
  }
}

__global__ __launch_bounds__(256) void fill_f32_kernel(float *dst, size_t n, float v) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) dst[i] = v;
}

}  // namespace

hipError_t launch_rmsnorm_fwd(const NormRows *groups, int n_groups, const void *g, bool g_bf16, int d, float eps, hipStream_t st) {
  if (n_groups < 1 || n_groups > 2 || d > 8192) return hipErrorInvalidValue;
  NormRows g0 = groups[0], g1 = {};
  if (n_groups > 1) g1 = groups[1];
  if (g0.rows < 0 || g1.rows < 0) return hipErrorInvalidValue;
  if (g0.rows + g1.rows == 0) return hipSuccess;
  const dim3 grid(g0.rows + g1.rows), blk(256);
  auto go = [&](auto nv) {
    if (g_bf16) hipLaunchKernelGGL((rmsnorm_fwd_kernel<decltype(nv)::value, true>), grid, blk, 0, st, g0, g1, g, d, eps);
    else hipLaunchKernelGGL((rmsnorm_fwd_kernel<decltype(nv)::value, false>), grid, blk, 0, st, g0, g1, g, d, eps);
  };
  if (d <= 1024) go(std::integral_constant<int, 1>{});
  else if (d <= 2048) go(std::integral_constant<int, 2>{});
  else if (d <= 4096) go(std::integral_constant<int, 4>{});
  else go(std::integral_constant<int, 8>{});
  return hipGetLastError();
}

template <bool XBF, bool GBF>
static void rmsnorm_bwd_nv(int nv, dim3 grid, hipStream_t st, const Parts &dy, const void *x, const int32_t *row_idx, const void *g,
                           const float *rstd, const float *resid, int rows, int d, float *dx_out, bf16_t *dx_bf,
                           float *dg_partial, int dense_out) {
  const dim3 blk(256);
  if (nv <= 1) hipLaunchKernelGGL((rmsnorm_bwd_kernel<XBF, GBF, 1>), grid, blk, 0, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
  else if (nv <= 2) hipLaunchKernelGGL((rmsnorm_bwd_kernel<XBF, GBF, 2>), grid, blk, 0, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
  else if (nv <= 4) hipLaunchKernelGGL((rmsnorm_bwd_kernel<XBF, GBF, 4>), grid, blk, 0, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
  else hipLaunchKernelGGL((rmsnorm_bwd_kernel<XBF, GBF, RB_MAXV>), grid, blk, 0, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
}

hipError_t launch_rmsnorm_bwd(const Parts &dy, const void *x, bool x_bf16, const int32_t *row_idx, const void *g,
                              bool g_bf16, const float *rstd, const float *resid, int rows, int d, float *dx_out,
                              bf16_t *dx_bf, float *dg_partial, int n_part, hipStream_t st, int dense_out) {
  if (rows <= 0 || n_part <= 0) return hipSuccess;
  if (d > 1024 * RB_MAXV) return hipErrorInvalidValue;
  const dim3 grid(n_part);
  const int nv = (d + 1023) / 1024;
  if (x_bf16 && g_bf16) rmsnorm_bwd_nv<true, true>(nv, grid, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
  else if (!x_bf16 && g_bf16) rmsnorm_bwd_nv<false, true>(nv, grid, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
  else if (!x_bf16 && !g_bf16) rmsnorm_bwd_nv<false, false>(nv, grid, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
  else rmsnorm_bwd_nv<true, false>(nv, grid, st, dy, x, row_idx, g, rstd, resid, rows, d, dx_out, dx_bf, dg_partial, dense_out);
  return hipGetLastError();
}

hipError_t launch_colsum(const float *part, int n_part, int d, float *scratch, float *out, int accumulate, hipStream_t st) {
  const int slices = n_part >= 4 * COLSUM_SLICES ? COLSUM_SLICES : 1;
  const dim3 blk(256);
  if (slices > 1) {
    hipLaunchKernelGGL(colsum_kernel, dim3(cdiv(d, 256), slices), blk, 0, st, part, n_part, d, slices, scratch, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    part = scratch;
    n_part = slices;
  }
  hipLaunchKernelGGL(colsum_kernel, dim3(cdiv(d, 256), 1), blk, 0, st, part, n_part, d, 1, out, accumulate);
  return hipGetLastError();
}

hipError_t launch_rope_split(const RopeRows *groups, int n_groups, const double *inv_freq, int Hq, int Hkv, int hd, void *cache_k,
                             void *cache_v, bool cache_bf16, long long num_slots, int block_size, hipStream_t st) {
  if (n_groups < 1 || n_groups > 2 || hd > 128 || hd % 8) return hipErrorInvalidValue;
  RopeRows g0 = groups[0], g1 = {};
  if (n_groups > 1) g1 = groups[1];
  if (g0.rows < 0 || g1.rows < 0) return hipErrorInvalidValue;
  const unsigned rows = (unsigned)(g0.rows + g1.rows);
  if (rows == 0) return hipSuccess;
  if (cache_bf16) hipLaunchKernelGGL((rope_split_kernel<true>), dim3(rows), dim3(256), 0, st, g0, g1, inv_freq, Hq, Hkv, hd, cache_k, cache_v, num_slots, block_size);
  else hipLaunchKernelGGL((rope_split_kernel<false>), dim3(rows), dim3(256), 0, st, g0, g1, inv_freq, Hq, Hkv, hd, cache_k, cache_v, num_slots, block_size);
  return hipGetLastError();
}

hipError_t launch_rope_table(const int32_t *positions, const double *inv_freq, int rows, int hd, float2 *cs, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (hd > 128) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rope_table_kernel, dim3(rows), dim3(64), 0, st, positions, inv_freq, hd >> 1, cs);
  return hipGetLastError();
}

hipError_t launch_swiglu_bwd(const bf16_t *dhm, const Parts &parts, const bf16_t *gu, int rows, int F, bf16_t *dgu, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  if (F % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(swiglu_bwd_kernel, dim3(rows, cdiv(F, 2048)), dim3(256), 0, st, dhm, parts, gu, F, dgu);
  return hipGetLastError();
}

hipError_t launch_swiglu_fwd(const SwigluRows *groups, int n_groups, int F, hipStream_t st) {
  if (n_groups < 1 || n_groups > 2 || F % 4) return hipErrorInvalidValue;
  SwigluRows g0 = groups[0], g1 = {};
  if (n_groups > 1) g1 = groups[1];
  if (g0.rows < 0 || g1.rows < 0) return hipErrorInvalidValue;
  if (g0.rows + g1.rows == 0) return hipSuccess;
  hipLaunchKernelGGL(swiglu_fwd_kernel, dim3(g0.rows + g1.rows, cdiv(F, 1024)), dim3(256), 0, st, g0, g1, F);
  return hipGetLastError();
}

hipError_t launch_split_f32(const SplitRange *ranges, int n_ranges, hipStream_t st) {
  if (n_ranges > MAX_SPLIT_RANGES) return hipErrorInvalidValue;
  SplitJobs jobs = {};
  int n = 0;
  unsigned blocks = 0;
  for (int i = 0; i < n_ranges; ++i) {
    const SplitRange &r = ranges[i];
    if (r.n == 0) continue;
    const size_t n4 = ((uintptr_t)r.src & 15) || (((uintptr_t)r.hi | (uintptr_t)r.lo) & 7) ? 0 : r.n / 4;
    const size_t want = ((n4 ? n4 + 3 : r.n) + 255) / 256;
    const unsigned count = (unsigned)(want < 16384 ? want : 16384);
    jobs.j[n++] = SplitJob{r, n4, blocks, count};
    blocks += count;
  }
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(split_f32_kernel, dim3(blocks), dim3(256), 0, st, jobs, n);
  return hipGetLastError();
}

namespace {
__global__ __launch_bounds__(256) void head_norm_stats_kernel(const float *__restrict__ norms, const int32_t *__restrict__ t_count,
                                                              int n, int H, float *__restrict__ abar, int32_t *__restrict__ last_used,
                                                              int window, float tau, int32_t *__restrict__ prune) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n * H) return;
  const int t = t_count[i / H];
  if (t < 1) return;              // a request that has had no decode iteration: nothing to average over
  const float v = norms[i], a = abar[i];
  abar[i] = a + (v - a) / (float)t;
  if (prune) {
    const bool low = v < tau;
    prune[i] = (t - last_used[i] > window || low) ? 1 : 0;
    if (!low) last_used[i] = t;
  }
}
}  // namespace

hipError_t launch_head_norm_stats(const float *norms, const int32_t *t_count, int n, int H, float *abar, int32_t *last_used,
                                  int window, float tau, int32_t *prune, hipStream_t st) {
  if (n <= 0 || H <= 0) return hipSuccess;
  hipLaunchKernelGGL(head_norm_stats_kernel, dim3((unsigned)cdiv(n * H, 256)), dim3(256), 0, st, norms, t_count, n, H, abar, last_used, window, tau, prune);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float *dst, size_t n, float v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const unsigned blocks = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
  hipLaunchKernelGGL(fill_f32_kernel, dim3(blocks), dim3(256), 0, st, dst, n, v);
  return hipGetLastError();
}

hipError_t launch_sum_parts(const SumRange *ranges, int n_ranges, bool out_bf16, hipStream_t st) {
  if (n_ranges < 1 || n_ranges > 3) return hipErrorInvalidValue;
  SumRange s[3] = {};
  size_t n = 0;
  for (int i = 0; i < n_ranges; ++i) {
    s[i] = ranges[i];
    n += s[i].n;
    if (s[i].n % 4) return hipErrorInvalidValue;
  }
  if (n == 0) return hipSuccess;
  const size_t want = (n / 4 + 255) / 256;
  const dim3 grid((unsigned)(want < 4096 ? want : 4096));
  if (out_bf16) hipLaunchKernelGGL(sum_parts_kernel<true>, grid, dim3(256), 0, st, s[0], s[1], s[2]);
  else hipLaunchKernelGGL(sum_parts_kernel<false>, grid, dim3(256), 0, st, s[0], s[1], s[2]);
  return hipGetLastError();
}
