// Decode attention: one query row per request against its paged context, HBM-bound.
//
// Split-KV: grid (kv head, split, request); a block streams `chunk` tokens of one (request, kv head)
// once, for all query heads of the GQA group, with 16-byte loads per lane (a token row of hd
// elements is covered by hd/8 consecutive lanes, so a wave load touches whole token rows that
// are contiguous inside a cache block).  Every lane keeps its own online soft-max state over the
// tokens it sees; states are merged across lanes, waves and finally splits.  bf16 caches use packed
// dot products (v_dot2_f32_bf16) for q.k, DPP row operations for the per-token reduction and
// nontemporal loads (the cache is read once per iteration and should not displace the weights).
#include "kernels.h"

#include <algorithm>
#include <cstdlib>

namespace {

constexpr int MIN_PINNED = 512, MAX_CHUNK = 4096;   // tokens per block: a power of two, 128 .. MAX_CHUNK chosen per launch, from MIN_PINNED on a caller's choice
constexpr int UNR = 4;       // token loads in flight per lane for K and for V

__device__ __forceinline__ float safe_scale(float m_old, float m_new) {
  return m_old == -INFINITY ? 0.f : exp2f(m_old - m_new);
}

// Sum over the LPT (8 or 16) consecutive lanes that share a token row, result in every lane, with
// DPP row operations (quad swaps, then mirrors inside 8 and 16 lanes) - no LDS traffic.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int LPT>
__device__ __forceinline__ float group_sum(float d) {
  d += dpp_mov<0xB1>(d);                         // quad_perm [1,0,3,2]
  d += dpp_mov<0x4E>(d);                         // quad_perm [2,3,0,1]
  d += dpp_mov<0x141>(d);                        // row_half_mirror: the other quad of the 8 lanes
  if constexpr (LPT == 16) d += dpp_mov<0x140>(d);   // row_mirror: the other half of the 16 lanes
  return d;
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}

// FAST: block_size >= tokens per wave-wide load, so the tokens of one load share a cache block
// and the block-table entry is read once per load (wave-uniform) instead of once per lane.
template <int HD, int GRP, bool CBF, bool FAST>
__global__ __launch_bounds__(256) void attn_decode_kernel(const bf16_t *__restrict__ q, const void *__restrict__ ck,
                                                          const void *__restrict__ cv, long long num_blocks, int B,
                                                          int bshift, const int32_t *__restrict__ block_tables,
                                                          int max_blocks, const int32_t *__restrict__ ctx_lens, int Hq,
                                                          int Hkv, int nsplit, int chunk, float *__restrict__ partial) {
  constexpr int LPT = HD / 8;          // lanes per token row
  constexpr int TPL = 64 / LPT;        // tokens per wave-wide load
  constexpr int NW = CBF ? 4 : 8;      // 32-bit words of the 8 elements a lane holds
  __shared__ float sm[4][GRP][HD + 2];
  const int kvh = blockIdx.x, split = blockIdx.y, req = blockIdx.z;
  const int n_tot = ctx_lens[req] + 1;                    // cached context plus the new token
  const int c0 = split * chunk;
  if (c0 >= n_tot) return;
  const int c1 = min(n_tot, c0 + chunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int e0 = (lane % LPT) * 8, tl = lane / LPT;
  const float sc = 1.4426950408889634f / sqrtf((float)HD);

  // q: packed bf16 pairs for the bf16 cache (dot2), scaled floats for the fp32 cache
  uint32_t qp[GRP][4];
  float qv[GRP][8];
#pragma unroll
  for (int gi = 0; gi < GRP; ++gi) {
    const uint4 u = *(const uint4 *)(q + (size_t)req * Hq * HD + (size_t)(kvh * GRP + gi) * HD + e0);
    qp[gi][0] = u.x; qp[gi][1] = u.y; qp[gi][2] = u.z; qp[gi][3] = u.w;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      qv[gi][2 * e] = __uint_as_float(qp[gi][e] << 16);
      qv[gi][2 * e + 1] = __uint_as_float(qp[gi][e] & 0xffff0000u);
    }
  }
  float m[GRP], l[GRP], acc[GRP][8];
#pragma unroll
  for (int gi = 0; gi < GRP; ++gi) {
    m[gi] = -INFINITY; l[gi] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[gi][e] = 0.f;
  }

  const int32_t *bt = block_tables + (size_t)req * max_blocks;
  const int wbeg = c0 + wave * (chunk / 4), wend = min(c1, wbeg + chunk / 4);
  for (int tb = wbeg; tb < wend; tb += UNR * TPL) {
    long long off[UNR];
    bool ok[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int t0 = tb + u * TPL, t = t0 + tl;
      ok[u] = t < wend;
      long long blk = 0;
      if constexpr (FAST) {
        // t0 is a multiple of TPL <= B: the TPL tokens sit in one block, t0 < wend holds for the first lanes
        blk = t0 < wend ? __builtin_amdgcn_readfirstlane(bt[t0 >> bshift]) : -1;
      } else if (ok[u]) {
        blk = bt[t >> bshift];
      }
      ok[u] = ok[u] && blk >= 0 && blk < num_blocks;      // a bad table entry is ignored, never dereferenced
      off[u] = ok[u] ? ((blk * Hkv + kvh) * B + (t & (B - 1))) * (long long)HD + e0 : 0;
    }
    uint32_t kr[UNR][NW], vr[UNR][NW];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      if constexpr (CBF) {
        const u32x4_t a = __builtin_nontemporal_load((const u32x4_t *)((const bf16_t *)ck + off[u]));   // streamed once
        kr[u][0] = a.x; kr[u][1] = a.y; kr[u][2] = a.z; kr[u][3] = a.w;
      } else {
        const uint4 a = *(const uint4 *)((const float *)ck + off[u]), b2 = *(const uint4 *)((const float *)ck + off[u] + 4);
        kr[u][0] = a.x; kr[u][1] = a.y; kr[u][2] = a.z; kr[u][3] = a.w; kr[u][4] = b2.x; kr[u][5] = b2.y; kr[u][6] = b2.z; kr[u][7] = b2.w;
      }
    }
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      if constexpr (CBF) {
        const u32x4_t a = __builtin_nontemporal_load((const u32x4_t *)((const bf16_t *)cv + off[u]));
        vr[u][0] = a.x; vr[u][1] = a.y; vr[u][2] = a.z; vr[u][3] = a.w;
      } else {
        const uint4 a = *(const uint4 *)((const float *)cv + off[u]), b2 = *(const uint4 *)((const float *)cv + off[u] + 4);
        vr[u][0] = a.x; vr[u][1] = a.y; vr[u][2] = a.z; vr[u][3] = a.w; vr[u][4] = b2.x; vr[u][5] = b2.y; vr[u][6] = b2.z; vr[u][7] = b2.w;
      }
    }
    // Ignored tokens have loaded the first token of the pool, which may hold anything, and weight 0 does not remove an infinity or a NaN.  Only the
    // last turn of a wave has any, or one with a bad table entry.
    bool whole = true;
#pragma unroll
    for (int u = 0; u < UNR; ++u) whole = whole && ok[u];
    if (!__all(whole)) {
#pragma unroll
      for (int u = 0; u < UNR; ++u)
#pragma unroll
        for (int w = 0; w < NW; ++w) vr[u][w] = ok[u] ? vr[u][w] : 0u;
    }
    float vf[UNR][8];
#pragma unroll
    for (int u = 0; u < UNR; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (CBF) vf[u][e] = __uint_as_float((e & 1) ? (vr[u][e >> 1] & 0xffff0000u) : (vr[u][e >> 1] << 16));
        else vf[u][e] = __uint_as_float(vr[u][e]);
      }
#pragma unroll
    for (int gi = 0; gi < GRP; ++gi) {
      float sv[UNR];
      float mx = m[gi];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        float d = 0.f;
        if constexpr (CBF) {
#pragma unroll
          for (int e = 0; e < 4; ++e) d = dot2_bf16(kr[u][e], qp[gi][e], d);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) d += __uint_as_float(kr[u][e]) * qv[gi][e];
        }
        d = group_sum<LPT>(d) * sc;
        sv[u] = ok[u] ? d : -INFINITY;
        mx = fmaxf(mx, sv[u]);
      }
      if (mx == -INFINITY) continue;                // nothing valid seen yet by this lane group
      const float alpha = safe_scale(m[gi], mx);
      m[gi] = mx;
      l[gi] *= alpha;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[gi][e] *= alpha;
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const float p = exp2f(sv[u] - mx);          // exp2(-inf) = 0 for ignored tokens
        l[gi] += p;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[gi][e] += p * vf[u][e];
      }
    }
  }

  // merge the TPL lane groups of the wave (lanes with equal e0)
#pragma unroll
  for (int gi = 0; gi < GRP; ++gi) {
#pragma unroll
    for (int o = LPT; o < 64; o <<= 1) {
      const float m2 = __shfl_xor(m[gi], o, 64), l2 = __shfl_xor(l[gi], o, 64);
      const float mn = fmaxf(m[gi], m2);
      const float a1 = safe_scale(m[gi], mn), a2 = safe_scale(m2, mn);
      l[gi] = l[gi] * a1 + l2 * a2;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[gi][e] = acc[gi][e] * a1 + __shfl_xor(acc[gi][e], o, 64) * a2;
      m[gi] = mn;
    }
    if (lane < LPT) {
#pragma unroll
      for (int e = 0; e < 8; ++e) sm[wave][gi][e0 + e] = acc[gi][e];
      if (lane == 0) { sm[wave][gi][HD] = m[gi]; sm[wave][gi][HD + 1] = l[gi]; }
    }
  }
  __syncthreads();
  // merge the 4 waves; thread t handles (gi, e) pairs
  for (int idx = tid; idx < GRP * HD; idx += 256) {
    const int gi = idx / HD, e = idx - gi * HD;
    float mn = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) mn = fmaxf(mn, sm[w][gi][HD]);
    float lo = 0.f, ao = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float a = safe_scale(sm[w][gi][HD], mn);
      lo += sm[w][gi][HD + 1] * a;
      ao += sm[w][gi][e] * a;
    }
    float *dst = partial + (((size_t)req * Hq + (kvh * GRP + gi)) * nsplit + split) * (HD + 2);
    dst[e] = ao;
    if (e == 0) { dst[HD] = mn; dst[HD + 1] = lo; }
  }
}

// Merges the splits of a (request, head): CG groups of HD threads take every CG-th split each, in one pass with its own soft-max
// state, and are merged through LDS, in order.  The time is the latency of the loads, so a group has those of CU splits in flight.
// (One group, first the maximum of all splits and then their sums: 8000 tokens in 32 splits 28 us with the kernel in front, in 63 splits 40;
// now 8000 tokens 12.2 and 12.8.)  Up to CU splits one group has all of them in flight, and idle groups would only fill the chip: 256 requests of 32 heads in
// one or two splits 7.9 us with four groups, 4.8 with one.
constexpr int CU = 4;
template <int HD, int CG>
__global__ __launch_bounds__(CG * HD) void attn_decode_combine_kernel(const float *__restrict__ partial,
                                                                      const int32_t *__restrict__ ctx_lens, int Hq, int nsplit, int chunk,
                                                                      bf16_t *__restrict__ out, float *__restrict__ norms, int frag_row0) {
  __shared__ float sa[CG][HD], sml[CG][2];
  const int req = blockIdx.x, h = blockIdx.y, e = threadIdx.x % HD, g = threadIdx.x / HD;
  const int ns = min(nsplit, (ctx_lens[req] + 1 + chunk - 1) / chunk);
  const float *src = partial + ((size_t)req * Hq + h) * nsplit * (HD + 2);
  float m = -INFINITY, l = 0.f, a = 0.f;
  for (int s0 = g; s0 < ns; s0 += CG * CU) {
    float mv[CU], lv[CU], av[CU], mn = m;
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const float *p = src + (size_t)min(s0 + u * CG, ns - 1) * (HD + 2);
      mv[u] = p[HD];
      lv[u] = p[HD + 1];
      av[u] = p[e];
    }
    // slots past the end add nothing (a sum can be infinite, so weight 0 alone does not do it); behind the asm, or every load gets a branch of its own
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      asm volatile("" : "+v"(mv[u]), "+v"(lv[u]), "+v"(av[u]));
      const bool ok = s0 + u * CG < ns;
      mv[u] = ok ? mv[u] : -INFINITY;
      lv[u] = ok ? lv[u] : 0.f;
      av[u] = ok ? av[u] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < CU; ++u) mn = fmaxf(mn, mv[u]);
    const float al = safe_scale(m, mn);
    l *= al;
    a *= al;
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const float w = safe_scale(mv[u], mn);
      l += lv[u] * w;
      a += av[u] * w;
    }
    m = mn;
  }
  if constexpr (CG > 1) {
    sa[g][e] = a;
    if (e == 0) { sml[g][0] = m; sml[g][1] = l; }
    __syncthreads();
  }
  // (every thread stays to the end: there is a barrier in the norms)
  float n2 = 0.f;
  if (g == 0) {
    if constexpr (CG > 1) {
      float mn = sml[0][0];
#pragma unroll
      for (int k = 1; k < CG; ++k) mn = fmaxf(mn, sml[k][0]);
      l = a = 0.f;
#pragma unroll
      for (int k = 0; k < CG; ++k) {
        const float w = safe_scale(sml[k][0], mn);
        l += sml[k][1] * w;
        a += sa[k][e] * w;
      }
    }
    const float v = l > 0.f ? a / l : 0.f;
    out[frag_row0 >= 0 ? frag_index(frag_row0 + req, h * HD + e, Hq * HD) : ((size_t)req * Hq + h) * HD + e] = f2bf(v);
    if (norms) n2 = wave_sum(v * v);             // L2 norm of the head's output vector (fp32 values)
  }
  if (norms) {
    if constexpr (HD > 64) {
      __shared__ float red[HD / 64];
      if (g == 0 && (e & 63) == 0) red[e >> 6] = n2;
      __syncthreads();
      n2 = red[0] + red[1];
    }
    if (threadIdx.x == 0) norms[(size_t)req * Hq + h] = sqrtf(n2);
  }
}

template <int HD, int GRP, bool CBF>
void launch_main(const bf16_t *q, const void *ck, const void *cv, long long num_blocks, int B, int bshift,
                 const int32_t *bt, int max_blocks, const int32_t *ctx, int n_decode, int Hq, int Hkv, int nsplit, int chunk,
                 float *partial, hipStream_t st) {
  if (B >= 64 / (HD / 8))
    hipLaunchKernelGGL((attn_decode_kernel<HD, GRP, CBF, true>), dim3(Hkv, nsplit, n_decode), dim3(256), 0, st, q, ck, cv, num_blocks, B, bshift, bt, max_blocks, ctx, Hq, Hkv, nsplit, chunk, partial);
  else
    hipLaunchKernelGGL((attn_decode_kernel<HD, GRP, CBF, false>), dim3(Hkv, nsplit, n_decode), dim3(256), 0, st, q, ck, cv, num_blocks, B, bshift, bt, max_blocks, ctx, Hq, Hkv, nsplit, chunk, partial);
}

template <int HD, bool CBF>
bool launch_grp(int grp, const bf16_t *q, const void *ck, const void *cv, long long num_blocks, int B, int bshift,
                const int32_t *bt, int max_blocks, const int32_t *ctx, int n_decode, int Hq, int Hkv, int nsplit, int chunk,
                float *partial, hipStream_t st) {
  switch (grp) {
    case 1: launch_main<HD, 1, CBF>(q, ck, cv, num_blocks, B, bshift, bt, max_blocks, ctx, n_decode, Hq, Hkv, nsplit, chunk, partial, st); return true;
    case 2: launch_main<HD, 2, CBF>(q, ck, cv, num_blocks, B, bshift, bt, max_blocks, ctx, n_decode, Hq, Hkv, nsplit, chunk, partial, st); return true;
    case 4: launch_main<HD, 4, CBF>(q, ck, cv, num_blocks, B, bshift, bt, max_blocks, ctx, n_decode, Hq, Hkv, nsplit, chunk, partial, st); return true;
    case 8: launch_main<HD, 8, CBF>(q, ck, cv, num_blocks, B, bshift, bt, max_blocks, ctx, n_decode, Hq, Hkv, nsplit, chunk, partial, st); return true;
    default: return false;
  }
}

}  // namespace

// Tokens per block.  A block's time has a fixed part (query, merge of its waves) and one that grows with its chunk; a grid that leaves the chip
// idle takes the time of one block, a larger one that of all its blocks.  In units of the work on 128 tokens a chunk of c tokens is priced as
//     LATENCY * hd / 64 * c / 128  +  blocks(c) * (c / 128 + fixed),    fixed = 0.08 query heads per kv head
// (a wave takes 32 tokens of 64-wide heads at a time, 16 of 128-wide ones), and the cheapest of 128, 256 and 512 is taken.  The constants are fitted to 936
// 1380 batches of 1 - 256 requests of 25 - 8000 tokens, 4 - 32 kv heads with 1 - 8 query heads each, 64 and 128 wide: on average 1.8 % above the best of the three
// (512 for all 22 % above it; 128 up to 4096 blocks, else 256 up to 10240 4.3 %, and up to 59 % above 512).  us at 128 / 256 / 512 tokens, both kernels, heads x kv heads x width
// 32 x 8 x 64: 1 request of 700 tokens 9.0 / 10.8 / 14.6; 32 of 400 - 1600 30.3 / 29.9 / 35.1; 64 of 100 - 400 27.3 / 23.9 / 25.1; 128 of 100 - 400 45.1 / 38.4 / 32.4;
// 256 of 50 - 200 47.8 / 38.3 / 45.7; 256 of 200 - 800 99 / 120 / 105; 128 of 400 - 1600 92 / 78 / 104; 32 x 32 x 128: 16 of 100 - 400 22.0 / 26.2 / 34.7; 64 of 100 -
// 400 51.7 / 55.7 / 52.4; 32 of 800 - 3200 165 / 158 / 161; 128 of 50 - 200 59.6 / 59.5 / 79.2.
// Past MOST_256 blocks of 256 the stream sets the time: long chunks mean fewer blocks that find nothing to do, fewer partial states to write and merge and a longer stream per
// block (6.2 -> 6.6 TB/s from 512 to 2048 tokens on a 256-request, 32-head batch) - as long as the grid still fills the chip several times over.
constexpr double LATENCY = 150;
constexpr long long MOST_256 = 10240;
static int decode_chunk_tokens(int n_decode, int Hq, int Hkv, int hd, int max_context, int chunk_tokens) {
  if (chunk_tokens) return chunk_tokens >= MIN_PINNED && chunk_tokens <= MAX_CHUNK && !(chunk_tokens & (chunk_tokens - 1)) ? chunk_tokens : -1;
  const long long streams = (long long)Hkv * n_decode;
  int chunk = 512;
  if (streams * cdiv(max_context + 1, 256) <= MOST_256) {
    double best = 0;
    for (int c = 128; c <= 512; c *= 2) {
      const double cost = LATENCY * hd / 64 * c / 128 + (double)(streams * cdiv(max_context + 1, c)) * (c / 128 + 0.08 * (Hq / Hkv));
      if (c == 128 || cost < best) { best = cost; chunk = c; }
    }
  }
  while (chunk >= 512 && chunk < MAX_CHUNK && streams * cdiv(max_context + 1, 2 * chunk) >= 8192) chunk *= 2;
  return chunk;
}

// Room for the partial states of this batch and of every smaller one (fewer requests, shorter contexts), which may take shorter chunks and have
// more blocks: the rule takes a chunk below MAX_CHUNK only up to a number of blocks, and a batch has at most streams * cdiv(context, chunk) of
// them.  256 tokens make at most MOST_256 blocks, 128 twice as many; 512 to 2048 are taken where twice the chunk makes fewer than 8192, so they make at most
// twice 8191 themselves.
size_t decode_partial_floats(int n_decode, int Hq, int Hkv, int hd, int max_context, int chunk_tokens) {
  const size_t streams = (size_t)n_decode * Hkv;
  auto blocks_of = [&](int chunk) { return streams * cdiv(max_context + 1, chunk); };
  size_t blocks;
  if (chunk_tokens) {
    const int chunk = decode_chunk_tokens(n_decode, Hq, Hkv, hd, max_context, chunk_tokens);
    blocks = blocks_of(chunk < 0 ? 512 : chunk);                       // an invalid override is rejected at launch; size for the worst case
  } else {
    blocks = std::max({std::min(blocks_of(128), (size_t)(2 * MOST_256)), std::min(blocks_of(256), (size_t)MOST_256), std::min(blocks_of(512), (size_t)2 * 8191),
                       blocks_of(MAX_CHUNK)});
  }
  return blocks * (Hq / Hkv) * (hd + 2);
}

hipError_t launch_attn_decode(const bf16_t *q, const void *cache_k, const void *cache_v, bool cache_bf16,
                              long long num_blocks, int block_size, const int32_t *block_tables, int max_blocks_per_req,
                              const int32_t *ctx_lens, int n_decode, int max_context, int Hq, int Hkv, int hd,
                              float *partial, bf16_t *out, float *norms, hipStream_t st, int chunk_tokens, int frag_row0) {
  if (n_decode <= 0) return hipSuccess;
  if (n_decode > 65535 || Hkv > 65535 || Hq > 65535) return hipErrorInvalidValue;
  int bshift = 0;
  while ((1 << bshift) < block_size) ++bshift;
  if ((1 << bshift) != block_size) return hipErrorInvalidValue;
  const int chunk = decode_chunk_tokens(n_decode, Hq, Hkv, hd, max_context, chunk_tokens);
  if (chunk < 0) return hipErrorInvalidValue;
  const int nsplit = cdiv(max_context + 1, chunk);
  if (nsplit > 65535) return hipErrorInvalidValue;
  const int grp = Hq / Hkv;
  bool ok = false;
  if (hd == 64) ok = cache_bf16 ? launch_grp<64, true>(grp, q, cache_k, cache_v, num_blocks, block_size, bshift, block_tables, max_blocks_per_req, ctx_lens, n_decode, Hq, Hkv, nsplit, chunk, partial, st)
                                : launch_grp<64, false>(grp, q, cache_k, cache_v, num_blocks, block_size, bshift, block_tables, max_blocks_per_req, ctx_lens, n_decode, Hq, Hkv, nsplit, chunk, partial, st);
  else if (hd == 128) ok = cache_bf16 ? launch_grp<128, true>(grp, q, cache_k, cache_v, num_blocks, block_size, bshift, block_tables, max_blocks_per_req, ctx_lens, n_decode, Hq, Hkv, nsplit, chunk, partial, st)
                                      : launch_grp<128, false>(grp, q, cache_k, cache_v, num_blocks, block_size, bshift, block_tables, max_blocks_per_req, ctx_lens, n_decode, Hq, Hkv, nsplit, chunk, partial, st);
  if (!ok) return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto combine = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(n_decode, Hq), dim3(threads), 0, st, partial, ctx_lens, Hq, nsplit, chunk, out, norms, frag_row0);
  };
  if (hd == 64) nsplit <= CU ? combine(attn_decode_combine_kernel<64, 1>, 64) : combine(attn_decode_combine_kernel<64, 4>, 256);
  else nsplit <= CU ? combine(attn_decode_combine_kernel<128, 1>, 128) : combine(attn_decode_combine_kernel<128, 4>, 512);
  return hipGetLastError();
}
