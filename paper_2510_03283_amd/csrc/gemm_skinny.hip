// Weight-streaming products of a few activation rows: C[m, n] = sum_k A[m, k] W[n, k], at most 128 rows m, W bf16 [N, K].
//
// With a handful of rows a product reads its weights once and does almost nothing else, so it is bound by the
// weight stream, not by the matrix cores.  The tiles of the large kernels put such a problem on N / 128 blocks that
// walk K one after the other (16 .. 250 of 256 CUs busy, one 64-wide k tile in flight each).  Here a block owns groups of
// 16 (8) weight rows, and its eight waves split K among them: a wave streams its own 64-wide k chunks global -> LDS
// into a ring of its own (no barrier in the loop) and multiplies them from there; the partial tiles of the eight waves
// are added through LDS once, in a fixed order.  The activations are re-read by every block, out of L2, in fragment
// order (frag_index), which the kernels in front write.
// The weights go through LDS although only one wave uses them: MFMA fragments loaded directly put neighbouring lanes on
// different rows, and the address path then takes 4 x the cycles of a load whose neighbouring lanes share a line
// (32000 x 4096 at one row: 55 us against 46; 2048 x 5632: 8.4 against 5.8).
// The row-wise work around such a product is folded into it, because a launch costs as much as a small product:
//  * RMSNorm.  C = rstd[m] * sum_k (x[m, k] g[k]) W[n, k], so bf16(x g) is what is multiplied and rstd is applied to the
//    sums.  In front of gate / up the output projection, which forms x, leaves bf16(x g) in fragment order and each
//    block's share of the rows' sums of squares; in front of QKV, for few rows, a block converts the rows as it loads
//    them and gathers the sum on the way (its waves together see all of K).
//  * epilogue: rotary embedding, operand rounding and cache append (QKV), SwiGLU (gate / up), residual (output and
//    down projections).  The partners of an epilogue sit in one block: rows i .. i + 7 and i + hd/2 .. of a head,
//    or the gate and the up rows of the same eight hidden units, and in lanes l and l + 32 of one wave.
#include "kernels.h"

#include <algorithm>

namespace {

constexpr int SK_HALF_BELOW = 192;      // 16-row groups below which 8-row groups are used (fp32 outputs)
constexpr int SK_KC = 64;      // k elements of a chunk: 128 bytes of a weight row

typedef __attribute__((ext_vector_type(4))) uint32_t sk_u32x4_t;
typedef __attribute__((address_space(3))) void sk_lds_void_t;
typedef __attribute__((address_space(1))) const void sk_gbl_void_t;

__device__ __forceinline__ sk_u32x4_t sk_ld(const char *base, uint32_t off) { return *(const sk_u32x4_t *)(base + off); }

__device__ __forceinline__ float sk_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float sk_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Fragment reads of NC groups out of a ring slot, STRIDE bytes apart.  `landed`: the last activations requested behind the slot's
// weights - the compiler waits for those, hence for the weights.  One block of asm that ends with its wait: the compiler takes
// the outputs as written when it ends.
template <int NC, int STRIDE>
__device__ __forceinline__ void sk_read(sk_u32x4_t (&w)[NC], uint32_t at, const sk_u32x4_t &landed) {
  if constexpr (NC == 1)
    asm volatile("ds_read_b128 %0, %1\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0])
                 : "v"(at), "v"(landed)
                 : "memory");
  else if constexpr (NC == 2)
    asm volatile("ds_read_b128 %0, %2\n\t"
                 "ds_read_b128 %1, %2 offset:%4\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1])
                 : "v"(at), "v"(landed), "i"(STRIDE)
                 : "memory");
  else if constexpr (NC == 3)
    asm volatile("ds_read_b128 %0, %3\n\t"
                 "ds_read_b128 %1, %3 offset:%5\n\t"
                 "ds_read_b128 %2, %3 offset:%6\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2])
                 : "v"(at), "v"(landed), "i"(STRIDE), "i"(2 * STRIDE)
                 : "memory");
  else if constexpr (NC == 4)
    asm volatile("ds_read_b128 %0, %4\n\t"
                 "ds_read_b128 %1, %4 offset:%6\n\t"
                 "ds_read_b128 %2, %4 offset:%7\n\t"
                 "ds_read_b128 %3, %4 offset:%8\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(at), "v"(landed), "i"(STRIDE), "i"(2 * STRIDE), "i"(3 * STRIDE)
                 : "memory");
  else if constexpr (NC == 6)
    asm volatile("ds_read_b128 %0, %6\n\t"
                 "ds_read_b128 %1, %6 offset:%8\n\t"
                 "ds_read_b128 %2, %6 offset:%9\n\t"
                 "ds_read_b128 %3, %6 offset:%10\n\t"
                 "ds_read_b128 %4, %6 offset:%11\n\t"
                 "ds_read_b128 %5, %6 offset:%12\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5])
                 : "v"(at), "v"(landed), "i"(STRIDE), "i"(2 * STRIDE), "i"(3 * STRIDE), "i"(4 * STRIDE), "i"(5 * STRIDE)
                 : "memory");
  else {
    static_assert(NC == 8, "one to four, six or eight groups");
    asm volatile("ds_read_b128 %0, %8\n\t"
                 "ds_read_b128 %1, %8 offset:%10\n\t"
                 "ds_read_b128 %2, %8 offset:%11\n\t"
                 "ds_read_b128 %3, %8 offset:%12\n\t"
                 "ds_read_b128 %4, %8 offset:%13\n\t"
                 "ds_read_b128 %5, %8 offset:%14\n\t"
                 "ds_read_b128 %6, %8 offset:%15\n\t"
                 "ds_read_b128 %7, %8 offset:%16\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
                 : "v"(at), "v"(landed), "i"(STRIDE), "i"(2 * STRIDE), "i"(3 * STRIDE), "i"(4 * STRIDE), "i"(5 * STRIDE), "i"(6 * STRIDE), "i"(7 * STRIDE)
                 : "memory");
  }
}

// Weight rows of a group, and the groups of a product.
template <bool HALF, int EPI>
__host__ __device__ constexpr int sk_groups(int N) { return EPI == SK_E_SWIGLU || HALF ? N / 8 : N / 16; }

// NW: waves of a block, which share K.  MT: 16-row tiles of A.  NC: 16-row groups of W per block.  HALF: groups of 8 rows (the upper half of an MFMA tile
// repeats the lower one and is dropped) for outputs too narrow to give every CU a block otherwise.  D: chunks in the
// ring of a wave, D - 1 of them in flight while one is multiplied.
template <int MT, int NC, int D, bool HALF, int ASRC, int EPI, int NW>
__global__ __launch_bounds__(64 * NW) void skinny_kernel(const SkinnyParams p) {
  constexpr int SK_WAVES = NW, SK_THR = 64 * NW;
  constexpr bool NORM = ASRC != SK_A_FRAG;
  constexpr bool SCALE = ASRC == SK_A_FRAG && EPI == SK_E_SWIGLU;   // rows scaled by rstd from partial sums of squares
  constexpr int WR = HALF ? 8 : 16;                  // weight rows of a group
  constexpr int NJ = WR / 8;                         // direct loads per group and chunk (8 rows x 128 bytes each)
  constexpr int SLOT = NC * WR * SK_KC * 2;          // bytes of a ring slot
  constexpr int RING = SK_WAVES * D * SLOT;
  constexpr int RED = SK_WAVES * MT * NC * 1024;      // the partial tiles of the waves, in the ring's place
  static_assert(RING <= 144 * 1024 && RED <= 144 * 1024, "LDS budget of a gfx950 CU");
  __shared__ __align__(16) unsigned char smem[RING > RED ? RING : RED];
  __shared__ float ssq[NORM ? SK_WAVES : 1][MT * 16];      // sums of squares by wave (SCALE: complete)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (uniform: matrix instructions ignore the lane mask)
  const int n = lane & 15, g = lane >> 4;
  // A block's groups: the blocks share all of them evenly (block b starts at group b groups / blocks), NC is the most one of them owns.  Whole shares and the rest come from the host: the two 64-bit
  // divisions were 300 of 400 instructions in front of the first request, 0.2 - 0.4 us of every launch (forward of one row through a layer of four products, 1536 wide, d_ff 3072, weights from HBM: 35.4 -> 33.8 us).
  const int groups = sk_groups<HALF, EPI>(p.N);
  int G0 = (int)blockIdx.x * p.share, own = p.share;
  if (p.rest) {      // (b rest < 2^32: sk_launch)
    const uint32_t z = blockIdx.x * (uint32_t)p.rest, q = z / gridDim.x;
    G0 += (int)q;
    own += z - q * gridDim.x + p.rest >= gridDim.x ? 1 : 0;
  }

  // weight rows: direct load j of group c takes rows 8 j + lane / 8 of the group, 16-byte piece lane % 8 of the chunk,
  // swizzled so that the fragment reads below meet no bank conflicts
  const char *wbase[NC][NJ];
  uint32_t woff[NC][NJ];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int G = G0 + min(c, own - 1);      // (groups past the last repeat it, their results are dropped)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int r8 = lane >> 3, r = 8 * j + r8;
      const uint32_t piece = (uint32_t)((lane & 7) ^ ((r >> 1) & 7)) * 16;
      long long row;
      if constexpr (EPI == SK_E_QKV) {
        const int gph = p.hd >> 4, head = G / gph, hq = p.Hq, hk = p.Hkv;
        wbase[c][j] = (const char *)(head < hq ? p.w[0] : (head < hq + hk ? p.w[1] : p.w[2]));
        row = (head < hq ? head : (head < hq + hk ? head - hq : head - hq - hk)) * p.hd + (G % gph) * 8 + r8 + j * (p.hd >> 1);
      } else if constexpr (EPI == SK_E_SWIGLU) {
        wbase[c][j] = (const char *)p.w[j];
        row = G * 8 + r8;
      } else {
        wbase[c][j] = (const char *)p.w[0];
        row = G * WR + r;
      }
      woff[c][j] = (uint32_t)(row * p.K * 2) + piece;
    }
  }
  // activation fragments of this lane in every row tile
  const char *arow[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    if constexpr (ASRC == SK_A_FRAG) arow[t] = (const char *)p.a + (size_t)min(t, (p.M - 1) >> 4) * (p.K >> 5) * 1024 + lane * 16;      // (a tile without rows repeats the last)
    else arow[t] = (const char *)p.a + ((long long)min(t * 16 + n, p.M - 1) * p.K + g * 8) * 2;      // (rows past the last repeat it, their results are dropped)
  }
  const char *const gbase = (const char *)p.gain;

  f32x4_t acc[MT][NC];
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[t][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float ss[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) ss[t] = 0.f;

  const int nch = p.K / SK_KC;
  // blocks of one XCD start at different chunks, so that they do not ask the same channels for their rows at once
  const int rot = (int)((blockIdx.x >> 3) * 8u % (unsigned)nch);
  struct Acts { sk_u32x4_t a[2][MT], gn[NORM ? 2 : 1]; };
  const uint32_t ring0 = (uint32_t)(uintptr_t)(sk_lds_void_t *)smem + wave * (D * SLOT);
  auto kbyte = [&](int c) __attribute__((always_inline)) -> uint32_t {
    int cc = c + rot;
    cc -= cc >= nch ? nch : 0;
    return (uint32_t)cc * (SK_KC * 2);
  };
  // The weights of a chunk are requested before its activations (kept in that order), and loads return in order: once
  // the activations are there, the weights are in LDS.
  auto load = [&](Acts &s, int slot, int c) __attribute__((always_inline)) {
    const uint32_t kb = kbyte(c);
#pragma unroll
    for (int cg = 0; cg < NC; ++cg)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        sk_gbl_void_t *const src = (sk_gbl_void_t *)(wbase[cg][j] + (woff[cg][j] + kb));
        sk_lds_void_t *const dst = (sk_lds_void_t *)(smem + wave * (D * SLOT) + slot * SLOT + (cg * NJ + j) * 1024);
        if (p.stream) __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 2);      // non-temporal
        else __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (NORM) s.gn[h] = sk_ld(gbase, kb + 64 * h + g * 16);
#pragma unroll
      for (int t = 0; t < MT; ++t) s.a[h][t] = sk_ld(arow[t], ASRC == SK_A_FRAG ? (kb + 64 * h) * 16 : kb + 64 * h);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // fragment of k step h, group cg: row n (HALF: n % 8), logical piece 4 h + g
  const uint32_t frow = HALF ? (n & 7) : n;
  uint32_t faddr[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) faddr[h] = ring0 + frow * 128 + (((4 * h + g) ^ ((frow >> 1) & 7)) << 4);
  auto mult = [&](Acts &s, int slot) __attribute__((always_inline)) {
    sk_u32x4_t w[2][NC];
#pragma unroll
    for (int h = 0; h < 2; ++h) sk_read<NC, WR * 128>(w[h], faddr[h] + (uint32_t)(slot * SLOT), s.a[1][MT - 1]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        sk_u32x4_t f;
        if constexpr (ASRC == SK_A_FRAG) {
          f = s.a[h][t];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x0 = sk_lo(s.a[h][t][e]), x1 = sk_hi(s.a[h][t][e]);
            ss[t] = fmaf(x0, x0, ss[t]);
            ss[t] = fmaf(x1, x1, ss[t]);
            f[e] = cvt_pk_bf16(x0 * sk_lo(s.gn[h][e]), x1 * sk_hi(s.gn[h][e]));
          }
        }
#pragma unroll
        for (int cg = 0; cg < NC; ++cg)
          acc[t][cg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[h][cg]), __builtin_bit_cast(bf16x8_t, f), acc[t][cg], 0, 0, 0);
      }
  };
  // Row scales from the partial sums of squares: SK_THR / rows threads share a row.  Requested before the ring is
  // filled and added while its first chunks are in flight (added behind the loop, row by row, it cost a 22016 x 4096
  // product of 64 rows 15 us of 70).
  constexpr int TPR = SK_THR / (MT > 4 ? 128 : (MT == 3 ? 64 : MT * 16));
  if constexpr (SCALE) {
    const int m = (int)threadIdx.x / TPR;
    float v = 0.f;
    if (p.ss_in && m < p.M) {
      const float *src = p.ss_in + (size_t)m * p.ss_n;
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
      for (int i = ((int)threadIdx.x % TPR) * 4; i < p.ss_n; i += TPR * 4) {      // ss_n % 4 == 0
        const float4 q = *(const float4 *)(src + i);
        a.x += q.x; a.y += q.y; a.z += q.z; a.w += q.w;
      }
      v = (a.x + a.y) + (a.z + a.w);
    }
#pragma unroll
    for (int o = 1; o < TPR; o <<= 1) v += __shfl_xor(v, o, 64);
    if (threadIdx.x % TPR == 0 && m < MT * 16) ssq[0][m] = v;
  }
  {
    // a wave's chunks are SK_WAVES apart
    Acts ring[D];
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
      if (wave + i * SK_WAVES < nch) load(ring[i], i, wave + i * SK_WAVES);
    for (int c = wave; c < nch; c += D * SK_WAVES) {
#pragma unroll
      for (int i = 0; i < D; ++i) {
        const int cl = c + (i + D - 1) * SK_WAVES;
        if (cl < nch) load(ring[(i + D - 1) % D], (i + D - 1) % D, cl);
        if (c + i * SK_WAVES < nch) mult(ring[i], i);
      }
    }
  }
  if constexpr (NORM) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      float v = ss[t];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (lane < 16) ssq[wave][t * 16 + lane] = v;
    }
  }
  typedef float4 (*red_t)[MT * NC][64];
  const red_t red = (red_t)smem;
  __syncthreads();      // the ring becomes the place of the partial tiles
  // sum over the waves: unit (tile, lane) of four outputs per thread
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int c = 0; c < NC; ++c) red[wave][t * NC + c][lane] = make_float4(acc[t][c][0], acc[t][c][1], acc[t][c][2], acc[t][c][3]);
  __syncthreads();
  for (int unit = wave; unit < MT * NC; unit += SK_WAVES) {
    const int t = unit / NC, c = unit % NC, G = G0 + c;
    if (c >= own) continue;
    float4 v = red[0][unit][lane];
#pragma unroll
    for (int w = 1; w < SK_WAVES; ++w) {
      const float4 o = red[w][unit][lane];
      v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
    }
    const int m = t * 16 + n;      // this lane: output row m, weight rows 4 g .. 4 g + 3 of the group
    if constexpr (NORM) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < SK_WAVES; ++w) s += ssq[w][m];
      const float rs = 1.0f / sqrtf(s / (float)p.K + p.eps);
      v.x *= rs; v.y *= rs; v.z *= rs; v.w *= rs;
    }
    if constexpr (SCALE) {
      if (p.ss_in) {
        const float rs = 1.0f / sqrtf(ssq[0][m] / (float)p.K + p.eps);
        v.x *= rs; v.y *= rs; v.z *= rs; v.w *= rs;
      }
    }
    if constexpr (EPI == SK_E_F32) {
      const int col = HALF ? G * 8 + 4 * g : G * 16 + 4 * g;
      if (m < p.M && (!HALF || g < 2)) {
        const size_t o = (size_t)m * p.N + col;
        if (p.resid_kind == 1) {
          const float4 r = *(const float4 *)((const float *)p.resid + o);
          v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
        } else if (p.resid_kind == 2) {
          const uint2 r = *(const uint2 *)((const bf16_t *)p.resid + o);
          v.x += sk_lo(r.x); v.y += sk_hi(r.x); v.z += sk_lo(r.y); v.w += sk_hi(r.y);
        }
        *(float4 *)((float *)p.c + o) = v;
        if (p.next_a) {
          // what the product behind the next RMSNorm needs of this row: bf16(v gain) in fragment order, and the
          // block's share of the sum of squares (columns of one row sit in lanes n, n + 16, ...)
          const uint2 gn = *(const uint2 *)(p.next_gain + col);
          *(uint2 *)((bf16_t *)p.next_a + frag_index(m, col, p.N)) =
              make_uint2(cvt_pk_bf16(v.x * sk_lo(gn.x), v.y * sk_hi(gn.x)), cvt_pk_bf16(v.z * sk_lo(gn.y), v.w * sk_hi(gn.y)));
        }
      }
      if (p.next_a) {
        // (written out: which square is rounded on its own is otherwise up to the code around it)
        float q = m < p.M && (!HALF || g < 2) ? fmaf(v.w, v.w, fmaf(v.z, v.z, fmaf(v.y, v.y, v.x * v.x))) : 0.f;
        q += __shfl_xor(q, 16, 64);
        q += __shfl_xor(q, 32, 64);
        if (lane < 16 && m < p.M) p.ss_out[(size_t)m * groups + G] = q;
      }
    } else {
      // lanes of g = 0, 1 hold the first partner of rows 4 g .. 4 g + 3, lanes of g = 2, 3 the second
      const float4 q = make_float4(__shfl_xor(v.x, 32, 64), __shfl_xor(v.y, 32, 64), __shfl_xor(v.z, 32, 64), __shfl_xor(v.w, 32, 64));
      if constexpr (EPI == SK_E_SWIGLU) {
        if (g < 2 && m < p.M) {
          const float gg[4] = {v.x, v.y, v.z, v.w}, uu[4] = {q.x, q.y, q.z, q.w};
          float h[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) h[e] = gg[e] / (1.0f + expf(-gg[e])) * uu[e];
          *(uint2 *)((bf16_t *)p.c + frag_index(m, G * 8 + 4 * g, p.N)) = make_uint2(cvt_pk_bf16(h[0], h[1]), cvt_pk_bf16(h[2], h[3]));
        }
      } else {
        if (m >= p.M) continue;
        const int hd = p.hd, half = hd >> 1, gph = hd >> 4, head = G / gph, i = (G % gph) * 8 + 4 * (g & 1);
        float o[4] = {v.x, v.y, v.z, v.w};
        if (head < p.Hq + p.Hkv) {
          const float x[4] = {v.x, v.y, v.z, v.w}, y[4] = {q.x, q.y, q.z, q.w};
          const int pos = p.positions[m];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float2 cs = rope_angle((double)pos * p.inv_freq[i + e]);
            o[e] = g < 2 ? x[e] * cs.x - y[e] * cs.y : x[e] * cs.x + y[e] * cs.y;
          }
        }
        const uint2 w = make_uint2(cvt_pk_bf16(o[0], o[1]), cvt_pk_bf16(o[2], o[3]));
        const int e0 = i + (g < 2 ? 0 : half);
        if (head < p.Hq) {
          *(uint2 *)((bf16_t *)p.q + (size_t)m * p.Hq * hd + head * hd + e0) = w;
        } else {
          const bool isk = head < p.Hq + p.Hkv;
          const int kh = head - p.Hq - (isk ? 0 : p.Hkv);
          *(uint2 *)((bf16_t *)(isk ? p.k : p.v) + (size_t)m * p.Hkv * hd + kh * hd + e0) = w;
          const long long slot = p.slots[m];
          if (slot >= 0 && slot < p.num_slots) {
            const long long B = p.block_size;
            bf16_t *cache = (bf16_t *)(isk ? p.cache_k : p.cache_v);
            *(uint2 *)(cache + ((slot / B) * p.Hkv + kh) * B * hd + (slot % B) * hd + e0) = w;
          }
        }
      }
    }
  }
}

template <int MT, int NC, int D, bool HALF, int ASRC, int EPI, int NW = 8>
hipError_t sk_launch(const SkinnyParams &params, int blocks, hipStream_t st, int tile[2]) {
  const int groups = sk_groups<HALF, EPI>(params.N);
  if (blocks > 65535) blocks = groups;      // no rest then
  SkinnyParams p = params;
  p.share = groups / blocks;
  p.rest = groups % blocks;
  tile[0] = MT * 16;
  tile[1] = groups * (HALF ? 8 : 16) / blocks;      // on average
  hipLaunchKernelGGL((skinny_kernel<MT, NC, D, HALF, ASRC, EPI, NW>), dim3(blocks), dim3(64 * NW), 0, st, p);
  return hipGetLastError();
}

// Groups of 16 weight rows per block.  A reduction of less than 1024, up to 16 rows, and outputs of fewer than 192 groups:
//  * four groups where that still gives most CUs a block: the activations then cross L2 -> CU once per 64 weight rows.  At most 16 rows prefer two where the
//    reduction is short, or where the last round of blocks of four would leave more than an eighth of the chip idle.  One / two / four groups in us, weights from
//    HBM (more copies in turn than the last-level cache holds), 16 rows: 32000 x 2048 23.4 / 21.6 / 23.6, 32000 x 4096 44.2 / 41.8 / 40.5, gate | up
//    2 x 11008 x 4096 (344 blocks of four) 32.6 / 29.4 / 35.7;
//  * between 512 and 1024 groups, at most 16 rows, one block a CU that owns three or four: gate | up 2 x 5632 x 2048 10.0 us (176 blocks of four 11.1), 12288 x 4096
//    17.4 (192 blocks of four 18.4);
//  * one otherwise; 8-row groups where 16-row groups would leave CUs without a block (2048 x 5632 at one row: 6.5 -> 5.8 us; 64 rows, 2048 x 2048 7.8 -> 7.1; at
//    192 groups whole ones are ahead: 3072 x 2048 at 16 rows 5.0 against 6.1, at 64 rows 8.1 against 12.1).
// More rows on more than that: loads of a wave return in order, so the weights (about 25 GB/s a CU, all CUs reading HBM) and the activations
// (L2, about 110) add up, per block  weights + activations  with one block a CU at a time.  Neither a deeper ring nor more blocks in flight changes that, only
// fewer activation reads and no partly filled round do: so all blocks run in whole rounds of one a CU, share the groups evenly, and own up to
// eight (four from 65 rows on, whose accumulators fill the registers); sk_cost prices the candidates.  Four waves leave a block of many groups its registers.
// (The waves that share K follow from rows and groups, and with them the order in which the products of a row are added: its last bits depend on the size of the batch.)
// us at 32 / 64 / 128 rows, blocks of four groups (before) and so: 12288 x 4096 21.0 / 26.9 / 39.6 -> 18.4 / 23.2 / 32.2, 2 x 11008 x 4096 43.4 / 50.6 / 77 -> 32.0 / 36.3 /
// 58.9, 32000 x 4096 47.6 / 54.9 / 78 -> 42.9 / 45.9 / 78, 2 x 5632 x 2048 12.6 / 15.6 / 23.3 -> 11.3 / 14.2 / 19.1, 32000 x 2048 28.2 / 32.9 / 47 -> 25.4 / 28.8 / 47.
constexpr int SK_CUS = 256;
template <int NC, int MT>
double sk_cost(int groups, int K) {      // in units of the time 25 weight rows take; a block's start and merge as 1500 elements of k
  const int rounds = cdiv(cdiv(groups, NC), SK_CUS);
  return rounds * (0.64 * NC + 0.145 * MT + 1500.0 / K);
}
template <int ASRC, int EPI, int MT, int NC>
hipError_t sk_even(const SkinnyParams &p, int groups, hipStream_t st, int tile[2]) {
  constexpr int NW = NC == 1 ? (MT > 4 ? 4 : 8) : (NC >= 6 || MT > 4 || (NC == 3 && MT > 2) ? 4 : 8);
  constexpr int D = NC == 1 ? (NW == 4 ? 4 : 3) : (NC <= 3 && NW == 4 ? 3 : 2);
  // whole rounds of blocks that own NC groups at most
  const int blocks = cdiv(groups, NC), even = cdiv(blocks, SK_CUS) * SK_CUS;
  return sk_launch<MT, NC, D, false, ASRC, EPI, NW>(p, cdiv(groups, even) == NC ? std::min(groups, even) : blocks, st, tile);
}
template <int ASRC, int EPI, int MT>
hipError_t sk_cheapest(const SkinnyParams &p, int groups, hipStream_t st, int tile[2]) {
  const double c1 = sk_cost<1, MT>(groups, p.K), c2 = sk_cost<2, MT>(groups, p.K), c3 = sk_cost<3, MT>(groups, p.K), c4 = sk_cost<4, MT>(groups, p.K);
  const double c = std::min(std::min(c1, c2), std::min(c3, c4));
  if constexpr (MT <= 4) {
    const double c6 = sk_cost<6, MT>(groups, p.K), c8 = sk_cost<8, MT>(groups, p.K);
    if (c8 < c && c8 < c6) return sk_even<ASRC, EPI, MT, 8>(p, groups, st, tile);
    if (c6 < c) return sk_even<ASRC, EPI, MT, 6>(p, groups, st, tile);
  }
  if (c == c1) return sk_even<ASRC, EPI, MT, 1>(p, groups, st, tile);
  if (c == c2) return sk_even<ASRC, EPI, MT, 2>(p, groups, st, tile);
  if (c == c3) return sk_even<ASRC, EPI, MT, 3>(p, groups, st, tile);
  return sk_even<ASRC, EPI, MT, 4>(p, groups, st, tile);
}
template <int ASRC, int EPI, int MT>
hipError_t sk_pick(const SkinnyParams &p, hipStream_t st, int tile[2]) {
  const int groups = sk_groups<false, EPI>(p.N);
  if constexpr (EPI == SK_E_F32) {
    if (groups < SK_HALF_BELOW) {
      if constexpr (MT > 6) return sk_launch<MT, 1, 4, true, ASRC, EPI, 4>(p, 2 * groups, st, tile);
      else return sk_launch<MT, 1, 3, true, ASRC, EPI>(p, 2 * groups, st, tile);
    }
  }
  if constexpr (MT > 4) {
    return sk_cheapest<ASRC, EPI, MT>(p, groups, st, tile);
  } else {
    if constexpr (MT > 1) {
      if (p.K >= 1024 && groups >= SK_HALF_BELOW) return sk_cheapest<ASRC, EPI, MT>(p, groups, st, tile);
    } else {
      if (p.K >= 1024 && groups > 2 * SK_CUS && groups <= 4 * SK_CUS - 1)
        return groups <= 3 * SK_CUS ? sk_launch<MT, 3, 2, false, ASRC, EPI>(p, SK_CUS, st, tile) : sk_launch<MT, 4, 2, false, ASRC, EPI>(p, SK_CUS, st, tile);
      const bool short_round = p.K >= 1024 && cdiv(groups, 4 * SK_CUS) * 4 * SK_CUS * 7 > 8 * groups;
      if ((p.K <= 2048 || short_round) && groups >= 1024 && groups % 2 == 0) return sk_launch<MT, 2, 2, false, ASRC, EPI>(p, groups / 2, st, tile);
    }
    if (groups >= 640 && groups % 4 == 0) return sk_launch<MT, 4, 2, false, ASRC, EPI>(p, groups / 4, st, tile);
    return sk_launch<MT, 1, 3, false, ASRC, EPI>(p, groups, st, tile);
  }
}

template <int ASRC, int EPI>
hipError_t sk_rows(const SkinnyParams &p, hipStream_t st, int tile[2]) {
  if constexpr (ASRC != SK_A_FRAG || EPI != SK_E_QKV)      // (so few rows of QKV come with their RMSNorm)
    if (p.M <= 16) return sk_pick<ASRC, EPI, 1>(p, st, tile);
  if constexpr (ASRC == SK_A_FRAG) {
    if (p.M <= 32) return sk_pick<ASRC, EPI, 2>(p, st, tile);
    if (p.M <= 48) return sk_pick<ASRC, EPI, 3>(p, st, tile);      // never many more tiles than the rows fill: they cost as if they were full
    if (p.M <= 64) return sk_pick<ASRC, EPI, 4>(p, st, tile);
    if (p.M <= 80) return sk_pick<ASRC, EPI, 5>(p, st, tile);
    if (p.M <= 96) return sk_pick<ASRC, EPI, 6>(p, st, tile);
    return sk_pick<ASRC, EPI, 8>(p, st, tile);
  }
  return hipErrorInvalidValue;
}

}  // namespace

// groups of columns a fp32-output product of N columns is cut into
int skinny_parts(int N) { return N / 16 < SK_HALF_BELOW ? N / 8 : N / 16; }

// Weights of this many bytes are read with the non-temporal hint.  A layer with such products has weights of 30 MB and more, so those of a model of nine layers
// and more (three, from 90 MB a layer on) pass through the 256 MB of the last-level cache without ever being found in it again, and the hint spares their way into it.  us without / with it, weights from HBM, 16 rows: 3072 x 2048
// (12 MB) 5.6 / 4.6, 2048 x 5632 8.4 / 7.3, 2 x 5632 x 2048 10.9 / 10.0, 12288 x 4096 19.0 / 17.4, 32000 x 2048 24.7 / 21.6, 32000 x 4096 46.2 / 40.5; 2048 x 2048 (8 MB) 4.0
// / 4.0, and 3.8 / 4.7 where 24 copies in turn stay in the cache.  Forward of a layer of 30, 47 and 90 MB, 16 rows, layers in turn that do not fit the cache: 34.9 / 32.5, 42.1 / 37.6, 49.6 / 45.6, 64 rows 50.6 / 48.6, 60.1 / 56.4, 73.3 / 68.8.
// Two layers in turn, which stay in it, pay for the hint: 33.7 / 33.9, 39.6 / 41.3, 44.7 / 47.7, and at 64 rows 46.4 / 47.5, 54.7 / 58.0, 63.2 / 71.3.
constexpr long long SK_STREAM_BYTES = 12ll << 20;

hipError_t launch_skinny(const SkinnyParams &params, int asrc, int epi, hipStream_t st, const char **why, int tile[2]) {
  *why = nullptr;
  SkinnyParams p = params;
  if (p.M <= 0) return hipSuccess;
  p.stream = (long long)p.N * p.K * (epi == SK_E_SWIGLU ? 4 : 2) >= SK_STREAM_BYTES;
  for (int i = 0; i < (epi == SK_E_QKV ? 3 : (epi == SK_E_SWIGLU ? 2 : 1)); ++i)
    if (!p.w[i] || ((uintptr_t)p.w[i] & 15)) {      // 16-byte pieces go straight to LDS
      *why = "gemm: weights must be 16-byte aligned";
      return hipErrorInvalidValue;
    }
  // 32-bit byte offsets into the weights; whole chunks of k, whole groups of weight rows
  if (p.M > SKINNY_MAX_ROWS || p.K % SK_KC || p.K <= 0 || p.N % 16 || (long long)p.N * p.K * 2 >= (1ll << 32)) return hipErrorInvalidValue;
  if (epi == SK_E_QKV) {
    if (asrc == SK_A_FRAG) return sk_rows<SK_A_FRAG, SK_E_QKV>(p, st, tile);
    if (asrc == SK_A_NORM_BF16) return sk_rows<SK_A_NORM_BF16, SK_E_QKV>(p, st, tile);
  } else if (epi == SK_E_SWIGLU) {
    if (asrc == SK_A_FRAG) return sk_rows<SK_A_FRAG, SK_E_SWIGLU>(p, st, tile);
  } else if (epi == SK_E_F32) {
    if (asrc == SK_A_FRAG) return sk_rows<SK_A_FRAG, SK_E_F32>(p, st, tile);
  }
  return hipErrorInvalidValue;
}
