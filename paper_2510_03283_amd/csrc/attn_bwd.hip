// Backward of the varlen causal attention of the fine-tune sequences (bf16 MFMA, fp32 outputs).
//
// Two kernels, each free of atomics and of cross-lane transposes:
//  * dq kernel:  a wave owns 32 queries (a lane owns one query column of S^T = K Q^T and of
//    dP^T = V dO^T), walks the keys, and accumulates dQ^T = K^T dS^T.
//  * dkdv kernel: a wave owns 32 keys (a lane owns one key column of S = Q K^T and dP = dO V^T),
//    walks the queries of every query head of its GQA group, and accumulates
//    dV^T = dO^T P and dK^T = Q^T dS.
// P is recomputed from the saved log-sum-exp; D = rowsum(dO * O) is formed by the dq kernel from the
// fragments it loads anyway and handed to the dk/dv kernel through memory.
// The backward of the rotary embedding is part of both epilogues: the two halves (i, i + hd/2) of a
// head row sit in one lane (accumulator tiles t and t + hd/64), so dq and dk are rotated back by the
// row's angles (a per-row (cos, sin) table) and written, like dv, as bf16 straight into the
// [rows, (Hq + 2 Hkv) hd] operand of the projection backward - no fp32 dq / dk / dv in memory.
// Tiles of 64 rows go global -> LDS directly in their memory layout, two stages deep; the same
// tile feeds the products that reduce over the head dimension (16-byte reads) and those that
// reduce over the tile rows (transposing reads), see attn_tile.h.
#include "attn_tile.h"
#include "kernels.h"

namespace {

using namespace attn;

constexpr int TB = 64;    // rows per staged LDS tile

__device__ __forceinline__ bf16x8_t as_bf8(uint4 u) { return __builtin_bit_cast(bf16x8_t, u); }

__device__ __forceinline__ bf16x8_t pack8(const float *v) {
  return as_bf8(make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7])));
}

// Epilogue of a gradient row held as NOT accumulator tiles of 32 head-dim indices (register 4*rq + e of
// tile t = index 32 t + 8 rq + 4 g + e): rotate the pairs (i, i + HD/2) back by the row's angles
// (cs = (cos, sin) of the row, HD/2 entries; null = no rotation) and store as bf16 at dst[0 .. HD).
template <int HD>
__device__ __forceinline__ void store_grad_row(const f32x16_t (&acc)[HD / 32], const float2 *__restrict__ cs, int g, bf16_t *__restrict__ dst) {
  constexpr int NOT = HD / 32, HT = NOT / 2;
#pragma unroll
  for (int t = 0; t < HT; ++t)
#pragma unroll
    for (int rq = 0; rq < 4; ++rq) {
      const int i = t * 32 + 8 * rq + 4 * g;
      float a[4], b[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) { a[e] = acc[t][4 * rq + e]; b[e] = acc[t + HT][4 * rq + e]; }
      if (cs) {
        const float4 c01 = *(const float4 *)(cs + i), c23 = *(const float4 *)(cs + i + 2);
        const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float ra = a[e] * co[e] + b[e] * si[e], rb = b[e] * co[e] - a[e] * si[e];
          a[e] = ra; b[e] = rb;
        }
      }
      *(uint2 *)(dst + i) = make_uint2(cvt_pk_bf16(a[0], a[1]), cvt_pk_bf16(a[2], a[3]));
      *(uint2 *)(dst + i + HD / 2) = make_uint2(cvt_pk_bf16(b[0], b[1]), cvt_pk_bf16(b[2], b[3]));
    }
}

// ------------------------------------------------------------------ dQ
template <int HD>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_kernel(const bf16_t *__restrict__ q, const bf16_t *__restrict__ k,
                                                          const bf16_t *__restrict__ v, const bf16_t *__restrict__ o,
                                                          const bf16_t *__restrict__ d_o,
                                                          const float *__restrict__ lse, float *__restrict__ dvec,
                                                          const int32_t *__restrict__ seg, int row_base, int Hq, int Hkv,
                                                          const float2 *__restrict__ cs, bf16_t *__restrict__ dqkv,
                                                          const int32_t *__restrict__ excl_lo,
                                                          const int32_t *__restrict__ excl_hi) {
  constexpr int NKK = HD / 16, NOT = HD / 32, RK = HD == 128 ? 2 : 4;      // RK: operands read at a time
  using T = Tile<TB, HD, 256>;
  constexpr int STAGE = 2 * T::ELEMS;       // K tile, V tile
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t *lds = (bf16_t *)smem_raw;         // [2][STAGE]
  // blocks are dealt to the XCDs round-robin: block x takes head (x % Hkv) * group + x / Hkv, so the query heads
  // of one kv head (and all their row tiles) run on one XCD and its K and V stay in that XCD's L2
  const int kvh = blockIdx.x % Hkv, h = kvh * (Hq / Hkv) + blockIdx.x / Hkv, s = turned_sequence();
  const int r0 = seg[s] - row_base, L = seg[s + 1] - seg[s];
  const int q0 = (gridDim.z - 1 - blockIdx.z) * 128;
  if (q0 >= L) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, j = lane & 31;
  const int qw0 = q0 + wave * 32, qi = qw0 + j;
  const size_t qld = (size_t)Hq * HD, kld = (size_t)Hkv * HD;
  const bf16_t *kbase = k + (size_t)r0 * kld + (size_t)kvh * HD, *vbase = v + (size_t)r0 * kld + (size_t)kvh * HD;
  const int kend = min(L, q0 + 128);
  const int ntiles = (kend + TB - 1) / TB;
  const int xlo = excl_lo ? excl_lo[s] : L, xhi = excl_lo ? excl_hi[s] : L;   // queries >= xhi skip keys xlo .. xhi-1
  const uint32_t lane_off = T::lane_offset(kld);
  auto issue_tile = [&](int it) {
    bf16_t *S = lds + (it & 1) * STAGE;
    T::issue(kbase, kld, it * TB, L, lane_off, S);
    T::issue(vbase, kld, it * TB, L, lane_off, S + T::ELEMS);
  };
  issue_tile(0);

  // q and dO fragments of this lane's query; D = rowsum(dO * O) is formed on the way (each lane of the pair
  // (j, j + 32) holds half of the row) and written out for the dk/dv kernel
  bf16x8_t qf[NKK], dof[NKK];
  float dpart = 0.f;
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    uint4 a = make_uint4(0, 0, 0, 0), b = make_uint4(0, 0, 0, 0), c = make_uint4(0, 0, 0, 0);
    if (qi < L) {
      const size_t off = (size_t)(r0 + qi) * qld + (size_t)h * HD + kk * 16 + g * 8;
      a = *(const uint4 *)(q + off);
      b = *(const uint4 *)(d_o + off);
      c = *(const uint4 *)(o + off);
    }
    qf[kk] = as_bf8(a);
    dof[kk] = as_bf8(b);
    const uint32_t bw[4] = {b.x, b.y, b.z, b.w}, cw[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      dpart += __uint_as_float(bw[e] << 16) * __uint_as_float(cw[e] << 16) +
               __uint_as_float(bw[e] & 0xffff0000u) * __uint_as_float(cw[e] & 0xffff0000u);
  }
  const float dv_ = dpart + __shfl_xor(dpart, 32);
  const float sc = 1.4426950408889634f / sqrtf((float)HD), rs = 1.0f / sqrtf((float)HD);
  float lse2 = 0.f;
  if (qi < L) {
    lse2 = lse[(size_t)(r0 + qi) * Hq + h] * 1.4426950408889634f;
    if (g == 0) dvec[(size_t)(r0 + qi) * Hq + h] = dv_;
  }
  // MFMA row j reads tile row swap23(j): register r = 8*mm + e then holds key 16*mm + 8*g + e
  const uint32_t fk = T::frag_k_lane(swap23(j), g);
  const typename T::FragT ft = T::frag_t_init(lane);
  f32x16_t acc[NOT];
#pragma unroll
  for (int t = 0; t < NOT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

  for (int it = 0; it < ntiles; ++it) {
    wait_vmcnt<0>();
    __syncthreads();                                     // tile it has landed; the other stage is free
    if (it + 1 < ntiles) issue_tile(it + 1);
    const int kb = it * TB;
    if (kb > qw0 + 31) continue;
    if (qw0 >= xhi && kb >= xlo && kb + TB <= xhi) continue;
    const uint32_t Ks = T::lds_addr(lds + (it & 1) * STAGE), Vs = Ks + T::ELEMS * 2;
    static_for<0, 2>([&](auto ST) __attribute__((always_inline)) {
      constexpr int st = decltype(ST)::value, off = st * 32 * HD * 2;
      f32x16_t sa, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) { sa[r] = 0.f; dp[r] = 0.f; }
      static_for<0, NKK / RK>([&](auto KH) __attribute__((always_inline)) {
        constexpr int kk0 = RK * decltype(KH)::value;
        bf16x8_t a[RK], b[RK];
        T::template read_k<RK, kk0, off>(Ks, fk, a);
#pragma unroll
        for (int i = 0; i < RK; ++i) sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], qf[kk0 + i], sa, 0, 0, 0);
        T::template read_k<RK, kk0, off>(Vs, fk, b);
#pragma unroll
        for (int i = 0; i < RK; ++i) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[i], dof[kk0 + i], dp, 0, 0, 0);
      });
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) ds[r] = __builtin_amdgcn_exp2f(fmaf(sa[r], sc, -lse2)) * (dp[r] - dv_) * rs;
      // (the key of register r minus that of this lane's first register is a constant)
      if (kb + TB - 1 > qw0 || kb + TB > L) {
        const int last = min(qi, L - 1) - kb - 8 * g;
#pragma unroll
        for (int r = 0; r < 16; ++r) ds[r] = st * 32 + 16 * (r >> 3) + (r & 7) > last ? 0.f : ds[r];
      }
      if (qw0 + 31 >= xhi && kb < xhi && kb + TB > xlo) {
        const int lo = xlo - kb - 8 * g, n_ex = qi >= xhi ? xhi - xlo : 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) ds[r] = (uint32_t)(st * 32 + 16 * (r >> 3) + (r & 7) - lo) < (uint32_t)n_ex ? 0.f : ds[r];
      }
      const bf16x8_t dsf[2] = {pack8(ds), pack8(ds + 8)};
#pragma unroll
      for (int t = 0; t < NOT; ++t) {
        bf16x8_t a[2];
        T::template read_t<2, 2 * st>(Ks, ft, t, a);
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mm], dsf[mm], acc[t], 0, 0, 0);
      }
    });
  }
  if (qi < L)
    store_grad_row<HD>(acc, cs + (size_t)(r0 + qi) * (HD / 2), g, dqkv + (size_t)(r0 + qi) * (qld + 2 * kld) + (size_t)h * HD);
}

// ------------------------------------------------------------------ dK, dV
// QS teams of four waves share a block's 128 keys and take every QS-th query tile each; their sums are added in LDS at the end.
template <int HD, int QS>
__global__ __launch_bounds__(256 * QS, QS == 1 ? 2 : 1) void attn_bwd_dkdv_kernel(const bf16_t *__restrict__ q, const bf16_t *__restrict__ k,
                                                            const bf16_t *__restrict__ v, const bf16_t *__restrict__ d_o,
                                                            const float *__restrict__ lse, const float *__restrict__ dvec,
                                                            const int32_t *__restrict__ seg, int row_base, int Hq,
                                                            int Hkv, const float2 *__restrict__ cs, bf16_t *__restrict__ dqkv,
                                                            const int32_t *__restrict__ excl_lo, const int32_t *__restrict__ excl_hi) {
  constexpr int NKK = HD / 16, NOT = HD / 32, RK = HD == 128 ? 2 : 4;      // RK: operands read at a time
  using T = Tile<TB, HD, 256>;
  constexpr int STAGE = 2 * T::ELEMS + 4 * TB;    // Q tile, dO tile, lse[TB] and D[TB] as fp32 (2 bf16 slots each)
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  const int team = QS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  bf16_t *lds = (bf16_t *)smem_raw + team * 2 * STAGE;      // [QS][2][STAGE]
  const int kvh = blockIdx.x, s = turned_sequence(), grp = Hq / Hkv;
  const int r0 = seg[s] - row_base, L = seg[s + 1] - seg[s];
  const int k0 = blockIdx.z * 128;
  if (k0 >= L) return;
  const int tid = QS == 1 ? threadIdx.x : threadIdx.x & 255, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 5, j = lane & 31;
  const int kw0 = k0 + wave * 32, ki = kw0 + j;      // this lane's key
  const size_t qld = (size_t)Hq * HD, kld = (size_t)Hkv * HD;
  const int xlo = excl_lo ? excl_lo[s] : L, xhi = excl_lo ? excl_hi[s] : L;   // queries >= xhi skip keys xlo .. xhi-1
  const int nqt = (L - k0 + TB - 1) / TB;            // query tiles per head (k0 is a multiple of TB)
  const int niter = grp * nqt;
  const uint32_t lane_off = T::lane_offset(qld, tid);
  auto issue_tile = [&](int it) {
    const int gi = it / nqt, qb = k0 + (it % nqt) * TB;
    const int h = kvh * grp + gi;
    bf16_t *S = lds + (it / QS & 1) * STAGE;
    T::issue(q + (size_t)r0 * qld + (size_t)h * HD, qld, qb, L, lane_off, S, tid);
    T::issue(d_o + (size_t)r0 * qld + (size_t)h * HD, qld, qb, L, lane_off, S + T::ELEMS, tid);
    if (wave < 2) {                                  // one 4-byte element per lane: lane's value lands at base + 4*lane
      const int qq = qb + lane;
      const float *src = wave ? dvec : lse;
      const float *p = qq < L ? src + (size_t)(r0 + qq) * Hq + h : (const float *)&zero16;
      __builtin_amdgcn_global_load_lds((gbl_void_t *)p, (lds_void_t *)(S + 2 * T::ELEMS + wave * 2 * TB), 4, 0, 0);
    }
  };
  if (team < niter) issue_tile(team);

  bf16x8_t kf[NKK], vf[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    uint4 a = make_uint4(0, 0, 0, 0), b = make_uint4(0, 0, 0, 0);
    if (ki < L) {
      const size_t o = (size_t)(r0 + ki) * kld + (size_t)kvh * HD + kk * 16 + g * 8;
      a = *(const uint4 *)(k + o);
      b = *(const uint4 *)(v + o);
    }
    kf[kk] = as_bf8(a);
    vf[kk] = as_bf8(b);
  }
  const float sc = 1.4426950408889634f / sqrtf((float)HD), rs = 1.0f / sqrtf((float)HD);
  // MFMA row j reads tile row swap23(j): register r = 8*mm + e then holds query 16*mm + 8*g + e
  const uint32_t fk = T::frag_k_lane(swap23(j), g);
  const typename T::FragT ft = T::frag_t_init(lane);
  f32x16_t dka[NOT], dva[NOT];
#pragma unroll
  for (int t = 0; t < NOT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dka[t][r] = 0.f; dva[t][r] = 0.f; }

  for (int it = team; it - team < niter; it += QS) {      // (every team takes as many turns)
    wait_vmcnt<0>();
    __syncthreads();                                 // tile it has landed; the other stage is free
    if (QS > 1 && it >= niter) continue;
    if (it + QS < niter) issue_tile(it + QS);
    const int qb = k0 + (it % nqt) * TB;
    if (qb + TB - 1 < kw0) continue;                 // every query of the tile precedes this wave's keys
    if (kw0 >= xlo && kw0 + 32 <= xhi && qb >= xhi) continue;   // ... or none of them may see these keys
    const bf16_t *const stage = lds + (it / QS & 1) * STAGE;
    const uint32_t Qs = T::lds_addr(stage), Os = Qs + T::ELEMS * 2;
    const float *lse_s = (const float *)(stage + 2 * T::ELEMS), *d_s = lse_s + TB;
    static_for<0, 2>([&](auto ST) __attribute__((always_inline)) {
      constexpr int st = decltype(ST)::value, off = st * 32 * HD * 2;
      // P = exp(S - lse), then dV before dP: S and P's operand form are gone when the registers of dP are needed
      f32x16_t sa;
#pragma unroll
      for (int r = 0; r < 16; ++r) sa[r] = 0.f;
      static_for<0, NKK / RK>([&](auto KH) __attribute__((always_inline)) {
        constexpr int kk0 = RK * decltype(KH)::value;
        bf16x8_t a[RK];
        T::template read_k<RK, kk0, off>(Qs, fk, a);
#pragma unroll
        for (int i = 0; i < RK; ++i) sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], kf[kk0 + i], sa, 0, 0, 0);
      });
      float pv[16];
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        const int qo = st * 32 + 16 * mm + 8 * g;    // first of the 8 queries in registers 8*mm .. 8*mm+7
        const float4 la = *(const float4 *)(lse_s + qo), lb = *(const float4 *)(lse_s + qo + 4);
        const float ll[8] = {la.x, la.y, la.z, la.w, lb.x, lb.y, lb.z, lb.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[8 * mm + e] = __builtin_amdgcn_exp2f(fmaf(sa[8 * mm + e], sc, -1.4426950408889634f * ll[e]));
      }
      // queries that do not see this lane's key: before it, past the sequence, behind the excluded rectangle.  (The
      // query of register r minus that of this lane's first register is a constant.)
      if (qb < kw0 + 31 || qb + TB > L || kw0 + 32 > L) {
        const int first = ki < L ? ki - qb - 8 * g : TB, n_q = L - qb - 8 * g;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int c = st * 32 + 16 * (r >> 3) + (r & 7);
          pv[r] = ((c < first) | (c >= n_q)) ? 0.f : pv[r];
        }
      }
      if (kw0 + 31 >= xlo && kw0 < xhi && qb + TB > xhi) {
        const int hi = ki >= xlo && ki < xhi ? xhi - qb - 8 * g : 2 * TB;
#pragma unroll
        for (int r = 0; r < 16; ++r) pv[r] = st * 32 + 16 * (r >> 3) + (r & 7) >= hi ? 0.f : pv[r];
      }
      {
        const bf16x8_t pf[2] = {pack8(pv), pack8(pv + 8)};
#pragma unroll
        for (int t = 0; t < NOT; ++t) {
          bf16x8_t a[2];
          T::template read_t<2, 2 * st>(Os, ft, t, a);
#pragma unroll
          for (int mm = 0; mm < 2; ++mm) dva[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mm], pf[mm], dva[t], 0, 0, 0);
        }
      }
      f32x16_t dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[r] = 0.f;
      static_for<0, NKK / RK>([&](auto KH) __attribute__((always_inline)) {
        constexpr int kk0 = RK * decltype(KH)::value;
        bf16x8_t b[RK];
        T::template read_k<RK, kk0, off>(Os, fk, b);
#pragma unroll
        for (int i = 0; i < RK; ++i) dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[i], vf[kk0 + i], dp, 0, 0, 0);
      });
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        const int qo = st * 32 + 16 * mm + 8 * g;
        const float4 da = *(const float4 *)(d_s + qo), db = *(const float4 *)(d_s + qo + 4);
        const float dd[8] = {da.x, da.y, da.z, da.w, db.x, db.y, db.z, db.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) pv[8 * mm + e] *= (dp[8 * mm + e] - dd[e]) * rs;
      }
      const bf16x8_t dsf[2] = {pack8(pv), pack8(pv + 8)};
#pragma unroll
      for (int t = 0; t < NOT; ++t) {
        bf16x8_t b[2];
        T::template read_t<2, 2 * st>(Qs, ft, t, b);
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) dka[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[mm], dsf[mm], dka[t], 0, 0, 0);
      }
    });
  }
  if constexpr (QS > 1) {
    static_assert(QS == 2, "one or two teams");
    float *const sum = (float *)smem_raw;            // [2 NOT * 16][256], in the place of the stages
    static_assert(2 * NOT * 16 * 256 * 4 <= QS * 2 * STAGE * 2, "the sums of a team fit the stages");
    __syncthreads();
    if (team == 1) {
#pragma unroll
      for (int t = 0; t < NOT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sum[((2 * t) * 16 + r) * 256 + tid] = dka[t][r];
          sum[((2 * t + 1) * 16 + r) * 256 + tid] = dva[t][r];
        }
    }
    __syncthreads();
    if (team == 1) return;
#pragma unroll
    for (int t = 0; t < NOT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        dka[t][r] += sum[((2 * t) * 16 + r) * 256 + tid];
        dva[t][r] += sum[((2 * t + 1) * 16 + r) * 256 + tid];
      }
  }
  if (ki < L) {
    bf16_t *row = dqkv + (size_t)(r0 + ki) * (qld + 2 * kld) + qld + (size_t)kvh * HD;     // dk of this kv head; dv sits kld further
    store_grad_row<HD>(dka, cs + (size_t)(r0 + ki) * (HD / 2), g, row);
    store_grad_row<HD>(dva, nullptr, g, row + kld);
  }
}

// Two teams where one wave a SIMD would be left (a block's turns are a chain: load, products, soft-max, products), i.e. up to about one block a CU: a block of two teams has a CU's
// waves to itself, so one past that waits for a whole other one.  The blocks are estimated from rows and sequences; light ones at the end of a sequence count half, for they fill in.  Not where
// the sequences alone are more blocks than CUs, and not with a single turn (query tiles times heads of the group), which leaves the second team nothing.
// us with one / two teams, 8 kv heads, 32 query heads of 64 unless it says otherwise: 8 sequences of 327 - 505 rows 90 / 58 (a step of one pair of that layer 936 -> 918); 24 of 134 35.6 / 27.8; 32 of 64 rows (256 blocks) 14.8 / 12.6,
// 36 (288) 16.5 / 21.5, 60 of 10 (480) 14.4 / 17.5; 8 query heads, 16 of 60 (one turn) 6.7 / 7.0, 8 of 396 (7 turns) 19.5 / 17.2.  Of 128-wide heads, the dQ kernel included: 10 sequences of 134 (12 turns) 91.8 / 82.2, of 100 (8) 61.7 / 57.9;
// about even to a tenth dearer where a second round of light blocks meets few turns (8 query heads, 8 and 10 of 400, 256 and 320 blocks, 64.6 / 64.9 and 68.6 / 78.0; a step of a 7B layer with 2 sequences of 396 2088 / 2098, of 520 2558 / 2564).
// Those keep two teams: a finer line would give a step at most what its runs differ by.  At 384 blocks of 128-wide heads every SIMD has its second wave already.
bool two_teams(int n_seq, int max_len, int rows, int group, int Hkv) {
  return (long long)Hkv * (rows / 128 + n_seq / 2) <= 320 && (long long)Hkv * n_seq <= 256 && group * cdiv(max_len, TB) >= 2;
}

template <int HD>
hipError_t launch_t(const bf16_t *q, const bf16_t *k, const bf16_t *v, const bf16_t *o, const bf16_t *d_o,
                    const float *lse, const int32_t *seg, int row_base, int n_seq, int max_len, int rows, int Hq,
                    int Hkv, float *dvec, const float2 *cs, bf16_t *dqkv, hipStream_t st, const int32_t *excl_lo,
                    const int32_t *excl_hi) {
  constexpr size_t lds_q = (size_t)2 * (2 * TB * HD) * sizeof(bf16_t);
  constexpr size_t lds_k = (size_t)2 * (2 * TB * HD + 4 * TB) * sizeof(bf16_t);
  static DeviceOnce attr_done;
  if (!attr_done.test()) {
    hipError_t e = hipFuncSetAttribute((const void *)attn_bwd_dq_kernel<HD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_q);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void *)attn_bwd_dkdv_kernel<HD, 1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_k);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void *)attn_bwd_dkdv_kernel<HD, 2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(2 * lds_k));
    if (e != hipSuccess) return e;
    attr_done.set();
  }
  dim3 grid_q(Hq, n_seq, cdiv(max_len, 128)), grid_k(Hkv, n_seq, cdiv(max_len, 128));
  hipLaunchKernelGGL((attn_bwd_dq_kernel<HD>), grid_q, dim3(256), lds_q, st, q, k, v, o, d_o, lse, dvec, seg, row_base, Hq, Hkv, cs, dqkv, excl_lo, excl_hi);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (two_teams(n_seq, max_len, rows, Hq / Hkv, Hkv))
    hipLaunchKernelGGL((attn_bwd_dkdv_kernel<HD, 2>), grid_k, dim3(512), 2 * lds_k, st, q, k, v, d_o, lse, dvec, seg, row_base, Hq, Hkv, cs, dqkv, excl_lo, excl_hi);
  else
    hipLaunchKernelGGL((attn_bwd_dkdv_kernel<HD, 1>), grid_k, dim3(256), lds_k, st, q, k, v, d_o, lse, dvec, seg, row_base, Hq, Hkv, cs, dqkv, excl_lo, excl_hi);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bwd(const bf16_t *q, const bf16_t *k, const bf16_t *v, const bf16_t *o, const bf16_t *d_o,
                           const float *lse, const int32_t *seg, int row_base, int n_seq, int max_len, int rows,
                           int Hq, int Hkv, int hd, float *dvec, const float2 *cs, bf16_t *dqkv, hipStream_t st,
                           const int32_t *excl_lo, const int32_t *excl_hi) {
  if (n_seq <= 0 || rows <= 0) return hipSuccess;
  if (n_seq > 65535 || max_len > 65535 * 64 || ((excl_lo == nullptr) != (excl_hi == nullptr))) return hipErrorInvalidValue;
  if (hd == 64) return launch_t<64>(q, k, v, o, d_o, lse, seg, row_base, n_seq, max_len, rows, Hq, Hkv, dvec, cs, dqkv, st, excl_lo, excl_hi);
  if (hd == 128) return launch_t<128>(q, k, v, o, d_o, lse, seg, row_base, n_seq, max_len, rows, Hq, Hkv, dvec, cs, dqkv, st, excl_lo, excl_hi);
  return hipErrorInvalidValue;
}
