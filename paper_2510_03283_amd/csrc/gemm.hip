// bf16 MFMA GEMM for gfx950: 32x32x16 MFMA tiles, direct global->LDS operand loads, LDS double
// buffer of 64-wide k tiles.
//
// Tiles sit in LDS in the layout they have in memory: a k-contiguous operand as [row][k], a
// row-contiguous operand as [k][row].  MFMA fragments (8 consecutive k of one row per lane) come
// from one 16-byte LDS read in the first case and from two transposing 8-byte LDS reads
// (ds_read_b64_tr_b16) in the second, so the NN and TN forms need no transposed copies in HBM
// and no in-register shuffles.
#include "gemm.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <utility>
#include <vector>

namespace {

constexpr int BK = 64;          // k extent of an LDS tile
constexpr int NSTAGES = 2;

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;   // per-lane byte offsets of up to four tile loads

constexpr int GROUP_M = 8;         // m tiles per swizzle group (L2 reuse of the B tiles)
constexpr int GROUP_M_MULTI = 4;   // the same for row groups with two-term operands (twice the A bytes per m tile)

// Operand tiles go global -> LDS directly (global_load_lds_dwordx4): no staging registers and no
// LDS store instructions.  A wave-wide load writes 64 consecutive 16-byte chunks, so LDS tiles
// are unpadded; bank conflicts are avoided by an XOR swizzle that is applied through the choice
// of the global address each lane fetches.
__device__ __align__(16) uint4 g_zero16 = {0u, 0u, 0u, 0u};   // source of out-of-range chunks

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void gbl_void_t;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {   // vmcnt <= N, no wait on the other counters
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

template <int ROWS, int LAYOUT, int BKT, int NTHR>
struct DirectStage {
  static constexpr int ELEMS = ROWS * BKT;
  static constexpr int NCH = ROWS * BKT / 8;             // 16-byte chunks
  static constexpr int NI = NCH / NTHR;                  // wave-wide loads per wave
  static_assert(NCH % NTHR == 0 && NI <= 4, "tile must split evenly over the waves, at most four loads per lane");
  static constexpr int CPR = LAYOUT == 0 ? BKT / 8 : ROWS / 8;   // chunks per LDS row
  static constexpr int RPB = LAYOUT == 0 ? 16 / CPR : 1;         // LDS rows per 256 bytes (LAYOUT 0)

  // LAYOUT 0: LDS [row][BKT], chunk position pos holds logical k-chunk pos ^ ((row / RPB) % CPR)
  // LAYOUT 1: LDS [k][ROWS],  logical row-chunk c sits at position c ^ ((k & 3) << 2) when CPR is a
  //           power of two, else at (c + 4 * (k & 3)) % CPR (same bank spread, any CPR % 4 == 0).  Of eight chunks, rows of 128
  //           bytes, every other row is half the banks further on by itself, and c ^ ((k & 2) << 1) spreads four of them.
  static constexpr bool POW2 = (CPR & (CPR - 1)) == 0;
  static __device__ __forceinline__ int swz(int k) { return CPR == 8 ? (k & 2) << 1 : (k & 3) << 2; }
  static_assert(LAYOUT == 0 || CPR % 4 == 0, "row-contiguous tiles need a multiple of 32 rows");
  static_assert(LAYOUT == 0 || !POW2 || CPR >= 8, "the swizzle stays inside a row");
  static __device__ __forceinline__ void issue(const bf16_t *base, long long ld, int row0, int rows, int k0, int K, bf16_t *S) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave + (NTHR / 64) * i;
      const int chunk = q * 64 + lane;
      const int lr = chunk / CPR, pos = chunk % CPR;
      const bf16_t *src;
      bool ok;
      if constexpr (LAYOUT == 0) {
        const int kc = pos ^ ((lr / RPB) % CPR);
        const int gr = row0 + lr;
        ok = gr < rows;
        src = base + (long long)gr * ld + k0 + kc * 8;
      } else {
        const int c = POW2 ? pos ^ swz(lr) : (pos + CPR - 4 * (lr & 3)) % CPR;
        const int k = k0 + lr, gr = row0 + 8 * c;
        ok = k < K && gr < rows;
        src = base + (long long)k * ld + gr;
      }
      if (!ok) src = (const bf16_t *)&g_zero16;
      __builtin_amdgcn_global_load_lds((gbl_void_t *)src, (lds_void_t *)(S + q * 512), 16, 0, 0);
    }
  }
  // SwiGLU mode (LAYOUT 0): LDS rows [64 w, 64 w + 32) hold gate rows f0 + 32 w .. and rows
  // [64 w + 32, 64 w + 64) the up rows of the same hidden units, so that the two 32-column MFMA
  // tiles of wave column w are G and U of one unit range.
  static __device__ __forceinline__ void issue_gu(const bf16_t *bg, const bf16_t *bu, long long ld, int f0, int F, int k0, bf16_t *S) {
    static_assert(LAYOUT == 0, "gate/up interleaving is defined for k-contiguous weights");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave + (NTHR / 64) * i;
      const int chunk = q * 64 + lane;
      const int lr = chunk / CPR, pos = chunk % CPR;
      const int kc = pos ^ ((lr / RPB) % CPR);
      const int f = f0 + (lr >> 6) * 32 + (lr & 31);
      const bf16_t *src = ((lr >> 5) & 1 ? bu : bg) + (long long)f * ld + k0 + kc * 8;
      if (f >= F) src = (const bf16_t *)&g_zero16;
      __builtin_amdgcn_global_load_lds((gbl_void_t *)src, (lds_void_t *)(S + q * 512), 16, 0, 0);
    }
  }
  // Fast path of the main loop: every lane keeps one 32-bit byte offset per load, relative to a tile
  // origin that is uniform over the block, so a k step costs scalar pointer arithmetic only and the
  // loads take the (scalar base + lane offset) form.  Rows past the matrix edge are clamped onto the
  // last valid row (8-row chunk): they only feed accumulator rows / columns that are never stored.
  // Tiles that cross the end of the k range go through issue() instead (zero fill).
  static __device__ __forceinline__ u32x4_t lane_offsets(long long ld, int row0, int rows, int wave) {
    const int lane = threadIdx.x & 63;
    u32x4_t off = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int chunk = (wave + (NTHR / 64) * i) * 64 + lane;
      const int lr = chunk / CPR, pos = chunk % CPR;
      if constexpr (LAYOUT == 0) {
        const int kc = pos ^ ((lr / RPB) % CPR);
        off[i] = (uint32_t)(((long long)min(lr, rows - 1 - row0) * ld + kc * 8) * 2);
      } else {
        const int c = POW2 ? pos ^ swz(lr) : (pos + CPR - 4 * (lr & 3)) % CPR;
        off[i] = (uint32_t)(((long long)lr * ld + min(8 * c, rows - 8 - row0)) * 2);
      }
    }
    return off;
  }
  static __device__ __forceinline__ u32x4_t lane_offsets_gu(long long ld, int f0, int F, int wave) {
    const int lane = threadIdx.x & 63;
    u32x4_t off = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int chunk = (wave + (NTHR / 64) * i) * 64 + lane;
      const int lr = chunk / CPR, pos = chunk % CPR;
      const int kc = pos ^ ((lr / RPB) % CPR);
      const int fr = (lr >> 6) * 32 + (lr & 31);
      off[i] = (uint32_t)(((long long)min(fr, F - 1 - f0) * ld + kc * 8) * 2);
    }
    return off;
  }
  static __device__ __forceinline__ void issue_fast(const char *origin, const u32x4_t off, int wave, bf16_t *S) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave + (NTHR / 64) * i;
      __builtin_amdgcn_global_load_lds((gbl_void_t *)(origin + off[i]), (lds_void_t *)(S + q * 512), 16, 0, 0);
    }
  }
  // SwiGLU mode: a wave-wide load covers 8 LDS rows, so it reads gate rows or up rows, never both
  static __device__ __forceinline__ void issue_fast_gu(const char *origin_g, const char *origin_u, const u32x4_t off, int wave, bf16_t *S) {
    static_assert(LAYOUT == 0 && CPR == 8, "gate/up interleaving is defined for k-contiguous 64-wide tiles");
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave + (NTHR / 64) * i;
      const char *origin = (q >> 2) & 1 ? origin_u : origin_g;
      __builtin_amdgcn_global_load_lds((gbl_void_t *)(origin + off[i]), (lds_void_t *)(S + q * 512), 16, 0, 0);
    }
  }
  // MFMA fragments (8 consecutive k of one row per lane).  The LDS reads are issued as asm and the
  // kernel counts them itself (s_waitcnt lgkmcnt(n) before the MFMAs that need them): while a direct
  // global->LDS load is in flight the compiler's own wait insertion turns every wait for an LDS
  // read into a wait for ALL outstanding LDS reads, which serialises fragment reads and MFMAs.
  // A read's result must not be touched before that wait; cook() turns it into the MFMA operand.
  static constexpr int RPF = LAYOUT == 0 ? 1 : 2;          // LDS read instructions per fragment
  struct Raw { u32x4_t q; u32x2_t lo, hi; };                // q: k-contiguous tile; lo, hi: transposing reads
  // per-lane byte offsets inside a tile: LAYOUT 0: v[kk] for the lane's first fragment at k step kk
  // (the swizzle depends on kk; fragment i sits i * 32 rows further); LAYOUT 1: v[i] for fragment i
  // at k step 0 (k step kk sits 16 kk rows further)
  struct FragAddr { uint32_t v[4]; };
  template <int NF>
  static __device__ __forceinline__ FragAddr frag_addr(int r0, int lane) {
    static_assert(NF <= 4 && BKT / 16 <= 4, "at most four fragments per wave and four k steps per tile");
    FragAddr f;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      if constexpr (LAYOUT == 0) {
        const int row = r0 + (lane & 31);
        const int c = (2 * x + (lane >> 5)) ^ ((row / RPB) % CPR);
        f.v[x] = (uint32_t)((row * BKT + c * 8) * 2);
      } else {
        const int grp = lane >> 4, j = lane & 15;
        const int cl = ((r0 + 32 * x) >> 3) + 2 * (grp & 1) + ((j & 3) >> 1);
        const int chunk = POW2 ? cl ^ swz(j >> 2) : (cl + 4 * (j >> 2)) % CPR;
        f.v[x] = x < NF ? (uint32_t)(((8 * (grp >> 1) + (j >> 2)) * ROWS + chunk * 8 + 4 * (j & 1)) * 2) : 0u;
      }
    }
    return f;
  }
  // tile: LDS byte address of the tile; kk, i: compile-time constants at every call site
  static __device__ __forceinline__ Raw read(uint32_t tile, const FragAddr &f, int kk, int i) {
    Raw r;
    if constexpr (LAYOUT == 0) {
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r.q) : "v"(tile + f.v[kk]), "i"(i * 32 * BKT * 2));
    } else {
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.lo) : "v"(tile + f.v[i]), "i"(kk * 16 * ROWS * 2));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.hi) : "v"(tile + f.v[i]), "i"(kk * 16 * ROWS * 2 + 4 * ROWS * 2));
    }
    return r;
  }
  static __device__ __forceinline__ bf16x8_t cook(const Raw &r) {
    if constexpr (LAYOUT == 0) {
      return __builtin_bit_cast(bf16x8_t, r.q);
    } else {
      const u32x4_t v = {r.lo[0], r.lo[1], r.hi[0], r.hi[1]};
      return __builtin_bit_cast(bf16x8_t, v);
    }
  }
};

template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {   // lgkmcnt <= N, no wait on the other counters
  static_assert(N >= 0 && N <= 15, "4-bit counter");
  __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (N << 8) | (3 << 14));
}

template <int BM, int BN, int WGM, int WGN, int LA, int LB, int BKT, int NST>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_dl_kernel(const GemmParams p) {
  constexpr int NTHR = 64 * WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int NKK = BKT / 16;
  constexpr int P = NST - 1;                      // tiles in flight ahead of the one being multiplied
  using SA = DirectStage<BM, LA, BKT, NTHR>;
  using SB = DirectStage<BN, LB, BKT, NTHR>;
  constexpr int STAGE = SA::ELEMS + SB::ELEMS;
  constexpr int LPT = SA::NI + SB::NI;            // loads per thread per tile
  extern __shared__ __align__(16) unsigned char smem_raw[];
  bf16_t *lds = (bf16_t *)smem_raw;

  // Block -> tile.  Row groups are laid out one after the other in block-id order (the launcher
  // sorts the multi-pass groups first, so the long tiles start first).  Inside a group, the blocks
  // that land on XCD x (block id % 8) take a contiguous chunk of the group's tile list, ordered in
  // bands of GROUP_M (GROUP_M_MULTI) m-tiles, so the tiles resident on one XCD share A and B panels in its L2 and
  // every XCD gets the same mix of long and short tiles.
  const int n_ns_eff = p.swiglu ? 1 : p.n_ns;      // SwiGLU mode: one logical column range of F hidden units
  const int total_nt = p.nt_start[n_ns_eff];
  int g = 0, first_blk = 0;
  while (g + 1 < p.n_mg && (int)blockIdx.x >= first_blk + (p.mt_start[g + 1] - p.mt_start[g]) * total_nt) {
    first_blk += (p.mt_start[g + 1] - p.mt_start[g]) * total_nt;
    ++g;
  }
  const int mtc = p.mt_start[g + 1] - p.mt_start[g], T = mtc * total_nt;
  int v = 0;
  {
    const int x = blockIdx.x & 7;
    for (int y = 0; y < x; ++y) {
      const int fy = (y - first_blk) & 7;            // first block of the group on XCD y (group-local id)
      v += fy < T ? (T - 1 - fy) / 8 + 1 : 0;
    }
    v += ((int)blockIdx.x - first_blk - ((x - first_blk) & 7)) >> 3;
  }
  const int band = p.mg[g].npass >= 2 ? GROUP_M_MULTI : GROUP_M;
  const int grp_sz = band * total_nt;
  const int first_m = (v / grp_sz) * band;
  const int gm = min(mtc - first_m, band);
  const int mt_l = first_m + (v % grp_sz) % gm, nt_g = (v % grp_sz) / gm;
  int s = 0;
  while (s + 1 < n_ns_eff && nt_g >= p.nt_start[s + 1]) ++s;
  const GemmMGroup &G = p.mg[g];
  const GemmNSeg &S = p.ns[s];
  const int m0 = mt_l * BM, n0 = p.swiglu ? nt_g * (BN / 2) : (nt_g - p.nt_start[s]) * BN;
  const int M = G.M, N = S.N, K = p.K;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = (K + BKT - 1) / BKT, n_it = nk * G.npass;
  // operand bases of this block's row group / column segment (scalar registers), and every lane's
  // byte offsets inside a tile
  const char *const a_hi = (const char *)G.a[0], *const a_lo = (const char *)G.a[1];
  const char *const b_hi = (const char *)(p.swiglu ? p.ns[0].b[0] : S.b[0]), *const b_lo = (const char *)(p.swiglu ? p.ns[0].b[1] : S.b[1]);
  const char *const u_hi = (const char *)p.ns[1].b[0], *const u_lo = (const char *)p.ns[1].b[1];      // SwiGLU mode: up weights
  const char *const ks_b0 = (const char *)p.kseg_b[0], *const ks_b1 = (const char *)p.kseg_b[1], *const ks_b2 = (const char *)p.kseg_b[2];
  const int ks_s1 = p.kseg_start[1], ks_s2 = p.kseg_start[2];
  const int n_kseg = p.n_kseg, swiglu = p.swiglu;
  const long long lda = p.lda, ldb = p.ldb;
  const u32x4_t offA = SA::lane_offsets(lda, m0, M, wave);
  u32x4_t offB;
  if constexpr (LB == 0) offB = swiglu ? SB::lane_offsets_gu(ldb, n0, N, wave) : SB::lane_offsets(ldb, n0, N, wave);
  else offB = SB::lane_offsets(ldb, n0, N, wave);
  const typename SA::FragAddr fa = SA::template frag_addr<TM>(wm * WTM, lane);
  const typename SB::FragAddr fb = SB::template frag_addr<TN>(wn * WTN, lane);
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_t *)lds;      // LDS byte address of stage 0
  constexpr int RPS = TM * SA::RPF + TN * SB::RPF;                       // LDS read instructions per k step
  static_assert(RPS <= 15, "the reads of one k step must fit the 4-bit LDS counter");

  // One loop requests and multiplies: iteration `it` first waits for tile `it`, then requests tile
  // it + P into the stage that tile it - 1 has just left, then multiplies tile `it`.  The first P
  // iterations (it < 0) only request.  (The request code appears once, in line: as a lambda called
  // from two places its captured bases end up in private memory.)
  int st_cur = 0, st_req = 0;
  for (int it = -P; it < n_it; ++it) {
    if (it >= 0) {
      // tile `it` has landed once at most the loads of the P-1 younger tiles are outstanding
      if (it + P - 1 < n_it) wait_vmcnt<(P - 1) * LPT>();
      else wait_vmcnt<0>();
      __syncthreads();   // tile it visible to every wave; every wave is done with the stage of tile it-1
    }
    if (it + P < n_it) {
      const int t = it + P;
      const int pass = t >= 2 * nk ? 2 : (t >= nk ? 1 : 0);
      const int k0 = (t - pass * nk) * BKT;
      bf16_t *st = lds + st_req * STAGE;
      st_req = st_req == NST - 1 ? 0 : st_req + 1;
      if ((LA == 1 || LB == 1) && k0 + BKT > K) {
        // the tile crosses the end of the k range: per-lane bounds checks and zero fill
        SA::issue((const bf16_t *)(pass == 1 ? a_lo : a_hi), lda, m0, M, k0, K, st);
        if (n_kseg > 1) {
          const int ks = (k0 >= ks_s1 ? 1 : 0) + (n_kseg > 2 && k0 >= ks_s2 ? 1 : 0);
          const int s0 = ks == 0 ? 0 : (ks == 1 ? ks_s1 : ks_s2), s1 = ks + 1 == n_kseg ? K : (ks == 0 ? ks_s1 : ks_s2);
          SB::issue((const bf16_t *)(ks == 0 ? ks_b0 : (ks == 1 ? ks_b1 : ks_b2)), ldb, n0, N, k0 - s0, s1 - s0, st + SA::ELEMS);
        } else {
          SB::issue((const bf16_t *)(pass == 2 ? b_lo : b_hi), ldb, n0, N, k0, K, st + SA::ELEMS);
        }
      } else {
        const char *ao = (pass == 1 ? a_lo : a_hi) + (LA == 0 ? (long long)m0 * lda + k0 : (long long)k0 * lda + m0) * 2;
        SA::issue_fast(ao, offA, wave, st);
        if (n_kseg > 1) {
          const int ks = (k0 >= ks_s1 ? 1 : 0) + (n_kseg > 2 && k0 >= ks_s2 ? 1 : 0);
          const int kl = k0 - (ks == 0 ? 0 : (ks == 1 ? ks_s1 : ks_s2));
          const char *bo = (ks == 0 ? ks_b0 : (ks == 1 ? ks_b1 : ks_b2)) + (LB == 0 ? (long long)n0 * ldb + kl : (long long)kl * ldb + n0) * 2;
          SB::issue_fast(bo, offB, wave, st + SA::ELEMS);
        } else if (swiglu) {
          if constexpr (LB == 0) {
            const long long o = ((long long)n0 * ldb + k0) * 2;
            SB::issue_fast_gu((pass == 2 ? b_lo : b_hi) + o, (pass == 2 ? u_lo : u_hi) + o, offB, wave, st + SA::ELEMS);
          }
        } else {
          const char *bo = (pass == 2 ? b_lo : b_hi) + (LB == 0 ? (long long)n0 * ldb + k0 : (long long)k0 * ldb + n0) * 2;
          SB::issue_fast(bo, offB, wave, st + SA::ELEMS);
        }
      }
    }
    if (it < 0) continue;
    const uint32_t Ac = lds_addr + st_cur * (STAGE * 2), Bc = Ac + SA::ELEMS * 2;
    typename SA::Raw ra[2][TM];
    typename SB::Raw rb[2][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) ra[0][i] = SA::read(Ac, fa, 0, i);
#pragma unroll
    for (int j = 0; j < TN; ++j) rb[0][j] = SB::read(Bc, fb, 0, j);
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      if (kk + 1 < NKK) {
#pragma unroll
        for (int i = 0; i < TM; ++i) ra[(kk + 1) & 1][i] = SA::read(Ac, fa, kk + 1, i);
#pragma unroll
        for (int j = 0; j < TN; ++j) rb[(kk + 1) & 1][j] = SB::read(Bc, fb, kk + 1, j);
        wait_lgkmcnt<RPS>();          // the fragments of step kk are in; those of step kk + 1 may be in flight
      } else {
        wait_lgkmcnt<0>();
      }
      __builtin_amdgcn_sched_barrier(0);
      bf16x8_t af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) af[i] = SA::cook(ra[kk & 1][i]);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[j] = SB::cook(rb[kk & 1][j]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    st_cur = st_cur == NST - 1 ? 0 : st_cur + 1;
  }

  // epilogue: accumulator register r of a 32x32 tile holds row 8*(r/4) + 4*(lane/32) + r%4, column lane%32.
  // bf16 outputs are stored as packed pairs: neighbouring lanes (columns f, f+1) swap one value of
  // a register pair (rows row, row+1), the even lane then stores columns (f, f+1) of row and the
  // odd lane columns (f-1, f) of row+1 - one 4-byte store per lane instead of two 2-byte ones.
  const int rk = p.resid_kind, obf = p.out_bf16;
  const long long ldc = p.ldc, ldr = p.ldr;
  const bool odd = lane & 1;
  auto swap_pair = [&](float mine_r, float mine_r1) -> float {     // returns the partner's value for the row this lane stores
    const float send = odd ? mine_r : mine_r1;
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), 0xB1, 0xF, 0xF, true));
  };
  if (p.swiglu) {
    if constexpr (TN == 2 && LB == 0) {
      const int f = n0 + wn * 32 + (lane & 31);
      const int F = N;
      bf16_t *hi = (bf16_t *)G.c, *lo = (bf16_t *)G.c_lo, *gu = (bf16_t *)G.c_gu;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int rbase = m0 + wm * WTM + i * 32 + 4 * (lane >> 5);
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const int row0 = rbase + 8 * (r >> 2) + (r & 3);
          float g2[2] = {acc[i][0][r], acc[i][0][r + 1]}, u2[2] = {acc[i][1][r], acc[i][1][r + 1]}, h2[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) h2[e] = g2[e] / (1.0f + expf(-g2[e])) * u2[e];
          const float hp = swap_pair(h2[0], h2[1]), gp = swap_pair(g2[0], g2[1]), up = swap_pair(u2[0], u2[1]);
          const int row = row0 + (odd ? 1 : 0), fc = f - (odd ? 1 : 0);          // this lane stores (row, fc .. fc+1)
          if (row < M && fc < F) {
            const float ha = odd ? hp : h2[0], hb = odd ? h2[1] : hp;
            uint32_t ph, pl;
            split_pk_bf16(ha, hb, ph, pl);
            *(uint32_t *)(hi + (long long)row * ldc + fc) = ph;
            if (lo) *(uint32_t *)(lo + (long long)row * ldc + fc) = pl;
            if (gu) {
              *(uint32_t *)(gu + (long long)row * 2 * F + fc) = cvt_pk_bf16(odd ? gp : g2[0], odd ? g2[1] : gp);
              *(uint32_t *)(gu + (long long)row * 2 * F + F + fc) = cvt_pk_bf16(odd ? up : u2[0], odd ? u2[1] : up);
            }
          }
        }
      }
    }
    return;
  }
  if (obf && !(N & 1) && !(S.c_col & 1)) {
    // packed bf16 path (every lane takes part in the swap, also those beyond the matrix edge)
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + wn * WTN + j * 32 + (lane & 31);
        const int rbase = m0 + wm * WTM + i * 32 + 4 * (lane >> 5);
        const long long cc = S.c_col + col;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
          const int row0 = rbase + 8 * (r >> 2) + (r & 3);
          float va = acc[i][j][r], vb = acc[i][j][r + 1];
          if (rk && col < N) {
            if (row0 < M) va += rk == 1 ? ((const float *)G.resid)[row0 * ldr + cc] : bf2f(((const bf16_t *)G.resid)[row0 * ldr + cc]);
            if (row0 + 1 < M) vb += rk == 1 ? ((const float *)G.resid)[(row0 + 1) * ldr + cc] : bf2f(((const bf16_t *)G.resid)[(row0 + 1) * ldr + cc]);
          }
          const float vp = swap_pair(va, vb);
          const int row = row0 + (odd ? 1 : 0);
          if (row < M && col - (odd ? 1 : 0) < N)
            *(uint32_t *)((bf16_t *)G.c + row * ldc + cc - (odd ? 1 : 0)) = cvt_pk_bf16(odd ? vp : va, odd ? vb : vp);
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + wn * WTN + j * 32 + (lane & 31);
      const int rbase = m0 + wm * WTM + i * 32 + 4 * (lane >> 5);
      if (col >= N) continue;
      const long long cc = S.c_col + col;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = rbase + 8 * (r >> 2) + (r & 3);
        if (row < M) {
          float v = acc[i][j][r];
          if (rk == 1) v += ((const float *)G.resid)[row * ldr + cc];
          else if (rk == 2) v += bf2f(((const bf16_t *)G.resid)[row * ldr + cc]);
          if (obf) ((bf16_t *)G.c)[row * ldc + cc] = f2bf(v);
          else ((float *)G.c)[row * ldc + cc] = v;
        }
      }
    }
  }
}

template <int BM, int BN>
int count_tiles(GemmParams &p) {
  int mt = 0, nt = 0;
  for (int g = 0; g < p.n_mg; ++g) { p.mt_start[g] = mt; mt += cdiv(p.mg[g].M, BM); }
  p.mt_start[p.n_mg] = mt;
  if (p.swiglu) {
    p.nt_start[0] = 0;
    nt = cdiv(p.ns[0].N, BN / 2);
    p.nt_start[1] = nt;
    return mt * nt;
  }
  for (int s = 0; s < p.n_ns; ++s) { p.nt_start[s] = nt; nt += cdiv(p.ns[s].N, BN); }
  p.nt_start[p.n_ns] = nt;
  return mt * nt;
}

#include "gemm_w4.h"

template <int BM, int BN, int WGM, int WGN, int LA, int LB, int BKT, int NST>
hipError_t launch_dl(GemmParams &p, hipStream_t stream) {
  const int tiles = count_tiles<BM, BN>(p);
  if (tiles == 0) return hipSuccess;
  constexpr int NTHR = 64 * WGM * WGN;
  constexpr size_t lds = (size_t)NST * (BM + BN) * BKT * sizeof(bf16_t);
  static_assert(lds <= 160 * 1024, "LDS budget of a gfx950 CU");
  static DeviceOnce attr_done;
  if (!attr_done.test()) {
    hipError_t e = hipFuncSetAttribute((const void *)gemm_bf16_dl_kernel<BM, BN, WGM, WGN, LA, LB, BKT, NST>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_done.set();
  }
  p.tile_m = BM; p.tile_n = BN;
  hipLaunchKernelGGL((gemm_bf16_dl_kernel<BM, BN, WGM, WGN, LA, LB, BKT, NST>), dim3((unsigned)tiles), dim3(NTHR), lds, stream, p);
  return hipGetLastError();
}

template <int LA, int LB, int TM>
hipError_t launch_w4_rows(GemmParams &p, hipStream_t stream) {
  const int tiles = count_tiles<32 * TM, 256>(p);
  if (tiles == 0) return hipSuccess;
  constexpr size_t lds = w4_lds_bytes<LA, LB>();
  static_assert(lds <= 160 * 1024, "LDS budget of a gfx950 CU");
  static DeviceOnce attr_done;
  if (!attr_done.test()) {
    hipError_t e = hipFuncSetAttribute((const void *)gemm_bf16_w4_kernel<LA, LB, TM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_done.set();
  }
  p.tile_m = 32 * TM; p.tile_n = 256;
  int blocks = 0;
  for (int g = 0; g < p.n_mg; ++g) {
    p.k_splits[g] = std::max(1, p.k_splits[g]);
    blocks += (p.mt_start[g + 1] - p.mt_start[g]) * (tiles / p.mt_start[p.n_mg]) * p.k_splits[g];
  }
  hipLaunchKernelGGL((gemm_bf16_w4_kernel<LA, LB, TM>), dim3((unsigned)blocks), dim3(256), lds, stream, p);
  return hipGetLastError();
}
// tile: as in choose_tile
template <int LA, int LB>
hipError_t launch_w4(GemmParams &p, int tile, hipStream_t stream) {
  if constexpr (LA == 0) {
    if (tile == 5) return launch_w4_rows<LA, LB, 7>(p, stream);
    if (tile == 2) return launch_w4_rows<LA, LB, 6>(p, stream);
  }
  return launch_w4_rows<LA, LB, 8>(p, stream);
}

bool aligned16(const void *q) { return ((uintptr_t)q & 15) == 0; }

// Tile choice.  256x256 tiles (four waves with 128x128 wave tiles, one block per CU) do half the LDS
// reads and half the L2 traffic of 128x128 tiles (4 waves, two blocks per CU), but quantise worse on
// small problems; tiles of 224 and 192 rows (four waves; 192x256 with 8 waves for the TN form and for what does not fit
// the four-wave kernel, bf16 output with a residual above all) sit between.  Each candidate is priced as
//   length of its schedule over the (CU x resident block) slots  x  tile area  /  relative efficiency,
// a tile of a row group with p passes taking p time units on its slot, and the cheapest is launched.  The
// efficiencies (0.69 for the eight-wave 192x256, 0.62 for 128x128, relative to the four-wave kernel) are fitted to whole steps
// of the benchmark configurations: step time was flat for factors between 0.68 and 0.8 of the kernels' long-run
// ratios (0.92, 0.83) and 1 - 6 % worse on either side.  (Fitted to the 32x32x16 loop of the four-wave kernel, which took 6 - 8 % longer
// on long reductions; kept, see product_us.)
//
// Tiles of 224 and 192 rows of the same kernel (k-contiguous A) take 0.90 and 0.80 of the time of one of 256 (0.875 and 0.75 of its products; its B tile in full).  us at 160, 256 and 512
// tiles, N = 4096, K = 4096, 256 / 224 / 192 rows: 83.7 / 74.9 / 65.4, 96.3 / 88.7 / 79.2, 192 / 171 / 155; two passes, 256 tiles: 169 / 156 / 138.  They pay where they leave less of the last m tile
// or of the last round empty.  CUs that stand idle leave the others their power: with few tiles a tile takes 0.77 of its time in a full round, so a round that is not full is priced by how full it is
// (among these three).  With the choice, us a pass: 3108 rows of a 7B layer (13 m tiles of 256,
// 14 of 224) 1659 -> 1592, a training step of an edge layer 2319 -> 2236, of a 7B layer beside 256 decode rows 6418 -> 6281.
constexpr double W4_224_TIME = 0.90, W4_192_TIME = 0.80, W4_IDLE_GAIN = 0.23;
template <int BM, int BN>
double tile_cost(const GemmParams &p, int slots, double slot_share, double eff, double idle_gain = 0.0) {
  int nt = 0;
  for (int s = 0; s < p.n_ns; ++s) nt += cdiv(p.ns[s].N, BN);
  // The dispatcher hands the next block to whichever slot is free, in block-id order (row groups one
  // after the other, multi-pass groups first).  Time in passes of one tile: free_at[t] slots fall free at t.
  double w = 0;
  for (int g = 0; g < p.n_mg; ++g) w += (double)cdiv(p.mg[g].M, BM) * nt * p.mg[g].npass;
  std::vector<int> free_at((size_t)(w / slots) + 8, 0);
  free_at[0] = slots;
  size_t t = 0, end = 0;
  long long last = 0;      // tiles that end last
  for (int g = 0; g < p.n_mg; ++g) {
    long long n = (long long)cdiv(p.mg[g].M, BM) * nt;
    const size_t c = (size_t)p.mg[g].npass;
    while (n > 0) {
      if (free_at[t] == 0) { ++t; continue; }
      const int k = (int)std::min<long long>(n, free_at[t]);
      free_at[t] -= k;
      free_at[t + c] += k;
      n -= k;
      last = t + c > end ? k : (t + c == end ? last + k : last);
      end = std::max(end, t + c);
    }
  }
  return ((double)end - idle_gain * (1.0 - (double)last / slots)) * BM * BN * slot_share / eff;
}

// The four-wave kernel has tiles of 224 and 192 rows for the product: k-contiguous A, and the product fits that kernel.
template <int LA, int LB>
bool w4_low(const GemmParams &p) { return LA == 0 && w4_fits<LA, LB>(p); }
int choose_tile(bool low, const GemmParams &p);
bool is_w4_tile(bool low, int tile);

bool has_rope(const GemmParams &p) {
  for (int g = 0; g < p.n_mg; ++g)
    if (p.mg[g].rope) return true;
  return false;
}

bool is_split(const GemmParams &p) {
  for (int g = 0; g < p.n_mg; ++g)
    if (p.k_splits[g] > 1) return true;
  return false;
}

template <int LA, int LB>
bool uses_w4(const GemmParams &p) {
  const bool low = w4_low<LA, LB>(p);
  return (p.force_w4 || is_w4_tile(low, choose_tile(low, p))) && w4_fits<LA, LB>(p);
}

// Length in microseconds of a schedule of equal blocks per row group on `slots` slots, in block-id order.
double makespan(int slots, int n_mg, const long long *n, const double *d) {
  struct Free { double t; long long k; };
  std::vector<Free> f{{0.0, slots}};                     // slots by the time they fall free, ascending
  double end = 0.0;
  for (int g = 0; g < n_mg; ++g) {
    long long left = n[g];
    while (left > 0) {
      const long long k = std::min(left, f.front().k);
      const double t = f.front().t + d[g];
      f.front().k -= k;
      if (f.front().k == 0) f.erase(f.begin());
      auto it = f.begin();
      while (it != f.end() && it->t < t) ++it;
      if (it != f.end() && it->t == t) it->k += k;
      else f.insert(it, {t, k});
      left -= k;
      end = std::max(end, t);
    }
  }
  return end;
}

// Estimated time of a product, microseconds.  A k tile takes a block of the four-wave kernel 1.07 us while most CUs are
// idle and 1.37 us when all are busy, a block of the 192x256 tile 1.45 us, of the 128x128 tile 0.68 us alone on its CU and
// 1.15 us beside a second one; starting and storing a tile adds 6 - 8 us.  Measured over 15 shapes from 128 x 4096 x
// 4096 to 3108 x 4096 x 11008, 2329 x 2048 x 2048 .. 5632, within 15 %, with the 32x32x16 loop of the four-wave kernel.  The present
// one takes 1.00 us a k tile at 12 - 64 blocks and 1.32 with all CUs busy, and 9.6 us a launch besides (256 x 3072 .. 16384, K = 512 and 1024).  Prices refitted to it changed 13 of 88
// choices, by at most 4 us and mostly for the worse, so the constants stay.  tile as in choose_tile.
// The 64x64 (64x128) tile, four (three) blocks of which share a CU: a k tile takes 0.29 (0.45) us with one block on a CU and 0.15 (0.3) more for each further one, 0.5 where the weights
// come from beyond L2; a tile 4.5 us besides.  us, NT, K = 2048, 136 / 400 / 704 / 1024 rows x 2048: 128x128 27.4 / 27.6 / 28.1 / 31.0, 64x64 14.5 / 15.4 / 20.7 / 20.2; x 3072: 27.6 / 28.2 / 30.6 / 31.8 and 14.9 /
// 18.8 / 24.9 / 25.6; 1536 x 3072 40.8, 42.6, 64x128 35.8; K = 4096, x 4096: 47.3 / 48.1 / 49.7 / 52.1 and 34.6 / 36.0 / 43.3 / 51.6.
// A bf16 output with a residual, which the four-wave kernel does not take, costs 0.3 us for each element a thread stores (each is loaded, added and stored before the next).  us, NN, K = 64, 64x64 / 64x128 / 128x128 /
// 192x256 / 256x256, x 4096: 900 rows 12.5 / 15.3 / 23.6 / 35.8 / 45.7, 2255 37.2 / 36.0 / 59.6 / 46.6 / 62.7, 5000 65.7 / 69.8 / 93.7 / 89.1 / 117, 16000 194 / 198 / 268 / 257 / 255.
double product_us(bool low, const GemmParams &p, int tile, const int *ks) {
  const int bm = tile == 1 ? 256 : (tile == 5 ? 224 : (tile == 2 ? 192 : (tile == 0 ? 128 : 64))), bn = tile == 0 || tile == 4 ? 128 : (tile == 3 ? 64 : 256);
  long long nt = 0, n[3] = {0, 0, 0}, blocks = 0, cols = 0;
  for (int s = 0; s < p.n_ns; ++s) { nt += cdiv(p.ns[s].N, bn); cols += p.ns[s].N; }
  for (int g = 0; g < p.n_mg; ++g) blocks += n[g] = (long long)cdiv(p.mg[g].M, bm) * nt * (ks ? ks[g] : 1);
  const int most = tile == 3 ? 4 : 3, per_cu = (int)std::min<long long>(most, std::max<long long>(1, (blocks + 255) / 256));      // resident blocks of the small tiles
  double d[3] = {0, 0, 0};
  for (int g = 0; g < p.n_mg; ++g) {
    const double it = std::ceil((double)cdiv(p.K, BK) * p.mg[g].npass / (ks ? ks[g] : 1));
    if (tile >= 3) d[g] = it * std::max(tile == 3 ? 0.14 + 0.15 * per_cu : 0.15 + 0.3 * per_cu, cols * p.K > (8 << 20) ? 0.5 : 0.0) + 4.5;
    else if (is_w4_tile(low, tile)) d[g] = (it * (1.07 + 0.3 * std::min(1.0, blocks / 256.0)) + 8) * (tile == 1 ? 1.0 : (tile == 5 ? W4_224_TIME : W4_192_TIME));
    else d[g] = (tile == 2 ? it * 1.45 + 8 : it * (blocks <= 256 ? 0.68 : 1.15) + 6);
    if (p.out_bf16 && !p.swiglu && p.resid_kind) d[g] += 0.3 * bm * bn / (bm > 128 ? 512 : 256);
  }
  return makespan(tile == 0 ? 512 : (tile >= 3 ? 256 * per_cu : 256), p.n_mg, n, d);
}

// 1: 256x256, 5: 224x256, 2: 192x256, 0: 128x128, 3: 64x64, 4: 64x128.  The small tiles, which read twice to four times as much per product, for reductions too short to be cut into slices of
// four k tiles several times over (longer ones of few rows are: 136 x 4096 x 11008 84 us on 64x64 tiles, 33 in 16 slices), where they are at least a tenth faster by product_us: few rows.  (SwiGLU
// mode needs the gate and the up columns of a wave in one tile: 64x128.)
bool is_w4_tile(bool low, int tile) { return tile == 1 || (low && (tile == 2 || tile == 5)); }
int choose_tile(bool low, const GemmParams &p) {
  const double c256 = tile_cost<256, 256>(p, 256, 1.0, 1.0), c128 = tile_cost<128, 128>(p, 512, 2.0, 0.62);
  int tile;
  if (!low) {
    const double c192 = tile_cost<192, 256>(p, 256, 1.0, 0.69);
    tile = c256 <= c192 && c256 <= c128 ? 1 : (c192 <= c128 ? 2 : 0);
  } else {
    // 256, 224 or 192 rows, then that against 128x128
    const double w256 = tile_cost<256, 256>(p, 256, 1.0, 1.0, W4_IDLE_GAIN), w224 = tile_cost<224, 256>(p, 256, 1.0, 0.875 / W4_224_TIME, W4_IDLE_GAIN),
                 w192 = tile_cost<192, 256>(p, 256, 1.0, 0.75 / W4_192_TIME, W4_IDLE_GAIN);
    tile = 0.98 * w256 <= std::min(w224, w192) ? 1 : (w224 <= w192 ? 5 : 2);
    const double c = tile == 1 ? c256 : (tile == 5 ? tile_cost<224, 256>(p, 256, 1.0, 0.875 / W4_224_TIME) : tile_cost<192, 256>(p, 256, 1.0, 0.75 / W4_192_TIME));
    // (one 128x128 block alone on its CU takes 0.6 of what two there take: 136 - 1024 rows x 2048, K = 2048, 27 - 31 us, on 192 rows 33 - 35; 1536 x 3072, 288 blocks, 41 and 33)
    int blocks128 = 0;
    for (int g = 0; g < p.n_mg; ++g)
      for (int s = 0; s < p.n_ns; ++s) blocks128 += cdiv(p.mg[g].M, 128) * cdiv(p.ns[s].N, 128);
    if ((blocks128 <= 256 ? 0.8 : 1.0) * c128 < c) tile = 0;
  }
  int steps = 0;
  for (int g = 0; g < p.n_mg; ++g) steps = std::max(steps, cdiv(p.K, BK) * p.mg[g].npass);
  if (steps > 12) return tile;
  const double us = 0.9 * product_us(low, p, tile, nullptr), u64 = p.swiglu ? us : product_us(low, p, 3, nullptr), u128 = product_us(low, p, 4, nullptr);
  return u64 < us || u128 < us ? (u64 <= u128 ? 3 : 4) : tile;
}

template <int LA, int LB>
hipError_t launch_layout(GemmParams &p, hipStream_t stream, const char **why) {
  const bool low = w4_low<LA, LB>(p);
  if (p.force_w4 || p.swiglu_bwd || has_rope(p) || is_split(p)) {      // forms that only the four-wave kernel has
    if (is_split(p) ? !w4_fits<LA, LB>(p) : !uses_w4<LA, LB>(p)) { *why = "gemm: the problem does not run on the four-wave kernel"; return hipErrorInvalidValue; }
    return launch_w4<LA, LB>(p, p.force_w4 || is_split(p) ? 1 : choose_tile(low, p), stream);
  }
  const int tile = choose_tile(low, p);
  if (is_w4_tile(low, tile)) {
    // the four-wave kernel, at every reduction length (measured against the eight-wave kernel of the same tile:
    // 5 % faster at K = 1024 .. 2048, 7 - 12 % at K >= 4096); the eight-wave kernel takes what does not fit it
    if (w4_fits<LA, LB>(p)) return launch_w4<LA, LB>(p, tile, stream);
    return launch_dl<256, 256, 2, 4, LA, LB, BK, NSTAGES>(p, stream);
  }
  if (tile == 2) return launch_dl<192, 256, 2, 4, LA, LB, BK, NSTAGES>(p, stream);
  if (tile == 3) return launch_dl<64, 64, 2, 2, LA, LB, BK, NSTAGES>(p, stream);
  if (tile == 4) return launch_dl<64, 128, 2, 2, LA, LB, BK, NSTAGES>(p, stream);
  return launch_dl<128, 128, 2, 2, LA, LB, BK, NSTAGES>(p, stream);
}

}  // namespace

hipError_t gemm_launch(int LA, int LB, GemmParams &p, hipStream_t stream, const char **why) {
  *why = nullptr;
  if (p.n_mg < 1 || p.n_mg > 3 || p.n_ns < 1 || p.n_ns > 3) { *why = "gemm: group count"; return hipErrorInvalidValue; }
  if (p.K <= 0) { *why = "gemm: K <= 0"; return hipErrorInvalidValue; }
  if (is_split(p)) {
    bool ok = !p.resid_kind && !p.out_bf16 && !p.swiglu && !p.swiglu_bwd && !has_rope(p);
    for (int g = 0; g < p.n_mg; ++g) {
      const int it = w4_tile_steps(LA, LB, cdiv(p.K, BK), p.mg[g].npass), ks = std::max(1, p.k_splits[g]);
      ok = ok && (ks == 1 || (p.mg[g].c_split_stride > 0 && cdiv(it, ks) * (ks - 1) < it));      // no empty slice
    }
    if (!ok) { *why = "gemm: k slices need plain fp32 output without residual and k tiles for every slice"; return hipErrorInvalidValue; }
  }
  if ((LA == 0 || LB == 0) && p.K % BK) { *why = "gemm: K of a k-contiguous operand must be a multiple of 64"; return hipErrorInvalidValue; }
  if (p.lda % 8 || p.ldb % 8) { *why = "gemm: leading dimension not a multiple of 8"; return hipErrorInvalidValue; }
  if (p.lda <= 0 || p.ldb <= 0 || p.lda >= (1 << 22) || p.ldb >= (1 << 22)) { *why = "gemm: leading dimension out of range"; return hipErrorInvalidValue; }
  for (int g = 0; g < p.n_mg; ++g) {
    const GemmMGroup &G = p.mg[g];
    if (G.M < 0 || G.npass < 1 || G.npass > 3) { *why = "gemm: bad row group"; return hipErrorInvalidValue; }
    if (G.M == 0) continue;
    if (!G.a[0] || !aligned16(G.a[0]) || !G.c) { *why = "gemm: A/C pointer"; return hipErrorInvalidValue; }
    if (G.npass >= 2 && (!G.a[1] || !aligned16(G.a[1]))) { *why = "gemm: A lo pointer"; return hipErrorInvalidValue; }
    if (LA == 1 && G.M % 8) { *why = "gemm: M of an m-contiguous operand must be a multiple of 8"; return hipErrorInvalidValue; }
    if (p.resid_kind && !G.resid) { *why = "gemm: residual pointer"; return hipErrorInvalidValue; }
    for (int s = 0; s < p.n_ns; ++s)
      if (G.npass == 3 && !p.ns[s].b[1]) { *why = "gemm: B lo pointer"; return hipErrorInvalidValue; }
  }
  for (int s = 0; s < p.n_ns; ++s) {
    const GemmNSeg &S = p.ns[s];
    if (S.N <= 0 || !S.b[0] || !aligned16(S.b[0]) || (S.b[1] && !aligned16(S.b[1]))) { *why = "gemm: bad column segment"; return hipErrorInvalidValue; }
    if (LB == 1 && S.N % 8) { *why = "gemm: N of an n-contiguous operand must be a multiple of 8"; return hipErrorInvalidValue; }
  }
  if (p.out_bf16 && p.ldc % 2) { *why = "gemm: bf16 output needs an even leading dimension"; return hipErrorInvalidValue; }
  if (p.swiglu) {
    if (LA != 0 || LB != 0 || p.n_ns != 2 || p.ns[0].N != p.ns[1].N || p.ns[0].N % 2 || p.resid_kind || p.n_kseg > 1 || p.ldc % 2) {
      *why = "gemm: SwiGLU mode needs the NT form, two equal column segments and a plain bf16 output";
      return hipErrorInvalidValue;
    }
  }
  if (has_rope(p)) {
    bool ok = LA == 0 && LB == 0 && !p.swiglu && !p.swiglu_bwd && !p.out_bf16 && !p.resid_kind && p.n_kseg <= 1 && (p.rope_hd == 64 || p.rope_hd == 128);
    for (int s = 0; s < p.n_ns; ++s) ok = ok && p.ns[s].N % 128 == 0;
    for (int g = 0; g < p.n_mg; ++g)
      for (int s = 0; s < p.n_ns; ++s) {
        if (p.mg[g].rope == 1) ok = ok && p.rope_cs && p.ns[s].rope_hi;
        if (p.mg[g].rope == 2) ok = ok && p.rope_cs_inf && p.ns[s].rope_inf && (!p.ns[s].rope_cache || (p.rope_slots && p.rope_hkv > 0 && p.rope_bshift >= 0));
      }
    if (!ok) { *why = "gemm: rotary mode needs the NT form, plain fp32 output for the other rows, segments of a multiple of 128 columns, 64- or 128-wide heads and angle tables"; return hipErrorInvalidValue; }
  }
  if (p.swiglu_bwd) {
    if (LA != 0 || LB != 1 || p.n_ns != 1 || p.ns[0].c_col != 0 || p.ns[0].N % 2 || !p.out_bf16 || p.resid_kind || p.swiglu ||
        p.ldc != 2ll * p.ns[0].N) {
      *why = "gemm: SwiGLU backward mode needs the NN form, one column segment, bf16 output [M, 2N] and no residual";
      return hipErrorInvalidValue;
    }
    for (int g = 0; g < p.n_mg; ++g)
      if (!p.mg[g].c_gu) { *why = "gemm: SwiGLU backward mode needs G | U of the forward"; return hipErrorInvalidValue; }
  }
  if (p.n_kseg > 1) {
    if (p.n_kseg > 3 || p.n_ns != 1 || p.kseg_start[0] != 0 || p.kseg_start[p.n_kseg] != p.K) { *why = "gemm: bad k segments"; return hipErrorInvalidValue; }
    for (int g = 0; g < p.n_mg; ++g)
      if (p.mg[g].npass != 1) { *why = "gemm: k segments need single-pass row groups"; return hipErrorInvalidValue; }
    for (int s = 0; s < p.n_kseg; ++s)
      if (!p.kseg_b[s] || !aligned16(p.kseg_b[s]) || p.kseg_start[s] % BK || p.kseg_start[s + 1] <= p.kseg_start[s]) { *why = "gemm: bad k segment"; return hipErrorInvalidValue; }
  }
  // multi-pass row groups first (stable): their tiles take longest and should start first
  for (int i = 1; i < p.n_mg; ++i)
    for (int j = i; j > 0 && p.mg[j].npass > p.mg[j - 1].npass; --j) {
      std::swap(p.mg[j], p.mg[j - 1]);
      std::swap(p.k_splits[j], p.k_splits[j - 1]);
    }
  if (LA == 0 && LB == 0) return launch_layout<0, 0>(p, stream, why);
  if (LA == 0 && LB == 1) return launch_layout<0, 1>(p, stream, why);
  if (LA == 1 && LB == 1) return launch_layout<1, 1>(p, stream, why);
  *why = "gemm: unsupported layout";
  return hipErrorInvalidValue;
}

static bool low_tiles(int LA, int LB, const GemmParams &p) { return LA == 0 && (LB == 0 ? w4_low<0, 0>(p) : w4_low<0, 1>(p)); }

double gemm_estimate_us(int LA, int LB, const GemmParams &p) {
  const bool low = low_tiles(LA, LB, p);
  return product_us(low, p, choose_tile(low, p), nullptr);
}

bool gemm_uses_four_wave(int LA, int LB, const GemmParams &p) {
  if (LA == 0 && LB == 0) return uses_w4<0, 0>(p);
  if (LA == 0 && LB == 1) return uses_w4<0, 1>(p);
  if (LA == 1 && LB == 1) return uses_w4<1, 1>(p);
  return false;
}

bool gemm_pick_splits(int LA, int LB, const GemmParams &base, const GemmParams &plain, size_t part_floats, double extra_us, int k_splits[3]) {
  for (int g = 0; g < 3; ++g) k_splits[g] = 1;
  const bool fits = LA == 0 ? (LB == 0 ? w4_fits<0, 0>(plain) : w4_fits<0, 1>(plain)) : w4_fits<1, 1>(plain);
  long long nt = 0, units = 0, rows = 0;
  for (int s = 0; s < plain.n_ns; ++s) nt += cdiv(plain.ns[s].N, 256);
  for (int g = 0; g < plain.n_mg; ++g) { units += cdiv(plain.mg[g].M, 256) * nt * plain.mg[g].npass; rows += plain.mg[g].M; }
  if (!fits || units >= 5 * 256) return false;           // five rounds and more: the last one is short beside the rest
  const bool round_trip = !(base.out_bf16 || base.swiglu || base.swiglu_bwd || has_rope(base));   // fp32 result written and read back anyway
  // (a residual costs an epilogue 3 - 7 us, and a consumer that adds slices next to nothing: 2329 x 2048 x 2048 with a bf16 residual 43 us on 192 rows, 33 in two slices and 6 more in the consumer.
  // Rotary mode costs the launch of its table, 5 us, and about 7 in the epilogue, which counts where the product is short: inference rows alone, in one pass.  Product, rotation and table or slices in us, in rotary mode / sliced: 1600, 2100 x 3072, K = 2048: 45.6, 47.4 / 40.2,
  // 47.4; 453 x 12288, K = 4096: 82 / 68; past these the former wins, 2800 x 3072 50 / 57 and 520 .. 2800 x 12288 by a tenth and more)
  const bool low = low_tiles(LA, LB, base);
  const double t0 = product_us(low, base, choose_tile(low, base), nullptr) + (base.resid_kind ? 4.0 : (has_rope(base) && plain.mg[0].npass == 1 ? 12.0 : 0.0));
  double best = 0.93 * t0;
  bool found = false;
  static const int cand[] = {2, 3, 4, 5, 6, 8, 12, 16};
  for (int c : cand) {
    // slices of about equal length: row groups with fewer passes are cut into fewer
    int ks[3] = {1, 1, 1}, most = 1;
    double floats = 0;
    bool ok = true;
    for (int g = 0; g < plain.n_mg; ++g) most = std::max(most, plain.mg[g].npass);
    for (int g = 0; g < plain.n_mg; ++g) {
      const int nk = cdiv(plain.K, BK), it = w4_tile_steps(LA, LB, nk, plain.mg[g].npass);
      ks[g] = std::max(1, (c * plain.mg[g].npass + most / 2) / most);
      if (it < nk * plain.mg[g].npass) ks[g] = cdiv(it, cdiv(it, ks[g]));      // steps of two passes: 88 make no 12 slices, but 11 (a training step of 84 rows, edge layer: 640 us with 8, 635 with 11)
      ok = ok && nk * plain.mg[g].npass / ks[g] >= 4 && cdiv(it, ks[g]) * (ks[g] - 1) < it;
      floats += (double)ks[g] * plain.mg[g].M * plain.ldc;
    }
    if (!ok || floats > (double)part_floats) continue;
    // every partial result is written and read once: 5 TB/s
    const double t = product_us(false, plain, 1, ks) + extra_us + (floats - (round_trip ? 1.0 : 0.0) * rows * plain.ldc) * 8.0 / 5e6;
    if (t < best) {
      best = t;
      found = true;
      for (int g = 0; g < 3; ++g) k_splits[g] = ks[g];
    }
  }
  return found;
}
