// 256x256x64 block tile on FOUR waves (2 x 2, wave tile 128x128; with TM = 7 and 6 224 and 192 rows, waves of
// 112 and 96), included by gemm.hip inside its anonymous namespace.
//
// One wave per SIMD owns all 512 registers of a lane: 256 accumulator registers (AGPRs) and 256
// VGPRs, of which 128 are two register sets that stage operand tiles on their way global -> VGPR
// -> LDS.  Compared with the 8-wave kernel (wave tile 128x64) the fragments of a k tile are 128 KB
// of LDS reads instead of 192 (a wave reads 32 for its 128 MFMAs), the tiles reach LDS through 16-byte ds_writes (a quarter of the LDS time of
// a direct global->LDS load) and every global load has two tile times to land.  Nothing covers a
// stall of the only wave of a SIMD, so the loop is written as an explicit schedule: one fragment
// read, or one half of a "move" (wait for a staged register and ds_write it; request the same register again for
// the tile three ahead) behind single MFMAs, one barrier per k tile, and the first fragments of the
// next tile read behind that barrier under the last MFMAs of the current one.
//
// The MFMAs are the 16x16x32 form.  What bounds the loop on real data is power: with 32x32x16 MFMAs the pipes were
// busy 0.72 - 0.81 of the cycles at a clock of 1.6 GHz.  A loop of nothing but MFMAs on random operands runs at
// 1.83 PFLOP/s with 32x32x16 and at 2.06 with 16x16x32, with the fragment reads of this kernel 1.73 and 1.95 (on zeros
// all of them 2.46): the 16x16 form moves half the accumulator bits per flop, which costs less than its doubled operand reads.
//
// Operand loads are buffer loads whose resource spans the operand from its first to its last
// element: a load beyond the end returns zeros, which is the whole edge handling (rows past M or N
// of a k-contiguous operand, k past K of a row-contiguous one).  The loads are issued as asm and
// counted by the kernel (s_waitcnt vmcnt(31) before the ds_write of a register: the load that
// filled it two tile times ago is followed by 31 younger ones); left to the compiler, its wait
// insertion settles on half that distance for one of the two phases of the loop.  A staged
// register is touched by nothing but its load and its ds_write; the build checks the generated
// code for that.

template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;
typedef __attribute__((address_space(3))) char lds_char_t;

#define W4_SB __builtin_amdgcn_sched_barrier(0)
#define W4_IC(n) std::integral_constant<int, (n)>{}
#define W4_INL __attribute__((always_inline))

// Tile tt of a block's reduction -> where its operands come from: the low and high words of the operand
// bases (a buffer resource is {base lo, base hi, bytes, format}; u: the up weights in SwiGLU mode, else the
// B base again), the extent of B and the byte offsets of the tile's origin.  Bases differ by pass (hi / lo
// term) and by k segment.  Plain scalars, and a free function with every input passed by value: a resource
// that is the phi of two branches lands in vector registers, and written as a lambda the selections between
// captured variables become selections between their addresses and keep all of them in private memory.
struct W4Cur { uint32_t a0, a1, b0, b1, u0, u1, b_bytes, oa, ob; };
template <int LA, int LB>
__device__ __forceinline__ W4Cur w4_tile_src(int tt, int nk, int m0, int n0, int N, int K, long long lda, long long ldb,
                                             const void *a_hi, const void *a_lo, const void *b_hi, const void *b_lo, const void *u_hi, const void *u_lo,
                                             int swiglu, int n_kseg, int ks_s1, int ks_s2, const void *ks_b0, const void *ks_b1, const void *ks_b2) {
  constexpr int BKT = 64;
  const int pass = tt >= 2 * nk ? 2 : (tt >= nk ? 1 : 0);
  const int k0 = (tt - pass * nk) * BKT;
  W4Cur r;
  const uint64_t ab = (uint64_t)(pass == 1 ? a_lo : a_hi);
  r.a0 = (uint32_t)ab;
  r.a1 = (uint32_t)(ab >> 32) & 0xffffu;
  r.oa = (uint32_t)((LA == 0 ? (long long)m0 * lda + k0 : (long long)k0 * lda + m0) * 2);
  // the k range may be a concatenation whose segment ks takes its B rows from its own matrix
  const int ks = n_kseg > 1 ? (k0 >= ks_s1 ? 1 : 0) + (n_kseg > 2 && k0 >= ks_s2 ? 1 : 0) : 0;
  const int s0 = ks == 0 ? 0 : (ks == 1 ? ks_s1 : ks_s2), s1 = ks + 1 >= n_kseg ? K : (ks == 0 ? ks_s1 : ks_s2);
  const int kl = k0 - s0;
  const uint64_t bb = (uint64_t)(n_kseg > 1 ? (ks == 0 ? ks_b0 : (ks == 1 ? ks_b1 : ks_b2)) : (pass == 2 ? b_lo : b_hi));
  const uint64_t ub = swiglu ? (uint64_t)(pass == 2 ? u_lo : u_hi) : bb;
  r.b0 = (uint32_t)bb;
  r.b1 = (uint32_t)(bb >> 32) & 0xffffu;
  r.u0 = (uint32_t)ub;
  r.u1 = (uint32_t)(ub >> 32) & 0xffffu;
  r.b_bytes = (uint32_t)(2 * (LB == 0 ? (long long)(N - 1) * ldb + (s1 - s0) : (long long)(s1 - s0 - 1) * ldb + N));
  r.ob = (uint32_t)((LB == 0 ? (long long)n0 * ldb + kl : (long long)kl * ldb + n0) * 2);
  return r;
}
// The resources of a tile in scalar registers.
struct W4Src { u32x4_t qa, qb, qu; uint32_t oa, ob; };
__device__ __forceinline__ uint32_t w4_sgpr(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
// dead: a request that only keeps the count of loads in flight constant (past the last tile) gets empty
// resources: its loads return zeros without going to memory.
__device__ __forceinline__ W4Src w4_resources(const W4Cur c, uint32_t a_bytes, bool dead = false) {
  W4Src r;
  a_bytes = dead ? 0u : a_bytes;
  const uint32_t b_bytes = dead ? 0u : c.b_bytes;
  r.qa = u32x4_t{w4_sgpr(c.a0), w4_sgpr(c.a1), w4_sgpr(a_bytes), 0x00020000u};
  r.qb = u32x4_t{w4_sgpr(c.b0), w4_sgpr(c.b1), w4_sgpr(b_bytes), 0x00020000u};
  r.qu = u32x4_t{w4_sgpr(c.u0), w4_sgpr(c.u1), w4_sgpr(b_bytes), 0x00020000u};
  r.oa = c.oa;
  r.ob = c.ob;
  return r;
}

// How an operand tile lies in LDS, for 256 threads and 16x16x32 fragments (8 consecutive k of one row per lane).
// Every address is one lane part plus constants.
// LAYOUT 0 (k contiguous): [row][64 k], 16-byte chunk kc of a row at position kc ^ ((row / 2) % 8).
// LAYOUT 1 (rows contiguous): [k][256 rows] with a pitch of 544 bytes and 128 more behind every eighth k.  A fragment
// comes from two transposing reads, whose lanes take 8 bytes of four k and, in the next 16 lanes, of the four k
// eight further on: 32 bytes each at eight different places of the 256 bytes of all banks.  (A swizzle would have to mix lane bits
// into the bits that select the fragment, i.e. take an address register per fragment.)
template <int LAYOUT>
struct W4Tile {
  static constexpr int BYTES = LAYOUT == 0 ? 256 * 128 : 8 * 4480;
  static constexpr int LOAD_STEP = LAYOUT == 0 ? 4096 : 4480;      // LDS bytes from one load of a thread to its next (of 8)
  static constexpr int LOAD_ROWS = LAYOUT == 0 ? 32 : 8;           // ... and rows of the matrix in memory
  static constexpr int NFA = LAYOUT == 0 ? 2 : 1;                  // lane addresses of fragments (LAYOUT 0: one per k step)
  static constexpr int RPF = LAYOUT == 0 ? 1 : 2;                  // LDS reads per fragment
  // byte offset in memory and in LDS of a thread's first load
  static __device__ __forceinline__ uint32_t global_offset(int thread, long long ld) {
    if constexpr (LAYOUT == 0) {
      const int lr = thread >> 3, kc = (thread & 7) ^ ((lr >> 1) & 7);
      return (uint32_t)((lr * ld + kc * 8) * 2);
    } else {
      return (uint32_t)(((thread >> 5) * ld + (thread & 31) * 8) * 2);
    }
  }
  static __device__ __forceinline__ uint32_t lds_offset(int thread) {
    return LAYOUT == 0 ? (uint32_t)thread * 16u : (uint32_t)((thread >> 5) * 544 + (thread & 31) * 16);
  }
  // fragment f of k step kk starts at frag_lane(w0, lane, kk) + frag_const(kk, f); w0: the wave's first row
  static __device__ __forceinline__ uint32_t frag_lane(int w0, int lane, int kk) {
    const int q = lane >> 4, j = lane & 15;
    if constexpr (LAYOUT == 0) return (uint32_t)((w0 + j) * 128 + (((4 * kk + q) ^ (j >> 1)) * 16));
    else return (uint32_t)((8 * q + (j >> 2)) * 544 + q * 128 + (w0 + 4 * (j & 3)) * 2);
  }
  static constexpr int frag_const(int kk, int f) { return LAYOUT == 0 ? f * 2048 : kk * (32 * 544 + 4 * 128) + f * 32; }
  static constexpr int FRAG_HALF = 4 * 544;                        // LAYOUT 1: from the first four k of a fragment to the others
};
template <int LA, int LB>
constexpr size_t w4_lds_bytes() { return 2 * ((size_t)W4Tile<LA>::BYTES + W4Tile<LB>::BYTES); }

// An accumulator element for the epilogue, read where it lives.  The accumulators stay in AGPRs from the loop to
// the end of the kernel; handed over as plain values, the register allocator copies whole 16-register blocks into
// VGPRs at the end of the loop for all epilogue variants at once, spills what does not fit and reloads a block
// per element between the stores (every reload a wait that drains the stores in flight).
__device__ __forceinline__ float w4_acc_rd(float a) {
  float v;
  asm("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
  return v;
}

// (asm: with the builtin the register allocator gives some of the 64 accumulators two homes and moves them around the loop)
__device__ __forceinline__ void w4_mfma(f32x4_t &c, const u32x4_t b, const u32x4_t a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(b), "v"(a));
}

__device__ __forceinline__ void w4_clear(f32x4_t &c) {
  c = f32x4_t{0.f, 0.f, 0.f, 0.f};
  asm volatile("" : "+a"(c));
}

// Steps of the reduction of an output tile, which slices are cut from: k tiles times passes, or - two passes of the NT form, which go through
// every k tile together - k tiles.
__host__ __device__ constexpr int w4_tile_steps(int LA, int LB, int nk, int npass) { return LA == 0 && LB == 0 && npass == 2 ? nk : nk * npass; }

// Moves of the quarters of a tile time, by how many there are in all, and how many are done before a quarter.
constexpr int w4_quarter_moves(int all, int quarter) {
  constexpr int PER_Q[7][8] = {{2, 2, 1, 1, 2, 2, 0, 0}, {2, 2, 1, 2, 2, 2, 0, 0}, {2, 2, 2, 2, 2, 2, 0, 0}, {}, {3, 3, 2, 2, 2, 2, 0, 0}, {3, 3, 2, 2, 3, 2, 0, 0}, {3, 3, 3, 3, 2, 2, 0, 0}};
  return PER_Q[all - 10][quarter];
}
constexpr int w4_moves_before(int all, int quarter) {
  int n = 0;
  for (int x = 0; x < quarter; ++x) n += w4_quarter_moves(all, x);
  return n;
}

// TM: blocks of 16 rows of a wave, 8 (256-row tiles), 7 or 6 (224 and 192 rows, k-contiguous A): row counts and rounds of tiles that 256 does not divide.
template <int LA, int LB, int TM>
__global__ __launch_bounds__(256) void gemm_bf16_w4_kernel(const GemmParams p) {
  constexpr int BM = 32 * TM, BN = 256, BKT = 64, NTHR = 256, WGN = 2, WTM = 16 * TM, WTN = 128, TN = 8;      // TM x TN blocks of 16x16
  static_assert(TM == 8 || (LA == 0 && (TM == 6 || TM == 7)), "six to eight blocks of rows; fewer than eight only of a k-contiguous A");
  using SA = W4Tile<LA>;
  using SB = W4Tile<LB>;
  constexpr int NL = BN * BKT / 8 / NTHR, NLA = BM * BKT / 8 / NTHR, NM = NLA + NL;      // 16-byte loads per lane of a B tile (8), of an A tile (TM), and both
  constexpr int AC0 = (TM + 1) / 2;            // A fragments of a wave's first half
  // LDS: A stage 0 | A stage 1 | B stage 0 | B stage 1
  extern __shared__ __align__(16) unsigned char smem_raw[];
  lds_char_t *const lbase = (lds_char_t *)(lds_void_t *)smem_raw;

  // The arguments span nine lines of the scalar cache, and the mapping below walks them in a chain of dependent loads; asked
  // for one line after the other the first block on a CU waits for each (1 us a launch, 3072 x 4096 x 1024: 33.2 -> 32.3 us).
  asm volatile("" ::"s"(p.mg[0].M), "s"(p.mg[1].M), "s"(p.mg[2].M), "s"(p.ns[0].N), "s"(p.ns[1].N), "s"(p.ns[2].N), "s"(p.K), "s"(p.n_kseg), "s"(p.k_splits[2]), "s"(p.mt_start[3]),
               "s"(p.nt_start[3]), "s"(p.swiglu_bwd));

  // block -> tile and k slice: the mapping of gemm_bf16_dl_kernel over the tiles; a tile of row group g takes k_splits[g]
  // blocks in a row
  const int n_ns_eff = p.swiglu ? 1 : p.n_ns;
  const int total_nt = p.nt_start[n_ns_eff];
  int g = 0, first_blk = 0, vb = (int)blockIdx.x;
  while (g + 1 < p.n_mg && vb >= (p.mt_start[g + 1] - p.mt_start[g]) * total_nt * p.k_splits[g]) {
    vb -= (p.mt_start[g + 1] - p.mt_start[g]) * total_nt * p.k_splits[g];
    first_blk += (p.mt_start[g + 1] - p.mt_start[g]) * total_nt;
    ++g;
  }
  const int ks = p.k_splits[g], slice = vb % ks;
  vb = first_blk + vb / ks;
  const int mtc = p.mt_start[g + 1] - p.mt_start[g], T = mtc * total_nt;
  int v = 0;
  {
    const int x = vb & 7;
    for (int y = 0; y < x; ++y) {
      const int fy = (y - first_blk) & 7;
      v += fy < T ? (T - 1 - fy) / 8 + 1 : 0;
    }
    v += (vb - first_blk - ((x - first_blk) & 7)) >> 3;
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
  const int swiglu = p.swiglu;
  const int m0 = mt_l * BM, n0 = swiglu ? nt_g * (BN / 2) : (nt_g - p.nt_start[s]) * BN;
  const int M = G.M, N = S.N, K = p.K;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WGN, wn = wave % WGN;

  // Block (i, j): the B fragment is the first operand, so register r of a lane holds row 16 i + lane % 16 and column
  // 16 j + 4 (lane / 16) + r - four neighbouring columns, which leave as one 16-byte store.
  f32x4_t acc[TM][TN];
  // (called behind the first requests, whose latency covers it; pinned there, or it ends up behind the first barrier)
  auto clear = [&]() W4_INL {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) w4_clear(acc[i][j]);
  };

  // (two passes that share their B tiles count as one: w4_tile_steps)
  const int nk = (K + BKT - 1) / BKT, n_steps = w4_tile_steps(LA, LB, nk, G.npass), nk_slice = (n_steps + ks - 1) / ks;
  const int tt0 = slice * nk_slice, n_it = min(nk_slice, n_steps - tt0);
  const long long lda = p.lda, ldb = p.ldb;
  const int n_kseg = p.n_kseg;
  const int ks_s1 = p.kseg_start[1], ks_s2 = p.kseg_start[2];
  const void *const ks_b0 = p.kseg_b[0], *const ks_b1 = p.kseg_b[1], *const ks_b2 = p.kseg_b[2];

  const uint32_t a_bytes = (uint32_t)(2 * (LA == 0 ? (long long)(M - 1) * lda + K : (long long)(K - 1) * lda + M));
  const void *const a_hi = G.a[0], *const a_lo = G.npass >= 2 ? G.a[1] : G.a[0];
  const void *const b_hi = swiglu ? p.ns[0].b[0] : S.b[0], *const b_lo = G.npass >= 3 ? (swiglu ? p.ns[0].b[1] : S.b[1]) : b_hi;
  const void *const u_hi = swiglu ? p.ns[1].b[0] : b_hi, *const u_lo = swiglu && G.npass >= 3 ? p.ns[1].b[1] : u_hi;
  using Src = W4Src;
  auto tile_cur = [&](int tt) W4_INL -> W4Cur {
    return w4_tile_src<LA, LB>(tt, nk, m0, n0, N, K, lda, ldb, a_hi, a_lo, b_hi, b_lo, u_hi, u_lo, swiglu, n_kseg, ks_s1, ks_s2, ks_b0, ks_b1, ks_b2);
  };
  auto tile_src = [&](int tt) W4_INL -> Src { return w4_resources(tile_cur(tt), a_bytes); };
  // a tile that continues the k run of the one before it lies stepA / stepB bytes further on
  const uint32_t stepA = (uint32_t)(LA == 0 ? BKT * 2 : BKT * lda * 2), stepB = (uint32_t)(LB == 0 ? BKT * 2 : BKT * ldb * 2);

  // Byte offset of this lane's first load inside an operand tile; load x of a tile lies x * strA (strB) bytes further on.
  const uint32_t offA = SA::global_offset((int)threadIdx.x, lda), offB = SB::global_offset((int)threadIdx.x, ldb);
  const uint32_t strA = (uint32_t)(SA::LOAD_ROWS * lda * 2), strB = (uint32_t)(SB::LOAD_ROWS * ldb * 2);
  // SwiGLU mode: the 128 columns of a wave are 64 gate columns and the 64 up columns of the same hidden units, so loads
  // 4 w .. 4 w + 3 of a tile fetch 64 gate and 64 up rows (32 a load) out of two matrices
  const uint32_t strB_w = swiglu ? 2 * strB : 4 * strB, strB_u = swiglu ? 0u : 2 * strB;
  uint32_t fa[2], fb[2];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    fa[x] = SA::frag_lane(wm * WTM, lane, x < SA::NFA ? x : 0);
    fb[x] = SB::frag_lane(wn * WTN, lane, x < SB::NFA ? x : 0) + 2 * SA::BYTES;
    // The B stages start 64 KB into LDS or further on, beyond the 16-bit offset field of an LDS instruction.  Their lane
    // addresses carry that and are made opaque, so that stage and fragment offsets stay immediates (seen
    // as "lane part + constant" the compiler folds all constants into one and keeps a register per sum).
    asm volatile("" : "+v"(fa[x]));
    asm volatile("" : "+v"(fb[x]));
  }
  uint32_t wofs = SA::lds_offset((int)threadIdx.x), wofs_b = SB::lds_offset((int)threadIdx.x) + 2 * SA::BYTES;
  asm volatile("" : "+v"(wofs));
  asm volatile("" : "+v"(wofs_b));

  u32x4_t ra[2][NLA], rb[2][NL];        // register sets: tile t waits in set (t + 1) & 1
  u32x4_t fra[TM], frb[TN];            // fragments of the current k step; a half of them is replaced as soon as it has been used

  auto bload = [&](u32x4_t &dst, const u32x4_t &rs, uint32_t voff, uint32_t soff) W4_INL {
    asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen" : "=v"(dst) : "v"(voff), "s"(rs), "s"(soff));
  };
  // load x (below NLA: A, then B) of the tile described by `src`
  auto request = [&](auto SET, auto X, const Src &src) W4_INL {
    constexpr int set = decltype(SET)::value, x = decltype(X)::value;
    if constexpr (x < NLA) {
      bload(ra[set][x], src.qa, offA, src.oa + x * strA);
    } else {
      constexpr int y = x - NLA;
      if constexpr (LB == 0) bload(rb[set][y], (y & 2) ? src.qu : src.qb, offB, src.ob + (y >> 2) * strB_w + ((y >> 1) & 1) * strB_u + (y & 1) * strB);
      else bload(rb[set][y], src.qb, offB, src.ob + y * strB);
    }
  };
  auto stage_write = [&](auto SET, auto X, auto ST) W4_INL {
    constexpr int set = decltype(SET)::value, x = decltype(X)::value, st = decltype(ST)::value;
    if constexpr (x < NLA) *(lds_u32x4_t *)(lbase + wofs + st * SA::BYTES + x * SA::LOAD_STEP) = ra[set][x];
    else *(lds_u32x4_t *)(lbase + wofs_b + st * SB::BYTES + (x - NLA) * SB::LOAD_STEP) = rb[set][x - NLA];
  };
  // fragment f of half HF of an operand (OP 0: A, 1: B) for k step kk out of stage st
  auto frag = [&](auto TL, uint32_t base, auto O) W4_INL -> u32x4_t {
    using T = decltype(TL);
    constexpr int o = decltype(O)::value;
    if constexpr (T::RPF == 1) {
      return *(lds_u32x4_t *)(lbase + base + o);
    } else {
      const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(lbase + base + o));
      const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(lbase + base + o + T::FRAG_HALF));
      const u32x2_t l2 = __builtin_bit_cast(u32x2_t, lo), h2 = __builtin_bit_cast(u32x2_t, hi);
      return u32x4_t{l2[0], l2[1], h2[0], h2[1]};
    }
  };
  auto read1 = [&](auto OP, auto ST, auto KK, auto HF, auto FF) W4_INL {
    constexpr int op = decltype(OP)::value, st = decltype(ST)::value, kk = decltype(KK)::value, f = (op == 0 ? AC0 : 4) * decltype(HF)::value + decltype(FF)::value;
    if constexpr (op == 0) fra[f] = frag(SA{}, fa[SA::NFA == 2 ? kk : 0], W4_IC(st * SA::BYTES + SA::frag_const(kk, f)));
    else frb[f] = frag(SB{}, fb[SB::NFA == 2 ? kk : 0], W4_IC(st * SB::BYTES + SB::frag_const(kk, f)));
  };
  auto mfma1 = [&](auto I, auto J) W4_INL {
    constexpr int i = decltype(I)::value, j = decltype(J)::value;
    w4_mfma(acc[i][j], frb[j], fra[i]);
  };

  // One tile time.
  // Eight quarters of sixteen MFMAs: a quarter multiplies one half of the A fragments (AH) with one half of the B
  // fragments (BH), in an order in which consecutive quarters share a half and each half is replaced in the quarter
  // behind its last use (RO: operand, RH: half, RK: k step; the last two out of the next tile).  A quarter walks the half that came
  // last in its outer loop (OUTER_B), so a fragment has about sixteen MFMAs from its read to its first use.
  // Inside a quarter every other row runs backwards, so that consecutive MFMAs always share an operand (1.5 % of an MFMA-only loop
  // on random operands; power again).
  // What follows an MFMA: RD a fragment read, MW / MR the write and the request of a move; the moves (PER_Q of the quarter) over the first six quarters.
  // An MFMA takes 16 cycles and an instruction of the one wave four, so a third instruction behind one is late: write and request
  // behind one MFMA cost 2 - 3 %, the moves spread over the whole quarter 1 - 2 %.  (16384 x 4096 x 4096: 1.34 us a k tile on
  // random operands with all of it, 1.32 without the output stores, 1.15 without the loads, 1.24 without the ds_writes, 1.06 without
  // both, 1.21 without the fragment reads; with 32x32x16 MFMAs 1.49.)
  // read(operand, from the next tile, k step, half, fragment); write(move), request(move); mid: between two MFMAs of the seventh
  // quarter, in front of the barrier; turn: right behind the barrier, before the first read from the next tile.
  auto tile_time = [&](auto MOVES, auto read, auto write, auto request_, auto mid, auto turn) W4_INL {
    static_for<0, 8>([&](auto PP) W4_INL {
      constexpr int pp = decltype(PP)::value;
      constexpr int AH[8] = {0, 0, 1, 1, 0, 0, 1, 1}, BH[8] = {0, 1, 1, 0, 1, 0, 0, 1};
      constexpr int RO[8] = {1, 0, 0, 1, 1, 0, 0, 1}, RH[8] = {1, 1, 0, 1, 0, 1, 0, 0}, RK[8] = {0, 0, 1, 1, 1, 1, 0, 0};
      constexpr bool OUTER_B[8] = {true, true, false, false, true, true, false, false};
      // (a quarter of three A fragments has twelve MFMAs)
      constexpr int NMV = decltype(MOVES)::value;
      static_assert(NMV == 16 || NMV == 15 || NMV == 14 || NMV == 12 || NMV == 11 || NMV == 10, "moves of a tile time");
      constexpr int per_q = w4_quarter_moves(NMV, pp), m0_q = w4_moves_before(NMV, pp);
      constexpr int ac = AH[pp] ? TM - AC0 : AC0, nq = 4 * ac;
      static_assert(nq == 16 || nq == 12, "three or four A fragments a half");
      static_for<0, nq>([&](auto Q) W4_INL {
        constexpr int q = decltype(Q)::value, in = OUTER_B[pp] ? ac : 4, o = q / in, n = o & 1 ? in - 1 - q % in : q % in;
        mfma1(W4_IC(AC0 * AH[pp] + (OUTER_B[pp] ? n : o)), W4_IC(4 * BH[pp] + (OUTER_B[pp] ? o : n)));
        W4_SB;
        constexpr int RD[2][16] = {{0, -1, -1, -1, 1, -1, -1, -1, 2, -1, -1, -1, 3, -1, -1, -1}, {0, -1, -1, 1, -1, -1, 2, -1, -1, 3, -1, -1, -1, -1, -1, -1}};
        constexpr int RD6[2][16] = {{-1, -1, -1, -1, -1, -1, -1, -1, 0, -1, 1, -1, 2, -1, 3, -1}, {-1, -1, -1, -1, -1, 0, -1, 1, -1, 2, -1, 3, -1, -1, -1, -1}};      // behind the barrier
        constexpr int MW[2][16] = {{-1, 0, -1, -1, -1, 1, -1, -1, -1, 2, -1, -1, -1, -1, -1, -1}, {-1, 0, -1, -1, 1, -1, -1, 2, -1, -1, -1, -1, -1, -1, -1, -1}};
        constexpr int MR[2][16] = {{-1, -1, 0, -1, -1, -1, 1, -1, -1, -1, 2, -1, -1, -1, -1, -1}, {-1, -1, 0, -1, -1, 1, -1, -1, 2, -1, -1, -1, -1, -1, -1, -1}};
        constexpr int tw = nq == 12, rd = pp == 6 ? RD6[tw][q] : RD[tw][q];
        if constexpr (pp == 6 && q == 2) { mid(); W4_SB; }
        if constexpr (pp == 6 && q == (tw ? 4 : 6)) { __syncthreads(); W4_SB; turn(); W4_SB; }
        if constexpr (rd >= 0 && rd < (RO[pp] == 1 ? 4 : (RH[pp] ? TM - AC0 : AC0))) { read(W4_IC(RO[pp]), W4_IC(pp >= 6), W4_IC(RK[pp]), W4_IC(RH[pp]), W4_IC(rd)); W4_SB; }
        if constexpr (MW[tw][q] >= 0 && MW[tw][q] < per_q) { write(W4_IC(m0_q + MW[tw][q])); W4_SB; }
        if constexpr (MR[tw][q] >= 0 && MR[tw][q] < per_q) { request_(W4_IC(m0_q + MR[tw][q])); W4_SB; }
      });
    });
  };

  // Two passes over the same B (activations in two bf16 terms, NT form): both terms of a k tile are multiplied while its B tile
  // is in LDS, so a tile time fetches and stages 12 instead of 16 pieces per thread.  LDS: A stage 0 holds the first term,
  // A stage 1 the second, the B stages alternate by k tile.  Registers: ra[0] / ra[1] the two terms, rb[0] B; a register is requested
  // again right behind its ds_write, a whole k tile (two tile times) before its data is due, and 24 moves make a turn, so
  // 23 younger loads follow the one that is waited for.  16384 x 4096 with two passes over K = 1024 / 4096 / 11008:
  // 217 / 759 / 2000 us one pass behind the other, 209 / 719 / 1888 so.
  constexpr bool HAS_PAIR = LA == 0 && LB == 0;
  const bool pair = HAS_PAIR && G.npass == 2;
  if constexpr (HAS_PAIR) {
    if (pair) {
      const int n_run = max(n_it, 2);      // k tiles: at least one turn of the loop and one tile behind it
      Src s0 = tile_src(tt0);
      u32x4_t ql = s0.qa;
      ql[0] = w4_sgpr((uint32_t)(uint64_t)a_lo);
      ql[1] = w4_sgpr((uint32_t)((uint64_t)a_lo >> 32) & 0xffffu);
      // byte offsets of the tiles requested next: first term and B; second term
      uint32_t oa = s0.oa, ol = s0.oa, ob = s0.ob;
      const uint32_t b_bytes = s0.qb[2];
      // H, L: the terms of A; requests past the last tile get empty resources
      auto rq_h = [&](auto X) W4_INL { bload(ra[0][decltype(X)::value], s0.qa, offA, oa + decltype(X)::value * strA); };
      auto rq_l = [&](auto X) W4_INL { bload(ra[1][decltype(X)::value], ql, offA, ol + decltype(X)::value * strA); };
      auto rq_b = [&](auto X) W4_INL {
        constexpr int y = decltype(X)::value;
        bload(rb[0][y], (y & 2) ? s0.qu : s0.qb, offB, ob + (y >> 2) * strB_w + ((y >> 1) & 1) * strB_u + (y & 1) * strB);
      };
      auto wr_h = [&](auto X) W4_INL { stage_write(W4_IC(0), X, W4_IC(0)); };
      auto wr_l = [&](auto X) W4_INL { stage_write(W4_IC(1), X, W4_IC(1)); };
      auto wr_b = [&](auto X) W4_INL { stage_write(W4_IC(0), W4_IC(NLA + decltype(X)::value), W4_IC(0)); };      // (wofs_b turns with the B stages)
      auto step_hb = [&](int tile) W4_INL {      // to this tile of the slice
        oa += stepA;
        ob += stepB;
        const bool live = tile < n_it;
        s0.qa[2] = live ? a_bytes : 0u;
        s0.qb[2] = live ? b_bytes : 0u;
        s0.qu[2] = live ? b_bytes : 0u;
      };
      // prologue: tile 0 of the first term and of B into LDS; the rest in the order in which the loop moves it
      static_for<0, NLA>(rq_h);
      static_for<0, NL>(rq_b);
      static_for<0, NLA>(rq_l);
      W4_SB;
      step_hb(1);
      ol += stepA;
      ql[2] = 1 < n_it ? a_bytes : 0u;
      W4_SB;
      clear();
      W4_SB;
      wait_vmcnt<NLA>();
      W4_SB;
      static_for<0, NLA>(wr_h);
      static_for<0, NL>(wr_b);
      W4_SB;
      static_for<0, NL / 2>(rq_b);
      static_for<0, NLA>(rq_h);
      static_for<NL / 2, NL>(rq_b);
      W4_SB;
      step_hb(2);
      wofs_b ^= (uint32_t)SB::BYTES;      // (the B stages lie 64 and 96 KB into LDS)
      __syncthreads();
      static_for<0, AC0>([&](auto F) W4_INL { read1(W4_IC(0), W4_IC(0), W4_IC(0), W4_IC(0), F); });
      static_for<0, 4>([&](auto F) W4_INL { read1(W4_IC(1), W4_IC(0), W4_IC(0), W4_IC(0), F); });
      W4_SB;
      // Pass ph over k tile u: the other term's tile (ph 0: second term of u; 1: first term of u + 1) into the other A stage and half of B
      // of tile u + 1 into the other B stage.
      auto phase = [&](auto PH, auto TAIL, int u) W4_INL {
        constexpr int ph = decltype(PH)::value;
        constexpr bool tail = decltype(TAIL)::value;
        auto write = [&](auto M) W4_INL {
          constexpr int m = decltype(M)::value;
          if constexpr (!tail) {
            wait_vmcnt<2 * NLA + NL - 1>();
            W4_SB;
          }
          if constexpr (tail && (ph == 1 || m >= NLA)) return;
          else if constexpr (m >= NLA) wr_b(W4_IC(m - NLA + ph * (NL / 2)));
          else if constexpr (ph == 0) wr_l(M);
          else wr_h(M);
        };
        auto request2 = [&](auto M) W4_INL {
          constexpr int m = decltype(M)::value;
          if constexpr (tail) return;
          else if constexpr (m >= NLA) rq_b(W4_IC(m - NLA + ph * (NL / 2)));
          else if constexpr (ph == 0) rq_l(M);
          else rq_h(M);
        };
        tile_time(W4_IC(NLA + NL / 2),
                  [&](auto OP, auto NEXT, auto KK, auto HF, auto FF) W4_INL {
                    read1(OP, W4_IC(decltype(OP)::value == 0 ? (decltype(NEXT)::value ? ph ^ 1 : ph) : 0), KK, HF, FF);
                  },
                  write, request2,
                  [&]() W4_INL {
                    if constexpr (!tail && ph == 0) {
                      ol += stepA;
                      ql[2] = u + 2 < n_it ? a_bytes : 0u;
                    }
                    if constexpr (!tail && ph == 1) step_hb(u + 3);
                  },
                  [&]() W4_INL {
                    if constexpr (ph == 1) {
                      wofs_b ^= (uint32_t)SB::BYTES;
#pragma unroll
                      for (int x = 0; x < 2; ++x) fb[x] ^= (uint32_t)SB::BYTES;
                    }
                  });
        if constexpr (!tail && ph == 1) {
          if (u + 2 >= n_run) {      // as below: nothing is in flight behind the loop
            wait_vmcnt<0>();
            W4_SB;
          }
        }
      };
      int u = 0;
      do {
        phase(W4_IC(0), std::false_type{}, u);
        phase(W4_IC(1), std::false_type{}, u);
        ++u;
      } while (u + 1 < n_run);
      phase(W4_IC(0), std::true_type{}, u);
      phase(W4_IC(1), std::true_type{}, u);
    }
  }
  if (!pair) {
  const int n_run = max(n_it, 3);      // tile times: at least one turn of the loop and one tile behind it
  const int rq_last = tt0 + n_it - 1;
  // The request cursor: the tile requested last, where it comes from, and how many tiles may follow it by a step of stepA /
  // stepB alone, without a change of pass or k segment.  Past the last tile the requests, which then only keep the
  // count of loads in flight constant, get empty resources: zeros, without going to memory.
  int rq_tt, rq_left;
  Src rq;
  auto run_length = [&](int tt) W4_INL -> int {
    const int pass_end = tt >= 2 * nk ? 3 * nk : (tt >= nk ? 2 * nk : nk);
    int e = min(pass_end, rq_last + 1);
    if (n_kseg > 1) {      // (k segments exclude passes)
      if (tt * BKT < ks_s1) e = min(e, ks_s1 / BKT);
      else if (tt * BKT < ks_s2) e = min(e, ks_s2 / BKT);
    }
    return (int)w4_sgpr((uint32_t)(e - 1 - tt));
  };
  auto advance = [&]() W4_INL {
    rq.oa += stepA;
    rq.ob += stepB;
    if (__builtin_expect(--rq_left < 0, 0)) {
      rq_tt = min(rq_tt, rq_last) + 1;
      const bool dead = rq_tt > rq_last;
      rq = w4_resources(tile_cur(min(rq_tt, rq_last)), a_bytes, dead);
      rq_left = dead ? 0x7fffffff : run_length(rq_tt);
      rq_tt = dead ? rq_tt : rq_tt + rq_left;      // the last tile of the run
    }
  };
  {
    // prologue: tile 0 -> set 1 -> stage 0; tile 1 -> set 0; tile 2 -> set 1.  Tiles past the last repeat
    // the last one (their data is never multiplied): the loop's wait counts assume every request is issued.
    {
      const Src s0 = tile_src(tt0);
      static_for<0, NM>([&](auto X) W4_INL { request(W4_IC(1), X, s0); });
      W4_SB;
      const Src s1 = w4_resources(tile_cur(tt0 + min(1, n_it - 1)), a_bytes, n_it < 2);
      static_for<0, NM>([&](auto X) W4_INL { request(W4_IC(0), X, s1); });
      W4_SB;
      clear();
      W4_SB;
      wait_vmcnt<NM>();      // tile 0 is in
      W4_SB;
      static_for<0, NM>([&](auto X) W4_INL { stage_write(W4_IC(1), X, W4_IC(0)); });
      W4_SB;
      rq_tt = tt0 + min(2, n_it - 1);
      rq = w4_resources(tile_cur(rq_tt), a_bytes, n_it < 3);
      rq_left = n_it < 3 ? 0x7fffffff : run_length(rq_tt);
      rq_tt += n_it < 3 ? 0 : rq_left;
      static_for<0, NM>([&](auto X) W4_INL { request(W4_IC(1), X, rq); });
      W4_SB;
      advance();
      W4_SB;
      __syncthreads();
      static_for<0, AC0>([&](auto F) W4_INL { read1(W4_IC(0), W4_IC(0), W4_IC(0), W4_IC(0), F); });
      static_for<0, 4>([&](auto F) W4_INL { read1(W4_IC(1), W4_IC(0), W4_IC(0), W4_IC(0), F); });
      W4_SB;
    }
    // Tile time t (phase ph = t & 1): multiply tile t out of stage ph; move tile t+1 from register set ph
    // into stage ph^1 (free since the barrier of tile time t-1), re-requesting each register right after
    // its ds_write for tile t+3; barrier in the seventh of eight quarters; the first fragments of
    // tile t+1 behind the barrier.
    auto phase = [&](auto PH, auto TAIL, int t) W4_INL {
      constexpr int ph = decltype(PH)::value;
      constexpr bool tail = decltype(TAIL)::value;
      // (the tiles behind the loop request nothing: what they would request lies past the last tile, and a
      // load still in flight when control leaves this code could land in a register that holds something else
      // by then; the last of them moves nothing either)
      auto move_write = [&](auto X) W4_INL {
        if constexpr (!tail) {
          wait_vmcnt<2 * NM - 1>();      // the load that filled this register is followed by 31 younger ones (fewer with a smaller A tile)
          W4_SB;
        }
        if constexpr (!(tail && ph == 1)) stage_write(W4_IC(ph), X, W4_IC(ph ^ 1));
      };
      auto move_request = [&](auto X) W4_INL {
        if constexpr (!tail) request(W4_IC(ph), X, rq);
      };
      tile_time(W4_IC(NM),
                [&](auto OP, auto NEXT, auto KK, auto HF, auto FF) W4_INL { read1(OP, W4_IC(decltype(NEXT)::value ? ph ^ 1 : ph), KK, HF, FF); },
                move_write, move_request, [&]() W4_INL { if constexpr (!tail) advance(); }, []() W4_INL {});
      // The compiler does not know which registers have a load in flight, and where control leaves the loop it
      // may copy or spill what is live there.  So the loop's last iteration ends with a wait for all loads (the
      // pipeline runs empty once per output tile), and the code behind the loop issues none.
      if constexpr (!tail && ph == 1) {
        if (t + 3 >= n_run) {
          wait_vmcnt<0>();
          W4_SB;
        }
      }
    };
    // The loop proper has no exit but its back edge; the last one or two tiles run behind it.  It always runs at
    // least once: a reduction of one or two tiles is padded with empty tiles (zeros, requested from empty
    // resources).  With a way around the loop the accumulators reach the code behind it in two register
    // assignments, and the loop's exit pays for the difference with a permutation of all of them.
    int t = 0;
    do {
      phase(W4_IC(0), std::false_type{}, t);
      phase(W4_IC(1), std::false_type{}, t + 1);
      t += 2;
    } while (t + 2 < n_run);
    phase(W4_IC(0), std::true_type{}, t);
    if (t + 1 < n_run) phase(W4_IC(1), std::true_type{}, t + 1);
  }
  }

  // Epilogue.  Register r of block (i, j) holds row 16 i + lane % 16 and column 16 j + 4 (lane / 16) + r of the wave's
  // 128x128.  Every access is a buffer instruction on a view of the wave's part of the
  // matrix (from its first row and column on, as many bytes as its existing rows take): the address is
  // "view + uniform row offset + lane offset".  The row offset is one scalar that walks down 16 rows at a time, the
  // lane offset one register per column block, and that is all the address arithmetic there is.  Edges need no
  // code: an access to a row past the last is out of the view's range, which the hardware drops (a load
  // returns zero), a lane whose columns do not exist carries an offset beyond any view, and an output that was
  // not asked for is an empty view.
  // fp32: lines of 32 columns, eight rows a store (emit).  bf16: the words of two
  // neighbouring blocks go through v_permlane16_swap, which gives every lane eight neighbouring columns: 16 bytes, 64 of 16 rows a store.
  // Column counts that do not divide by that (the NT form only) take narrow accesses at the same places (WIDE = 0, emit_narrow).
  // Against 32x32 blocks, whose lanes own columns of single rows: a quarter of the store instructions, no pair swaps.
  // (no lambda below may name p, G or S: captured by reference the kernel arguments are copied to private memory)
  // (the reads of the accumulators are asm, which the compiler's hazard handling does not look into: the wait
  // states between the last MFMA and the first read of its result are given here)
  asm volatile("s_nop 15\n\ts_nop 15");
  W4_SB;
  const int rk = p.resid_kind, obf = p.out_bf16;
  void *const Cp = G.c;
  const void *const Rp = G.resid;
  const int c_col = S.c_col;
  const long long ldc = p.ldc, ldr = p.ldr;
  const int row_u = m0 + wm * WTM;                                  // the wave's first row
  const int rows_v = max(0, min(WTM, M - row_u));                   // how many of its rows exist
  const int lrow = lane & 15, lq = lane >> 4, lcol = 4 * lq;        // a lane's row and first column in a block
  const int pcol = 16 * (lq & 1) + 8 * (lq >> 1);                   // its first column in a pair of blocks behind the swap
  constexpr uint32_t OUT = 0x80000000u;                             // lane offset of a column that does not exist
  auto view = [](const void *base, long long bytes) W4_INL {
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)bytes, 0x00020000);
  };
  // Cache policy of the stores.  Residual forms and the four outputs of a fine-tune row's SwiGLU, which move most beside the tile itself,
  // carry the non-temporal hint (2), which keeps them out of the way of the operand panels in L2: two passes over 16384 x 4096 x 4096
  // with fp32 / bf16 residual 820 / 806 -> 810 / 800 us, SwiGLU of 16384 x 11008 x 4096 4252 -> 4187.  So do weight gradients (TN), which nothing reads in this call
  // and which would push the weights out of the memory cache: 1 pair on the edge layer, 84 rows, 674 -> 636 us a step.  Other fp32 outputs, slices among them, are read by
  // the next launch and are written through (16): left in L2 they are written back behind the last block, 256 x 16384 x 512 20.5 us, written through 18.1,
  // non-temporal 18.5 but 5 - 8 us more in the readers of an edge layer of 256 rows.  bf16 outputs lose by the hint: 16384 x 4096 x 1024 119 -> 124 us.
  constexpr int PLAIN_STORE = LA == 1 ? 2 : 16, RES_STORE = 2;
  auto store32 = [](uint32_t w, __amdgpu_buffer_rsrc_t q, uint32_t voff, uint32_t soff) W4_INL {
    __builtin_amdgcn_raw_buffer_store_b32(w, q, (int)voff, (int)soff, 0);
  };
  auto store128 = [](auto NT, u32x4_t w, __amdgpu_buffer_rsrc_t q, uint32_t voff, uint32_t soff) W4_INL {
    __builtin_amdgcn_raw_buffer_store_b128(w, q, (int)voff, (int)soff, decltype(NT)::value ? 2 : 0);
  };
  // The bf16 words of two neighbouring blocks (x: even, y: odd; columns +0, +1 and +2, +3 of the lane's four).  vw: lane offset
  // of the pair form; vn, left: of the lane's first column in the even block, and how many columns exist from there on.
  auto store_pair = [&](auto WIDE, auto NT, uint32_t x0, uint32_t x1, uint32_t y0, uint32_t y1, __amdgpu_buffer_rsrc_t q, uint32_t vw, uint32_t vn, int left, uint32_t soff) W4_INL {
    if constexpr (decltype(WIDE)::value != 0) {
      const u32x2_t a = __builtin_amdgcn_permlane16_swap(x0, y0, false, false), b = __builtin_amdgcn_permlane16_swap(x1, y1, false, false);
      store128(NT, u32x4_t{a[0], b[0], a[1], b[1]}, q, vw, soff);
    } else {
      store32(x0, q, left > 0 ? vn : OUT, soff);
      store32(x1, q, left > 2 ? vn + 4u : OUT, soff);
      store32(y0, q, left > 16 ? vn + 32u : OUT, soff);
      store32(y1, q, left > 18 ? vn + 36u : OUT, soff);
    }
  };
  if (swiglu) {
    if constexpr (LA == 0 && LB == 0) {
      // column blocks j and j + 4 (j < 4) of a wave are G and U of the same 16 hidden units
      const int F = N;
      bf16_t *const hi = (bf16_t *)Cp, *const lo = (bf16_t *)G.c_lo, *const gu = (bf16_t *)G.c_gu;
      const int f_u = n0 + wn * (WTN / 2);
      uint32_t vh[2], vg[2], vu[2];      // lane offsets by pair of blocks; U lies F units behind G
#pragma unroll
      for (int jp = 0; jp < 2; ++jp) {
        const bool ok = f_u + jp * 32 + pcol < F;
        vh[jp] = ok ? (uint32_t)((int)(lrow * ldc) + jp * 32 + pcol) * 2u : OUT;
        vg[jp] = ok ? (uint32_t)(lrow * 2 * F + jp * 32 + pcol) * 2u : OUT;
        vu[jp] = ok ? vg[jp] + (uint32_t)F * 2u : OUT;
      }
      const uint32_t nh = (uint32_t)((int)(lrow * ldc) + lcol) * 2u, ng = (uint32_t)(lrow * 2 * F + lcol) * 2u, nu = ng + (uint32_t)F * 2u;
      const auto qh = view(hi + (long long)row_u * ldc + f_u, rows_v * ldc * 2);
      const auto ql = view(lo + (long long)row_u * ldc + f_u, lo ? rows_v * ldc * 2 : 0);
      const auto qg = view(gu + (long long)row_u * 2 * F + f_u, gu ? (long long)rows_v * F * 4 : 0);
      // (row strides go through w4_sgpr: a stride that shares a subexpression with a lane offset is otherwise
      // computed in vector registers, and a vector register as the scalar offset of a buffer instruction
      // becomes a loop over its distinct values)
      const uint32_t h16 = w4_sgpr((uint32_t)(ldc * 32)), g16 = w4_sgpr((uint32_t)F * 64u);      // 16 rows
      // KIND 0: only hm (inference rows); 1: hm in two terms and G, U kept (fine-tune rows)
      auto emit = [&](auto KIND, auto WIDE) W4_INL {
        constexpr int kind = decltype(KIND)::value;
        uint32_t sh = 0, sg = 0;      // row offsets in hm (both terms) and in G|U
        static_for<0, TM>([&](auto I) W4_INL {
          constexpr int i = decltype(I)::value;
          static_for<0, 2>([&](auto JP) W4_INL {
            constexpr int jp = decltype(JP)::value;
            uint32_t wh[4], wl[4], wg[4], wu[4];
            static_for<0, 4>([&](auto W) W4_INL {      // word w: columns 2 (w % 2), + 1 of block 2 jp + w / 2
              constexpr int w = decltype(W)::value, j = 2 * jp + w / 2, r = 2 * (w % 2);
              const float g2[2] = {w4_acc_rd(acc[i][j][r]), w4_acc_rd(acc[i][j][r + 1])};
              const float u2[2] = {w4_acc_rd(acc[i][j + 4][r]), w4_acc_rd(acc[i][j + 4][r + 1])};
              float h2[2];
#pragma unroll
              for (int e = 0; e < 2; ++e) h2[e] = g2[e] * __builtin_amdgcn_rcpf(1.0f + __expf(-g2[e])) * u2[e];
              split_pk_bf16(h2[0], h2[1], wh[w], wl[w]);
              if constexpr (kind != 0) {
                wg[w] = cvt_pk_bf16(g2[0], g2[1]);
                wu[w] = cvt_pk_bf16(u2[0], u2[1]);
              }
            });
            const int left = F - f_u - jp * 32 - lcol;
            store_pair(WIDE, KIND, wh[0], wh[1], wh[2], wh[3], qh, vh[jp], nh + jp * 64u, left, sh);
            if constexpr (kind != 0) {
              store_pair(WIDE, KIND, wl[0], wl[1], wl[2], wl[3], ql, vh[jp], nh + jp * 64u, left, sh);
              store_pair(WIDE, KIND, wg[0], wg[1], wg[2], wg[3], qg, vg[jp], ng + jp * 64u, left, sg);
              store_pair(WIDE, KIND, wu[0], wu[1], wu[2], wu[3], qg, vu[jp], nu + jp * 64u, left, sg);
            }
          });
          sh += h16;
          sg += g16;
          W4_SB;
        });
      };
      if (F % 8 == 0) {
        if (!lo && !gu) emit(W4_IC(0), W4_IC(1));
        else emit(W4_IC(1), W4_IC(1));
      } else {
        emit(W4_IC(1), W4_IC(0));
      }
    }
    return;
  }
  const int col_u = n0 + wn * WTN;                                  // the wave's first column
  if (G.rope) {
    if constexpr (LA == 0 && LB == 0) {
      // Rotary embedding and operand split in the epilogue of the QKV product: the wave's 128 columns are one head of 128
      // or two of 64, so element i of a head sits in the column blocks of its first half and its partner i + HD / 2 in the
      // same register of those of its second half.  (cos, sin) of (row, i) come from the group's table; the rotated (Q, K) or
      // plain (V) values leave as two bf16 terms (fine-tune rows), or as one, K and V also into the paged cache (inference rows).
      // Segments are multiples of 128 columns, so a wave's columns never straddle two.  Bound by its stores; a kernel of its own would
      // read back what the product had written in fp32 (12 bytes per element instead of 2 or 4).  Measured for the inference rows
      // against that kernel: forward of a 7B-class serving batch 1.62 -> 1.57 ms, of a 2329-row prefill of the edge-class layer 339 -> 331 us.
      const int rot = S.rope_rot, Hkv = p.rope_hkv, bshift = p.rope_bshift;
      const bool inf = G.rope == 2;
      bf16_t *const ohi = (bf16_t *)(inf ? S.rope_inf : S.rope_hi), *const olo = inf ? nullptr : (bf16_t *)S.rope_lo, *const cache = inf ? (bf16_t *)S.rope_cache : nullptr;
      const bool ok = col_u < N;
      const long long num_slots = p.rope_num_slots;
      const float *const table = inf ? p.rope_cs_inf : p.rope_cs;
      const auto qs = view(p.rope_slots + row_u, cache ? (long long)rows_v * 4 : 0);
      const uint32_t vo = ok ? (uint32_t)(lrow * N + pcol) * 2u : OUT;      // output rows are N wide; 64 bytes per pair of blocks
      const auto qh = view(ohi + (long long)row_u * N + col_u, (long long)rows_v * N * 2);
      const auto ql = view(olo + (long long)row_u * N + col_u, olo ? (long long)rows_v * N * 2 : 0);
      const uint32_t o16 = w4_sgpr((uint32_t)N * 32u);      // 16 output rows
      auto rows = [&](auto HDC) W4_INL {
        constexpr int HD = decltype(HDC)::value, NH = 128 / HD, HB = 8 / NH;      // heads of a wave, column blocks of a head
        const uint32_t vt = (uint32_t)(lrow * (HD / 2) + lcol) * 8u;              // table; 128 bytes per block
        const auto qt = view(table + (long long)row_u * HD, (long long)rows_v * HD * 4);
        uint32_t so = 0, st = 0;      // row offsets of the outputs and of the table
        static_for<0, (TM + 1) / 2>([&](auto IH) W4_INL {
          u32x4_t cs[2][HB / 2][2];      // the table entries of 32 rows, requested together: (cos, sin) of columns +0, +1 and +2, +3
          int slot[2];
          static_for<0, 2>([&](auto II) W4_INL {
            constexpr int ii = decltype(II)::value, i = 2 * decltype(IH)::value + ii;
            if constexpr (i < TM) {
              static_for<0, HB / 2>([&](auto J) W4_INL {
                static_for<0, 2>([&](auto E) W4_INL {
                  constexpr int j = decltype(J)::value, e = decltype(E)::value;
                  cs[ii][j][e] = __builtin_amdgcn_raw_buffer_load_b128(qt, (int)(vt + j * 128u + e * 16u), (int)(st + ii * (HD * 64u)), 0);
                });
              });
              slot[ii] = (int)__builtin_amdgcn_raw_buffer_load_b32(qs, (16 * i + lrow) * 4, 0, 0);
            }
          });
          st += 2u * (HD * 64u);
          W4_SB;
          static_for<0, 2>([&](auto II) W4_INL {
            constexpr int ii = decltype(II)::value, i = 2 * decltype(IH)::value + ii;
            if constexpr (i < TM) {
              // the row's place in the cache; slots outside it are skipped
              const bool keep = cache && ok && 16 * i + lrow < rows_v && slot[ii] >= 0 && slot[ii] < num_slots;
              bf16_t *const row = cache + ((((long long)(slot[ii] >> bshift) * Hkv + col_u / HD) << bshift) + (slot[ii] & ((1 << bshift) - 1))) * HD + pcol;
              static_for<0, NH>([&](auto HEAD) W4_INL {
                static_for<0, HB / 4>([&](auto JP) W4_INL {
                  constexpr int jp = decltype(JP)::value, hd = decltype(HEAD)::value;
                  uint32_t wh[2][4], wl[2][4];      // first half of the head, second half
                  static_for<0, 4>([&](auto W) W4_INL {
                    constexpr int w = decltype(W)::value, j = 2 * jp + w / 2, e = w % 2, r = 2 * e;
                    float v[2] = {w4_acc_rd(acc[i][HB * hd + j][r]), w4_acc_rd(acc[i][HB * hd + j][r + 1])};
                    float u[2] = {w4_acc_rd(acc[i][HB * hd + j + HB / 2][r]), w4_acc_rd(acc[i][HB * hd + j + HB / 2][r + 1])};
                    if (rot) {
#pragma unroll
                      for (int x = 0; x < 2; ++x) {
                        const float c = __uint_as_float(cs[ii][j][e][2 * x]), sn = __uint_as_float(cs[ii][j][e][2 * x + 1]);
                        const float a = v[x], b = u[x];
                        v[x] = a * c - b * sn;
                        u[x] = b * c + a * sn;
                      }
                    }
                    split_pk_bf16(v[0], v[1], wh[0][w], wl[0][w]);
                    split_pk_bf16(u[0], u[1], wh[1][w], wl[1][w]);
                  });
                  static_for<0, 2>([&](auto H) W4_INL {
                    constexpr int hh = decltype(H)::value, col = HD * hd + (HD / 2) * hh + 32 * jp;
                    const u32x2_t a = __builtin_amdgcn_permlane16_swap(wh[hh][0], wh[hh][2], false, false), b = __builtin_amdgcn_permlane16_swap(wh[hh][1], wh[hh][3], false, false);
                    const u32x4_t q = {a[0], b[0], a[1], b[1]};
                    store128(W4_IC(0), q, qh, vo + col * 2u, so);
                    if (keep) *(u32x4_t *)(row + ((long long)hd << bshift) * HD + (HD / 2) * hh + 32 * jp) = q;
                    if (!inf) store_pair(W4_IC(1), W4_IC(0), wl[hh][0], wl[hh][1], wl[hh][2], wl[hh][3], ql, vo + col * 2u, 0u, 0, so);
                  });
                });
              });
              so += o16;
            }
          });
          W4_SB;
        });
      };
      if (p.rope_hd == 64) rows(W4_IC(64));
      else rows(W4_IC(128));
    }
    return;
  }
  const long long c_col0 = c_col + slice * G.c_split_stride;
  if (p.swiglu_bwd) {
    if constexpr (LA == 0 && LB == 1) {
      // SwiGLU backward in the epilogue of dHm = dY Wd: the tile of dHm never leaves the registers.  With G and U of
      // the forward (bf16 [M, 2F], G | U) it becomes dG = dHm U s (1 + G (1 - s)) and dU = dHm G s, s = sigmoid(G),
      // written as bf16 [M, 2F] (dG | dU) - the same layout, so G, U, dG and dU share one lane
      // offset (U and dU lie F columns further on).  The swap of the pair form is done on
      // the fp32 values, so that a lane computes on the eight columns it loads and stores (F is a multiple of 8).
      const int F = N;
      uint32_t vg[4], vu[4];      // lane offsets by pair of blocks, G / dG and U / dU
#pragma unroll
      for (int jp = 0; jp < 4; ++jp) {
        const bool ok = col_u + jp * 32 + pcol < F;
        vg[jp] = ok ? (uint32_t)(lrow * 2 * F + jp * 32 + pcol) * 2u : OUT;
        vu[jp] = ok ? vg[jp] + (uint32_t)F * 2u : OUT;
      }
      const auto qo = view((bf16_t *)Cp + (long long)row_u * 2 * F + col_u, (long long)rows_v * F * 4);
      const auto qi = view((const bf16_t *)G.c_gu + (long long)row_u * 2 * F + col_u, (long long)rows_v * F * 4);
      const uint32_t s16 = w4_sgpr((uint32_t)F * 64u);      // 16 rows
      uint32_t sc = 0;
      static_for<0, (TM + 3) / 4>([&](auto IH) W4_INL {
        // G and U of 64 rows are requested together (nothing else covers the latency)
        u32x4_t gw[4][4], uw[4][4];
        {
          uint32_t q = sc;
          static_for<0, 4>([&](auto II) W4_INL {
            static_for<0, 4>([&](auto JP) W4_INL {
              constexpr int ii = decltype(II)::value, jp = decltype(JP)::value;
              if constexpr (4 * decltype(IH)::value + ii < TM) {
                gw[ii][jp] = __builtin_amdgcn_raw_buffer_load_b128(qi, (int)vg[jp], (int)q, 0);
                uw[ii][jp] = __builtin_amdgcn_raw_buffer_load_b128(qi, (int)vu[jp], (int)q, 0);
              }
            });
            q += s16;
          });
        }
        W4_SB;
        static_for<0, 4>([&](auto II) W4_INL {
          constexpr int ii = decltype(II)::value, i = 4 * decltype(IH)::value + ii;
          if constexpr (i < TM) static_for<0, 4>([&](auto JP) W4_INL {
            constexpr int jp = decltype(JP)::value;
            float dh[8];
            static_for<0, 4>([&](auto R) W4_INL {
              constexpr int r = decltype(R)::value;
              const u32x2_t t = __builtin_amdgcn_permlane16_swap(__float_as_uint(w4_acc_rd(acc[i][2 * jp][r])), __float_as_uint(w4_acc_rd(acc[i][2 * jp + 1][r])), false, false);
              dh[r] = __uint_as_float(t[0]);
              dh[r + 4] = __uint_as_float(t[1]);
            });
            u32x4_t og, ou;
            static_for<0, 4>([&](auto W) W4_INL {
              constexpr int w = decltype(W)::value;
              const uint32_t g2 = gw[ii][jp][w], u2 = uw[ii][jp][w];
              float dg[2], du[2];
#pragma unroll
              for (int e = 0; e < 2; ++e) {
                const float g = e ? __uint_as_float(g2 & 0xffff0000u) : __uint_as_float(g2 << 16);
                const float u = e ? __uint_as_float(u2 & 0xffff0000u) : __uint_as_float(u2 << 16);
                const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-g));
                du[e] = dh[2 * w + e] * g * sg;
                dg[e] = dh[2 * w + e] * u * sg * (1.0f + g * (1.0f - sg));
              }
              og[w] = cvt_pk_bf16(dg[0], dg[1]);
              ou[w] = cvt_pk_bf16(du[0], du[1]);
            });
            store128(W4_IC(0), og, qo, vg[jp], sc);
            store128(W4_IC(0), ou, qo, vu[jp], sc);
          });
          sc += s16;
        });
        W4_SB;
      });
    }
    return;
  }
  if (obf) {
    // packed bf16 (even column count and offset, no residual)
    uint32_t vp[TN / 2];      // lane offsets by pair of blocks
#pragma unroll
    for (int jp = 0; jp < TN / 2; ++jp) vp[jp] = col_u + jp * 32 + pcol < N ? (uint32_t)((int)(lrow * ldc) + jp * 32 + pcol) * 2u : OUT;
    const uint32_t vn = (uint32_t)((int)(lrow * ldc) + lcol) * 2u;
    const auto qc = view((bf16_t *)Cp + (long long)row_u * ldc + c_col + col_u, rows_v * ldc * 2);
    const uint32_t p16 = w4_sgpr((uint32_t)(ldc * 32));      // 16 rows
    auto emit = [&](auto WIDE) W4_INL {
      uint32_t sc = 0;
      static_for<0, TM>([&](auto I) W4_INL {
        constexpr int i = decltype(I)::value;
        static_for<0, TN / 2>([&](auto JP) W4_INL {
          constexpr int jp = decltype(JP)::value;
          uint32_t w[4];
          static_for<0, 4>([&](auto W) W4_INL {
            constexpr int x = decltype(W)::value, j = 2 * jp + x / 2, r = 2 * (x % 2);
            w[x] = cvt_pk_bf16(w4_acc_rd(acc[i][j][r]), w4_acc_rd(acc[i][j][r + 1]));
          });
          store_pair(WIDE, W4_IC(0), w[0], w[1], w[2], w[3], qc, vp[jp], vn + jp * 64u, N - col_u - jp * 32 - lcol, sc);
        });
        sc += p16;
        W4_SB;
      });
    };
    if constexpr (LB == 1) {
      emit(W4_IC(1));
    } else {
      if (N % 8 == 0) emit(W4_IC(1));
      else emit(W4_IC(0));
    }
    return;
  }
  // fp32 output; RES 0: no residual, 1: + fp32 residual (projections onto an fp32 stream, weight gradients that
  // accumulate), 2: + bf16 residual.  The residuals of 64 rows are requested together before the first is
  // added: with one wave per SIMD nothing else covers the latency of a request.
  // A CU takes a 16-byte access of 64 lanes in 16 cycles where every four neighbouring lanes lie in one piece of 64 bytes, and lane by lane, in 64, where they
  // do not: the rows of a block, one in each of 16 neighbouring lanes, cost 8 us a tile of 256 KB.  So two neighbouring blocks, 32 columns or a line of 128 bytes, are
  // turned: the lanes of eight rows exchange their pieces with those of the other eight (a rotation by eight inside sixteen lanes), which
  // makes two halves of eight whole rows, and a permutation puts the eight pieces of a row into eight neighbouring lanes.  us of 256 x 4096 x 512, 1024 x 4096 x 1024,
  // 4096 x 4096 x 4096 with 64 bytes of 16 rows a store and so: plain 21.0 / 31.2 / 109 -> 17.7 / 26.4 / 107, fp32 residual 27.3 / 36.1 / 120 -> 20.8 / 30.2 / 114.
  auto emit = [&](auto RES) W4_INL {
    constexpr int res = decltype(RES)::value, rsz = res == 2 ? 2 : 4;
    const int prow = lane >> 3, pcol4 = 4 * (lane & 7), from = 4 * (16 * (lane & 3) + 8 * ((lane >> 2) & 1) + prow);
    uint32_t vc[TN / 2], vr[TN / 2];      // lane offsets by pair of blocks, in C and in the residual
#pragma unroll
    for (int jp = 0; jp < TN / 2; ++jp) {
      const bool ok = col_u + 32 * jp + pcol4 < N;
      vc[jp] = ok ? (uint32_t)((int)(prow * ldc) + 32 * jp + pcol4) * 4u : OUT;
      vr[jp] = ok ? (uint32_t)((int)(prow * ldr) + 32 * jp + pcol4) * (uint32_t)rsz : OUT;
    }
    const auto qc = view((char *)Cp + ((long long)row_u * ldc + c_col0 + col_u) * 4, rows_v * ldc * 4);
    const auto qr = view((const char *)Rp + ((long long)row_u * ldr + c_col0 + col_u) * rsz, res ? rows_v * ldr * rsz : 0);
    const uint32_t c8 = w4_sgpr((uint32_t)(ldc * 32)), r8 = w4_sgpr((uint32_t)(ldr * (8 * rsz)));      // 8 rows
    uint32_t sc = 0, sr = 0;
    static_for<0, (TM + 3) / 4>([&](auto IH) W4_INL {
      u32x4_t rv[8][TN / 2];      // by eight rows
      if constexpr (res != 0) {
        static_for<0, 8>([&](auto R8) W4_INL {
          static_for<0, TN / 2>([&](auto JP) W4_INL {
            constexpr int r = decltype(R8)::value, jp = decltype(JP)::value;
            if constexpr (4 * decltype(IH)::value + r / 2 >= TM) {
              rv[r][jp] = u32x4_t{0u, 0u, 0u, 0u};
            } else if constexpr (res == 1) {
              rv[r][jp] = __builtin_amdgcn_raw_buffer_load_b128(qr, (int)vr[jp], (int)sr, 0);
            } else {
              const u32x2_t t = __builtin_amdgcn_raw_buffer_load_b64(qr, (int)vr[jp], (int)sr, 0);
              rv[r][jp] = u32x4_t{t[0], t[1], 0u, 0u};      // widened when it is added
            }
          });
          sr += r8;
        });
        W4_SB;
      }
      static_for<0, 4>([&](auto II) W4_INL {
        constexpr int ii = decltype(II)::value, i = 4 * decltype(IH)::value + ii;
        if constexpr (i < TM) static_for<0, TN / 2>([&](auto JP) W4_INL {
          constexpr int jp = decltype(JP)::value;
          u32x4_t v[2];      // rows 0 .. 7 and 8 .. 15
          static_for<0, 4>([&](auto E) W4_INL {
            constexpr int e = decltype(E)::value;
            const int x = __float_as_int(w4_acc_rd(acc[i][2 * jp][e])), y = __float_as_int(w4_acc_rd(acc[i][2 * jp + 1][e]));
            v[0][e] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, __builtin_amdgcn_update_dpp(x, y, 0x128, 0xF, 0xC, false));      // lanes 8 .. 15: y of the lane eight before
            v[1][e] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, __builtin_amdgcn_update_dpp(y, x, 0x128, 0xF, 0x3, false));      // lanes 0 .. 7: x of the lane eight behind
          });
          static_for<0, 2>([&](auto H) W4_INL {
            constexpr int h = decltype(H)::value;
            static_for<0, 4>([&](auto E) W4_INL {
              constexpr int e = decltype(E)::value;
              const u32x4_t &t = rv[2 * ii + h][jp];
              if constexpr (res == 1) v[h][e] = __float_as_uint(__uint_as_float(v[h][e]) + __uint_as_float(t[e]));
              if constexpr (res == 2) v[h][e] = __float_as_uint(__uint_as_float(v[h][e]) + __uint_as_float(e % 2 ? t[e / 2] & 0xffff0000u : t[e / 2] << 16));
            });
            __builtin_amdgcn_raw_buffer_store_b128(v[h], qc, (int)vc[jp], (int)(sc + h * c8), res ? RES_STORE : PLAIN_STORE);
          });
        });
        sc += 2 * c8;
        W4_SB;
      });
    });
  };
  // The same value by value, for column counts and bf16 residual rows that have no whole pieces (NT form only, but for the latter).
  auto emit_narrow = [&](auto RES) W4_INL {
    constexpr int res = decltype(RES)::value, rsz = res == 2 ? 2 : 4;
    uint32_t vc[TN], vr[TN];      // lane offsets by column block, in C and in the residual
    int left[TN];                 // how many columns exist from the lane's first one on
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      left[j] = N - col_u - j * 16 - lcol;
      vc[j] = left[j] > 0 ? (uint32_t)((int)(lrow * ldc) + lcol + j * 16) * 4u : OUT;
      vr[j] = left[j] > 0 ? (uint32_t)((int)(lrow * ldr) + lcol + j * 16) * (uint32_t)rsz : OUT;
    }
    const auto qc = view((char *)Cp + ((long long)row_u * ldc + c_col0 + col_u) * 4, rows_v * ldc * 4);
    const auto qr = view((const char *)Rp + ((long long)row_u * ldr + c_col0 + col_u) * rsz, res ? rows_v * ldr * rsz : 0);
    const uint32_t c16 = w4_sgpr((uint32_t)(ldc * 64)), r16 = w4_sgpr((uint32_t)(ldr * (16 * rsz)));      // 16 rows
    uint32_t sc = 0, sr = 0;
    static_for<0, (TM + 3) / 4>([&](auto IH) W4_INL {
      u32x4_t rv[4][TN];
      if constexpr (res != 0) {
        static_for<0, 4>([&](auto II) W4_INL {
          static_for<0, TN>([&](auto J) W4_INL {
            static_for<0, 4>([&](auto E) W4_INL {
              constexpr int ii = decltype(II)::value, j = decltype(J)::value, e = decltype(E)::value;
              const int o = left[j] > e ? (int)(vr[j] + e * rsz) : (int)OUT;
              if constexpr (4 * decltype(IH)::value + ii >= TM) rv[ii][j][e] = 0u;
              else if constexpr (res == 1) rv[ii][j][e] = __builtin_amdgcn_raw_buffer_load_b32(qr, o, (int)sr, 0);
              else rv[ii][j][e] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(qr, o, (int)sr, 0) << 16;
            });
          });
          sr += r16;
        });
        W4_SB;
      }
      static_for<0, 4>([&](auto II) W4_INL {
        constexpr int ii = decltype(II)::value, i = 4 * decltype(IH)::value + ii;
        if constexpr (i < TM) static_for<0, TN>([&](auto J) W4_INL {
          static_for<0, 4>([&](auto E) W4_INL {
            constexpr int j = decltype(J)::value, e = decltype(E)::value;
            float f = w4_acc_rd(acc[i][j][e]);
            if constexpr (res != 0) f += __uint_as_float(rv[ii][j][e]);
            store32(__float_as_uint(f), qc, left[j] > e ? vc[j] + e * 4u : OUT, sc);
          });
        });
        sc += c16;
        W4_SB;
      });
    });
  };
  // (rows of a bf16 residual that start on odd elements have no aligned 8-byte pieces; 16-byte accesses to fp32 rows need
  // no more than the 4 bytes every float has)
  const bool wide = LB == 1 || N % 4 == 0, wide_r = wide && rk == 2 && ldr % 2 == 0 && (((uintptr_t)Rp + 2 * c_col0) & 3) == 0;
  if (rk == 0) {
    if constexpr (LB == 1) emit(W4_IC(0));
    else if (wide) emit(W4_IC(0));
    else emit_narrow(W4_IC(0));
  } else if (rk == 1) {
    if constexpr (LB == 1) emit(W4_IC(1));
    else if (wide) emit(W4_IC(1));
    else emit_narrow(W4_IC(1));
  } else {
    if (wide_r) emit(W4_IC(2));
    else emit_narrow(W4_IC(2));
  }
}

// Operand views must fit the 32-bit byte offsets of a buffer load, and 128 rows of an output or residual the
// 31 bits of an offset inside a wave's view.  bf16 output is stored in column pairs and takes no residual here.
template <int LA, int LB>
bool w4_fits(const GemmParams &p) {
  const long long lim = (1ll << 32) - 65536;
  for (int g = 0; g < p.n_mg; ++g) {
    const long long rows = LA == 0 ? p.mg[g].M : p.K;
    if (rows * p.lda * 2 >= lim) return false;
  }
  for (int s = 0; s < p.n_ns; ++s) {
    const long long rows = LB == 0 ? p.ns[s].N : p.K;
    if (rows * p.ldb * 2 >= lim) return false;
    if (p.out_bf16 && !p.swiglu && ((p.ns[s].N & 1) || (p.ns[s].c_col & 1))) return false;
    if (p.swiglu && (p.ns[s].N & 1)) return false;
  }
  if (p.out_bf16 && !p.swiglu && p.resid_kind != 0) return false;
  if (p.swiglu_bwd && !(LA == 0 && LB == 1)) return false;
  for (int g = 0; g < p.n_mg; ++g)
    if (p.mg[g].rope && !(LA == 0 && LB == 0)) return false;
  if (p.ldc >= (1ll << 21) || p.ldr >= (1ll << 21)) return false;
  return true;
}
