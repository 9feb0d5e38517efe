// LDS tiles of the attention kernels (gfx950): ROWS token rows x HD head-dim elements of one
// head, bf16, in their memory layout [row][HD], filled by direct global->LDS loads.
//
// The same tile serves two kinds of MFMA operand:
//  * read_k: 8 consecutive head-dim elements of one tile row per lane (reduction over the head
//    dimension), one 16-byte LDS read;
//  * read_t: for head-dim index 32 t + lane%32, the 8 tile rows kk*16 + 8*(lane/32) .. +7
//    (reduction over the tile rows), two transposing 8-byte reads (ds_read_b64_tr_b16);
// so no transposed copy of a tile is ever built.  A wave-wide direct load writes 64 consecutive
// 16-byte chunks, hence tiles are unpadded; the chunk position inside a row is XOR-swizzled
// with a function of the row that keeps BOTH read patterns free of bank conflicts:
// 16 consecutive rows at one logical chunk (read_k) and 4 consecutive rows x 4 consecutive
// chunks (read_t) each touch 16 different 16-byte bank groups.
#pragma once
#include "common.h"

#include <type_traits>

namespace attn {

template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) const void gbl_void_t;

static __device__ __align__(16) uint4 zero16 = {0u, 0u, 0u, 0u};   // source of the rows of a paged tile beyond the sequence

template <int N>
__device__ __forceinline__ void wait_vmcnt() {   // vmcnt <= N, no wait on the other counters
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// swap bits 2 and 3: the MFMA output row held in register r of lane half g is
// 8*(r/4) + 4*g + r%4; reading operand row swap23(i) for MFMA row i makes register r = 8*mm + e
// of half g hold tile row 16*mm + 8*g + e, the order a B operand wants its 8 reduction indices in.
__device__ __forceinline__ int swap23(int i) { return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1); }

// Sequence of a block of the grid (head, sequence, row tile).  Blocks go to the CUs in turn and all of a small grid are resident at once, so with the sequence
// index as it is a CU gets every row tile of one sequence, and the one with the longest sequence sets the time: turned by the row tile, it gets tiles of several.
// Paged prefill of 160 - 419 rows behind 512 cached ones, 32 heads of 64: 43.5 -> 40.7 us; plain 18.4 -> 16.1.
__device__ __forceinline__ int turned_sequence() { return (int)((blockIdx.y + blockIdx.z) % gridDim.y); }

template <int ROWS, int HD, int NTHR>
struct Tile {
  static constexpr int CPR = HD / 8;                 // 16-byte chunks per row (8 or 16)
  static constexpr int ELEMS = ROWS * HD;
  static constexpr int NCH = ROWS * CPR;
  static constexpr int NI = NCH / NTHR;              // wave-wide loads per wave
  static_assert(HD == 64 || HD == 128, "head dim");
  static_assert(NCH % NTHR == 0, "tile must split evenly over the waves");

  static __device__ __forceinline__ int swz(int row) {
    if constexpr (CPR == 16) return ((row & 3) << 2) | ((row >> 2) & 3);
    else return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
  }

  // Rows row0 .. row0+ROWS-1 of src (row pitch ld elements; src points at row 0, column 0 of the
  // head); rows >= row_end read zeros.  The loads go through a buffer resource that spans the tile's existing rows (its
  // range check is the zero fill): beyond lane_offset, kept from tile to tile, an address costs no vector arithmetic.
  static constexpr int RSTEP = NTHR / CPR;           // rows between two loads of a lane
  static_assert(RSTEP % 16 == 0, "the swizzle of a lane's rows must not change from load to load");
  // (tid: thread among the NTHR that load the tile)
  static __device__ __forceinline__ uint32_t lane_offset(size_t ld, int tid = threadIdx.x) {
    const int lr = tid / CPR, c = (tid % CPR) ^ swz(lr);
    return (uint32_t)(lr * ld * 2) + c * 16;
  }
  static __device__ __forceinline__ void issue(const bf16_t *src, size_t ld, int row0, int row_end, uint32_t lane_off, bf16_t *S, int tid = threadIdx.x) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rows = min(row_end - row0, ROWS);
    const auto q = __builtin_amdgcn_make_buffer_rsrc((void *)(src + (size_t)row0 * ld), 0, (int)(((rows - 1) * ld + HD) * 2), 0x00020000);
#pragma unroll
    for (int i = 0; i < NI; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(q, (lds_void_t *)(S + (wave + (NTHR / 64) * i) * 512), 16, (int)lane_off, (int)(i * RSTEP * ld * 2), 0, 0);
  }

  // Same tile, but row p (a token position of one request) is fetched from a paged cache
  // [blocks, Hkv, B, HD]: block id from the request's block table, B = 1 << bshift.  Positions at or
  // beyond row_end, and block ids outside [0, num_blocks), read zeros.  The entries of this lane's rows are read
  // (paged_entries) a tile time ahead of the loads that need them.
  static __device__ __forceinline__ void paged_entries(const int32_t *bt, int bshift, int row0, int row_end, int32_t (&blk)[NI]) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int pos = row0 + ((wave + (NTHR / 64) * i) * 64 + lane) / CPR;
      blk[i] = pos < row_end ? bt[pos >> bshift] : -1;
    }
  }
  static __device__ __forceinline__ void issue_paged(const bf16_t *cache, const int32_t (&blk)[NI], int bshift, int Hkv, int kvh,
                                                     long long num_blocks, int row0, bf16_t *S) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = wave + (NTHR / 64) * i;
      const int chunk = q * 64 + lane;
      const int lr = chunk / CPR, c = (chunk % CPR) ^ swz(lr);
      const int pos = row0 + lr;
      const bf16_t *p = blk[i] >= 0 && blk[i] < num_blocks
                            ? cache + ((((size_t)blk[i] * Hkv + kvh) << bshift) + (pos & ((1 << bshift) - 1))) * HD + c * 8
                            : (const bf16_t *)&zero16;
      __builtin_amdgcn_global_load_lds((gbl_void_t *)p, (lds_void_t *)(S + q * 512), 16, 0, 0);
    }
  }

  // Operands are read by blocks of asm that end with their wait.  Written with the builtin, a transposing read makes the
  // compiler wait for every direct global->LDS load in flight first (it does not know that they fill the other
  // stage), so the prefetch of the next tile ends where the current one is multiplied; plain reads it hands out one
  // or two at a time between the products.  Addresses are LDS byte addresses.
  // Measured with the buffer loads, the early block-table entries, the constant-against-bound masks and two blocks per CU for the
  // 128-wide dK/dV kernel, which came with it: dK/dV 16 x 768 rows, 32 heads of 128, 507 -> 324 us, two-term forward 391 -> 375, dQ 273 -> 263;
  // 8 x 420 rows, 32 heads of 64, 92 -> 74, 47 -> 41, 43 -> 37; paged prefill of 2329 rows behind 512 cached ones 56 -> 46.
  static __device__ __forceinline__ uint32_t lds_addr(const bf16_t *S) { return (uint32_t)(uintptr_t)(lds_void_t *)S; }
  // chunk (2 kk + half) ^ sw of the row sits at lane address ^ 32 kk: 2 kk has no bit in common with half, a row starts at
  // a multiple of its CPR chunks and a tile at a multiple of 256 bytes.  (The flip is applied behind the addition of the
  // tile: flipped lane addresses are invariants that the compiler would keep in a register each.)
  static __device__ __forceinline__ uint32_t frag_k_lane(int row, int half) { return (uint32_t)(row * HD * 2 + ((half ^ swz(row)) << 4)); }
  // head-dim elements (KK0 + i) * 16 + 8 * half .. +7, i < N (2 or 4), of the row, OFF bytes into the tile
  template <int N, int KK0, int OFF>
  static __device__ __forceinline__ void read_k(uint32_t tile, uint32_t lane, bf16x8_t (&f)[N]) {
    static_assert(N == 2 || N == 4, "two or four operands");
    __builtin_amdgcn_sched_barrier(0);      // (hoisted over the products in front of them, the reads only take registers)
    const uint32_t a0 = (tile + lane) ^ (32 * KK0), a1 = a0 ^ 32, a2 = a0 ^ 64, a3 = a1 ^ 64;
    if constexpr (N == 4)
      asm volatile("ds_read_b128 %0, %4 offset:%8\n\t"
                   "ds_read_b128 %1, %5 offset:%8\n\t"
                   "ds_read_b128 %2, %6 offset:%8\n\t"
                   "ds_read_b128 %3, %7 offset:%8\n\t"
                   "s_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[N - 2]), "=&v"(f[N - 1])
                   : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "i"(OFF)
                   : "memory");
    else
      asm volatile("ds_read_b128 %0, %2 offset:%4\n\t"
                   "ds_read_b128 %1, %3 offset:%4\n\t"
                   "s_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0]), "=&v"(f[1])
                   : "v"(a0), "v"(a1), "i"(OFF)
                   : "memory");
  }

  // operand row = head-dim index 32 t + lane%32.  Tile t reads chunk 4 t + (0..3), whose bits do not overlap, so its
  // addresses are those of t = 0 with 64 t flipped.
  struct FragT { uint32_t a0, a1; };
  static __device__ __forceinline__ FragT frag_t_init(int lane) {
    const int grp = lane >> 4, j = lane & 15;
    const int row = 8 * (grp >> 1) + (j >> 2);                       // + 16*kk (+4 for the second read)
    const int c = 2 * (grp & 1) + ((j & 3) >> 1);
    FragT f;
    f.a0 = (row * HD + ((c ^ swz(row)) << 3) + 4 * (j & 1)) * 2;
    f.a1 = ((row + 4) * HD + ((c ^ swz(row + 4)) << 3) + 4 * (j & 1)) * 2;
    return f;
  }
  // the N (2 or 4) operands of tile rows 16 (KK0 + i) .. + 15, i < N
  template <int N, int KK0>
  static __device__ __forceinline__ void read_t(uint32_t tile, const FragT &f, int t, bf16x8_t (&out)[N]) {
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    constexpr int RS = 16 * HD * 2;      // bytes of 16 rows
    const uint32_t a0 = (tile + KK0 * RS + f.a0) ^ (64 * t), a1 = (tile + KK0 * RS + f.a1) ^ (64 * t);
    u32x2 l[N], h[N];
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (N == 4) {
      asm volatile("ds_read_b64_tr_b16 %0, %8\n\t"
                   "ds_read_b64_tr_b16 %1, %9\n\t"
                   "ds_read_b64_tr_b16 %2, %8 offset:%10\n\t"
                   "ds_read_b64_tr_b16 %3, %9 offset:%10\n\t"
                   "ds_read_b64_tr_b16 %4, %8 offset:%11\n\t"
                   "ds_read_b64_tr_b16 %5, %9 offset:%11\n\t"
                   "ds_read_b64_tr_b16 %6, %8 offset:%12\n\t"
                   "ds_read_b64_tr_b16 %7, %9 offset:%12\n\t"
                   "s_waitcnt lgkmcnt(0)"
                   : "=&v"(l[0]), "=&v"(h[0]), "=&v"(l[1]), "=&v"(h[1]), "=&v"(l[2]), "=&v"(h[2]), "=&v"(l[3]), "=&v"(h[3])
                   : "v"(a0), "v"(a1), "i"(RS), "i"(2 * RS), "i"(3 * RS)
                   : "memory");
    } else {
      static_assert(N == 2, "two or four operands");
      asm volatile("ds_read_b64_tr_b16 %0, %4\n\t"
                   "ds_read_b64_tr_b16 %1, %5\n\t"
                   "ds_read_b64_tr_b16 %2, %4 offset:%6\n\t"
                   "ds_read_b64_tr_b16 %3, %5 offset:%6\n\t"
                   "s_waitcnt lgkmcnt(0)"
                   : "=&v"(l[0]), "=&v"(h[0]), "=&v"(l[1]), "=&v"(h[1])
                   : "v"(a0), "v"(a1), "i"(RS)
                   : "memory");
    }
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = __builtin_bit_cast(bf16x8_t, u32x4{l[i][0], l[i][1], h[i][0], h[i][1]});
  }
};

}  // namespace attn
