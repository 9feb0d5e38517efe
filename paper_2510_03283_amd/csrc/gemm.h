// Grouped bf16 MFMA GEMM used by every dense contraction of the iteration.
#pragma once
#include "common.h"

// C[m, n] = sum_k A[m, k] * B[n, k]  (+ residual), over up to three row groups that share B and
// up to three column segments that share A.  Row groups let inference rows (one bf16 pass) and
// fine-tune rows (two- or three-pass split operands) ride in one launch; column segments let
// several weight matrices with separate base pointers (Wq|Wk|Wv, Wg|Wu) ride in one launch.
//
// Operand layouts (element type bf16):
//   LA = 0: A is [M, K] row-major (k contiguous).   LA = 1: A is [K, M] row-major (m contiguous).
//   LB = 0: B is [N, K] row-major (k contiguous).   LB = 1: B is [K, N] row-major (n contiguous).
// Requirements checked by gemm_launch: K % 64 == 0 for a k-contiguous operand; M % 8 == 0
// (N % 8 == 0) for an m- (n-) contiguous operand; all leading dimensions and column offsets
// multiples of 8 elements; pointers 16-byte aligned.
struct GemmMGroup {
  const bf16_t *a[2];   // [0] = hi (or only) operand, [1] = lo term (passes 2..)
  void *c;              // first output row of the group
  const void *resid;    // first residual row of the group (may be null)
  int M;                // rows in the group
  int npass;            // 1: A0*B0   2: + A1*B0   3: + A0*B1
  long long c_split_stride;   // elements between the partial results of two k slices (k_splits > 1)
  // SwiGLU mode only: c receives hm = silu(G) * U as bf16 [M, F]; c_lo (nullable) its second bf16
  // term; c_gu (nullable) G and U as bf16 [M, 2F] (G in columns [0,F), U in [F,2F)).
  void *c_lo;
  void *c_gu;
  // Rotary mode (NT form, four-wave kernel only - ask gemm_uses_four_wave first; head dimension 64 or 128): the rows
  // of this group are not written to c; every column segment writes its part as bf16 [M, N] (row stride N), rotated by the group's
  // angle table where the segment says so.  1 (fine-tune rows): two terms into its rope_hi / rope_lo.  2 (inference rows): one term into
  // its rope_inf, and into its rope_cache (nullable) at the rows' slots.
  int rope;
};
struct GemmNSeg {
  const bf16_t *b[2];   // [0] = hi (or only) operand, [1] = lo term (pass 3)
  int N;                // columns in the segment
  int c_col;            // first output column of the segment
  // rotary mode (row groups with rope != 0): outputs of this segment and whether its heads are rotated (Q, K) or
  // only split into two terms (V)
  void *rope_hi, *rope_lo, *rope_inf, *rope_cache;
  int rope_rot;
};
struct GemmParams {
  GemmMGroup mg[3];
  GemmNSeg ns[3];
  int n_mg, n_ns;
  int K;
  long long lda, ldb, ldc, ldr;
  int out_bf16;     // 0: C is fp32, 1: C is bf16
  int resid_kind;   // 0 none, 1 fp32, 2 bf16 ; C = acc + resid
  // K segments (optional, n_kseg > 1; needs n_ns == 1 and one pass): the k range is a concatenation
  // and segment s (k in [kseg_start[s], kseg_start[s+1]), boundaries multiples of 64) takes its B
  // rows from kseg_b[s] instead of ns[0].b[0] - several weight matrices stacked along the reduction
  // (dX = dQ Wq + dK Wk + dV Wv as one product).
  int n_kseg;
  const bf16_t *kseg_b[3];
  int kseg_start[4];
  // SwiGLU mode (NT form only): ns[0] = gate weights, ns[1] = up weights, both [F, K]; every wave
  // multiplies 32 gate columns and the 32 up columns of the same hidden units, and the epilogue
  // writes silu(G) * U instead of G and U (ldc = F).
  int swiglu;
  // k slices of the tiles of every row group, 1 = none (0 counts as 1).  More than one (four-wave kernel, fp32 output, no
  // residual - see gemm_pick_splits): slice z writes its partial sums at c + z * c_split_stride of the group, for a
  // consumer that adds them in order.
  int k_splits[3];
  int mt_start[4];  // filled by gemm_launch
  int nt_start[4];
  int tile_m, tile_n;   // filled by gemm_launch: the block tile its cost model chose
  // SwiGLU backward mode (NN form, four-wave kernel only - ask gemm_uses_four_wave first): the product is dHm [M, N = F];
  // instead of it the epilogue writes dG | dU as bf16 [M, 2F] into c (ldc = 2F) from G | U of the forward, bf16 [M, 2F]
  // in c_gu (read only): dG = dHm U s (1 + G (1 - s)), dU = dHm G s, s = sigmoid(G).
  int swiglu_bwd;
  // rotary mode: (cos, sin) of row r of a rope group and pair index i at [2 (rope_hd / 2 * r + i)], by kind of group; the paged cache
  // [blocks, rope_hkv, 1 << rope_bshift, rope_hd] and the rows' slots in it (one outside 0 .. rope_num_slots - 1 is skipped)
  const float *rope_cs, *rope_cs_inf;
  const int32_t *rope_slots;
  long long rope_num_slots;
  int rope_hd, rope_hkv, rope_bshift;
  int force_w4;     // 1: the 256x256 four-wave kernel whatever the cost model says (rejected if the problem does not fit it)
};

// Whether cutting the reduction of a product into slices pays.  base: the product as it would be launched otherwise
// (with its fused epilogue, bf16 output or residual); plain: the same product with plain fp32 output, as the slices
// would write it for a consumer that adds them (c and ldc as for one slice; only sizes are read).  part_floats: room for
// the partial results; extra_us: what the consumer costs beyond the consumer of `base` (a launch).  On true k_splits
// holds the slices of every row group.  Products that leave CUs idle or whose last round of tiles is nearly empty
// gain; priced with product_us in gemm.hip plus the traffic of the partial results.
bool gemm_pick_splits(int LA, int LB, const GemmParams &base, const GemmParams &plain, size_t part_floats, double extra_us, int k_splits[3]);

// Whether gemm_launch would run this problem on the four-wave kernel (its cost model picks the 256x256 tile, or
// force_w4 is set, and the problem fits the kernel).  Forms that only that kernel has are launched after asking.
bool gemm_uses_four_wave(int LA, int LB, const GemmParams &p);

// About how long the product takes on an otherwise idle GPU, microseconds.
double gemm_estimate_us(int LA, int LB, const GemmParams &p);

// Returns hipSuccess or the launch error; a non-null *why is set on a rejected shape.
hipError_t gemm_launch(int LA, int LB, GemmParams &p, hipStream_t stream, const char **why);
