// Internal launch interface between the stage orchestration and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ah {

enum GemmLayout { GEMM_NN = 0, GEMM_NT = 1, GEMM_TN = 2 };
enum GemmEpilogue {
  EPI_BF16 = 0,      // C = acc (+ bias[n])
  EPI_GELU = 1,      // C = u = acc + bias[n];  C2 = gelu(u)
  EPI_RESID = 2,     // C = acc (+ bias[n]) + aux[m, n]
  EPI_GELU_BWD = 3,  // C = acc * gelu'(aux[m, n])
  EPI_F32_ACC = 4,   // C (fp32) = beta * C + acc  (callers use this one; beta selects the kernel)
  EPI_F32_SET = 5,   // C (fp32) = acc            (internal: EPI_F32_ACC with beta == 0)
  EPI_RESID_F32 = 6,        // C (fp32) = acc (+ bias[n]) + aux[m, n] (fp32): the residual stream kept in fp32
  EPI_RESID_F32_OUT16 = 7,  // C (bf16) = acc (+ bias[n]) + aux[m, n] (fp32): the last layer's output
  // NN only, B = [K, 2F] holding gate | up: the launch's N is 2F, every tile pairs gate columns with their up
  // columns; C[M, 2F] (ldc) = gate | up as bf16 (kept for backward), C2[M, F] (ldc2) = silu(gate) * up taken from
  // the fp32 accumulators.  No bias.  F = swiglu_F, a multiple of 128.
  EPI_SWIGLU = 8,
  // NT only, the input gradient of the SwiGLU block's second matrix with the activation's backward fused: with
  // dm = acc [M, F] and aux = gate | up [M, 2F] (ld_aux), C[M, 2F] (ldc) = dm up silu'(gate) | dm silu(gate).
  // N = F = swiglu_F; dm itself is not stored.
  EPI_SWIGLU_BWD = 9,
  // NN only, no bias: C = acc with the rotary embedding applied to columns [0, rope_cols) on the fp32 sums (heads of
  // rope_d columns, pairs (i, i + rope_d / 2), position = row % rope_S, table rope_cs[pos][i] = (cos, sin)).  Every
  // tile's wave strip must hold whole heads: launch_gemm takes such tiles only.
  EPI_ROPE = 10
};

constexpr int kMaxGemmSegments = 16;

struct GemmArgs {
  const void* A;     // NN/NT: [M, K] row-major;  TN: [K, M] row-major
  const void* B;     // NN/TN: [K, N] row-major;  NT: [N, K] row-major
  void* C;           // [M, N]
  void* C2;          // EPI_GELU second output
  const void* bias;  // [N] bf16 or NULL
  const void* aux;   // [M, N] bf16 (residual, or the pre-activation for EPI_GELU_BWD); fp32 for the _F32 residual epilogues
  int lda, ldb, ldc, ld_aux;
  int ldc2, swiglu_F;  // EPI_SWIGLU, EPI_SWIGLU_BWD
  const float* rope_cs;  // EPI_ROPE only
  int rope_S, rope_d, rope_cols;
  int M, N, K;
  int beta;
  int beside;          // kernels of another stream share the CUs: a launch of few tiles leaves them their LDS (same bits)
  int group, xcd_remap;  // tile rasterisation (set by launch_gemm; group 0: by the tile rows of the launch)
  // TN only: the k axis may be the concatenation of n_seg pieces of seg_k rows each (K = n_seg * seg_k), piece i
  // of A starting at segA[i] and of B at segB[i] (same leading dimensions).  n_seg == 0: one piece, A and B.
  int seg_k, n_seg;
  // TN only, optional: room for partial sums, with which launch_gemm may cut the k axis into k_shares parts (each a
  // whole number of pieces) that run side by side; their sums are added up by a second kernel.
  float* k_part;
  size_t k_part_floats;
  int k_shares;        // set by launch_gemm
  // EPI_GELU_BWD only, optional: column sums of the (bf16-rounded) output over each slab of 64 rows (or, in tiles of 192 rows, over
  // three ranges of rows that cover the tile) are written
  // to colsum_part[m / 64][n] (leading dimension ld_colsum), for the bias gradient.  Needs M % 64 == 0 (it is).
  float* colsum_part;
  int ld_colsum, colsum_acc;  // colsum_acc != 0: added to what is there
  const void* segA[kMaxGemmSegments];
  const void* segB[kMaxGemmSegments];
};

// M, N, K multiples of 128, all leading dimensions multiples of 8.
hipError_t launch_gemm(GemmLayout layout, GemmEpilogue epi, const GemmArgs& a, hipStream_t s);
bool gemm_shape_ok(int M, int N, int K);
// Weight gradients (GEMM_TN, EPI_F32_ACC) of the same K, pieces and beta in one launch.  gemm_group_tile: the tile to launch
// them with, or -1 where launches of their own are expected to be faster; it depends on the shapes alone.
constexpr int kMaxGemmGroup = 4;   // a layer's matrices
struct GemmShape { int M, N; };
int gemm_group_tile(const GemmShape* p, int n, int K, int n_seg, size_t part_floats);
hipError_t launch_gemm_group(int tile, const GemmArgs* p, int n, hipStream_t s);
bool gemm_rope_pays(int M, int N, int K, int rope_d, int rope_cols);  // EPI_ROPE can be had and beats EPI_BF16 and the rotary kernel
// A weight gradient's time by the launcher's model; of it, that of launches whose blocks leave room for others on their
// CUs, and of the other launches the share of the CUs that stays idle.
struct GemmTime { float us, room_us, idle_us; };
GemmTime gemm_wgrad_time(int M, int N, int K, int n_seg, size_t part_floats);
size_t gemm_k_part_floats(int M, int N, int K, int n_seg);  // what k_part should hold for a weight gradient over n_seg pieces (0: it would not be used)
// The launches that launch_gemm covers an output with: column ranges of cols[i], tiles of bm x bn whose waves take wgk
// shares of each k-block, walked in groups of `raster` tile rows, the k axis cut into `shares` parts between blocks.
// head: EPI_ROPE's head width (else 0).
struct GemmPlanInfo { int launches, shares, cols[2], bm[2], bn[2], wgk[2], raster[2]; };
bool gemm_plan(GemmLayout layout, int M, int N, int K, int n_seg, size_t part_floats, int head, GemmPlanInfo* out);
bool gemm_segments_ok(int seg_k, int n_seg);  // seg_k a positive multiple of 128, 1 <= n_seg <= kMaxGemmSegments

// ---- attention (d = 64 or 128, S multiple of 128) ----
// causal: query i attends to keys 0..i of its sequence; otherwise to all S keys
hipError_t launch_attention_fwd(const void* qkv, void* o, float* lse, int B, int S, int nh, int d, bool causal, hipStream_t s);
hipError_t launch_attention_bwd(const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv,
                                float* delta, int B, int S, int nh, int d, bool causal, hipStream_t s);

// ---- row-wise / element-wise kernels (bf16 I/O, fp32 math) ----
// a = norm(x) * gamma (+ beta); stats[2*T] = (mean, rstd) per row (RMS: mean slot unused = 0)
// x_f32: x is fp32 (the residual stream kept in fp32) instead of bf16
// keep, optional (x in bf16): a copy of x, in fp32 with keep_f32
hipError_t launch_norm_fwd(bool rms, const void* x, const void* gamma, const void* beta, void* a, float* stats,
                           int T, int h, float eps, hipStream_t s, bool x_f32 = false, void* keep = nullptr, bool keep_f32 = false);
// partial column sums of a bf16 matrix m[T, n] (n a multiple of 8) -> part[colsum_blocks(T)][n] (acc != 0: added to what is there)
struct ColsumJob { const void* m; float* part; int n, acc; };
hipError_t launch_colsum_partial(const ColsumJob& c, int T, hipStream_t s);
int colsum_blocks(int T);
// dx = dres + norm_bwd(da);  partial column sums of (da*xhat, da, dres) go to `part` ([3][nblk][h] fp32),
// written, or with acc != 0 added to what is there (a group of micro-batches sharing one set of partial sums)
// keep, optional: a copy of dres;  job, optional: column sums of a matrix of T rows that run beside it (the bits of launch_colsum_partial)
hipError_t launch_norm_bwd(bool rms, const void* da, const void* x, const float* stats, const void* gamma,
                           const void* dres, void* dx, float* part, int T, int h, hipStream_t s, int acc = 0, bool x_f32 = false, void* keep = nullptr,
                           const ColsumJob* job = nullptr);
int norm_bwd_blocks(int T);
// g[c] = beta * g[c] + sum_b part[b][c] for the vectors of a list (n a multiple of 64), in one launch
struct FoldList {
  static constexpr int kMax = 8;   // a layer's vector gradients
  const float* part[kMax];
  float* g[kMax];
  int n[kMax], nblk[kMax], first[kMax + 1], count;   // first: block of the launch at which a vector begins
  void add(const float* p, int blocks, int width, float* out) {
    if (count == 0) first[0] = 0;
    part[count] = p; nblk[count] = blocks; n[count] = width; g[count] = out;
    first[count + 1] = first[count] + width / 64;
    count++;
  }
  // the three arrays that a norm backward leaves in `p`
  void add3(const float* p, int blocks, int width, float* g0, float* g1, float* g2) {
    add(p, blocks, width, g0);
    add(p + (size_t)blocks * width, blocks, width, g1);
    add(p + (size_t)2 * blocks * width, blocks, width, g2);
  }
};
hipError_t launch_fold(const FoldList& a, int beta, hipStream_t s);
// rotary embedding in place on the Q and K blocks of qkv[T, 3*nh*d]; sign = +1 forward, -1 backward
hipError_t launch_rope(void* qkv, const float* cos_sin, int T, int S, int nh, int d, float sign, hipStream_t s);
// device-to-device copy of a multiple of 16 bytes
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);

}  // namespace ah
