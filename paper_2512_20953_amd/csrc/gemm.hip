// bf16 GEMM for gfx950: MFMA 16x16x32 (32x32x16 in the smallest tiles), fp32 accumulators, tiles staged through
// LDS by direct global->LDS loads (16 B per lane) through a ring of operand tiles.
//
// Three operand layouts cover the linear layers of a decoder layer (the GEMM is
// the core of the stage's time, paper Section II-B):
//   NN  y  = x W        (forward)            A[M,K] k-contiguous, B[K,N] k-strided
//   NT  dx = dy W^T     (input gradient)     A[M,K], B[N,K] both k-contiguous
//   TN  dW += x^T dy    (weight gradient)    A[K,M], B[K,N] both k-strided
// A k-contiguous operand is read from LDS with 16-byte reads; a k-strided one
// with the transposing 8-byte LDS read, so no transposed copy is ever made.
//
// Work split: 256 threads = 4 waves in a 2 x 2 grid; each wave owns a
// (BM/2) x (BN/2) sub-tile as 16 x 16 MFMA blocks (in the smallest tiles the
// waves share a sub-tile of 32 x 32 blocks and split the k axis).  The MFMA is issued with the
// operands swapped (D = B^T A^T) so that a lane ends up with 4 consecutive
// columns of one output row: 8-byte bf16 or 16-byte fp32 accesses in the epilogue.
#include "common.h"
#include "kernels.h"
#include <algorithm>
#include <cstdlib>
#include <mutex>
#include <type_traits>
#include <vector>

namespace ah {

// Three pipelines share the tile mapping, the LDS layouts, the fragment reads and the epilogue.  The forward and
// input-gradient products (at least one k-contiguous operand) use 64-wide k tiles in a ring of operand
// buffers, so that every loader instruction fetches whole 128-byte lines of the k-contiguous operand; the weight
// gradient (both operands k-strided, rows of a tile are 256 or 512 bytes anyway) keeps 32-wide k stages in a ring of
// four, whose loads all run three stages ahead.  Measured in the stage: the first is 2-13 % faster on the former
// products, the second 1-5 % faster on the latter.  The third is that of the smallest tiles (namespace ksplit).

// ---------------------------------------------------------------------------
// LDS layouts, for a tile of BK = 64 or 32 k-values (all permutations are of 16-byte pieces, the unit of the loader)
//  k-contiguous tile: [rows][BK k]; row = 2 BK bytes = BK/8 pieces; piece p of row r is stored at piece
//    p ^ ((r >> 1) & 7) (BK = 64) or p ^ ((r >> 2) & 3) (BK = 32): 16 consecutive rows hit 16 distinct 16-byte bank
//    groups for the fragment reads.  With BK = 64 a loader instruction fetches 8 rows x 128 B: full cache lines
//    (64-byte row pieces, as BK = 32 gives, cost the memory pipeline twice the requests and showed up as ~10 % of
//    MFMA utilisation where an operand is k-contiguous).
//  k-strided tile: [BK k][W cols]; row = 2W bytes.  Half a wave must cover all banks once in a transposing read.  For fragments
//    of 16 columns x 32 k it fetches 8 rows (k .. k + 3 and k + 8 .. k + 11) x 32 B: the 32-byte granule g of row k is stored at
//    granule g ^ (k & 3 | (k >> 1) & 4).  For those of 32 columns x 16 k (the smallest tiles) 4 rows x 64 B: the 64-byte granule g of row
//    k at g ^ (k & 3) (W = 64, two granules: g ^ (k >> 1 & 1)).
// A k-strided tile may gather its columns from two column ranges of the matrix (`gw` > 0: tile columns in groups of
// gw, even groups from columns c, odd groups from columns F + c): the fused gate|up product of the SwiGLU block then
// has a gate column and its up column in the same wave's accumulators.
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ int granule_swizzle(int k) {  // a 64-wide row has two granules only: 4 rows x 64 B then span two bank cycles
  static_assert(W >= 64, "a row holds whole granules");
  return W >= 128 ? k & 3 : (k >> 1) & 1;
}

template <int W>
__device__ __forceinline__ int granule32_swizzle(int k) {  // of 32-byte granules
  // rows start 0, 128 (W = 192) or 64 (W = 160) bytes further along the banks than the one before
  static_assert(W % 128 == 0 || W == 192 || W == 160, "where a row begins among the banks");
  if (W % 128 == 64) return (k & 2) | ((k >> 3) & 1);
  if (W % 128 == 32) return (k >> 3) & 1;
  return (k & 3) | ((k >> 1) & 4);
}

// K16: the tile's fragments are 32 columns x 16 k
template <int BK, int W, bool KS, bool K16 = false>
__device__ __forceinline__ uint32_t loader_src_offset(int chunk, int lane, int ld, int gw = 0, int F = 0) {  // in bytes
  const int pos = chunk * 1024 + lane * 16;
  if (!KS) {
    constexpr int PR = BK / 8;                 // pieces per row
    constexpr int SH = BK == 64 ? 1 : 2;
    const int r = pos / (2 * BK), q = (pos >> 4) & (PR - 1);
    const int p = q ^ ((r >> SH) & (PR - 1));
    return (uint32_t)(r * ld + p * 8) * 2u;
  } else {
    constexpr int RB = W * 2;
    const int k = pos / RB, q = (pos % RB) >> 4;
    int p;
    if constexpr (K16) p = q ^ (granule_swizzle<W>(k) << 2);
    else p = q ^ (granule32_swizzle<W>(k) << 1);
    int col = p * 8;
    if (gw > 0) col = ((col / gw) & 1) * F + (col / (2 * gw)) * gw + col % gw;
    return (uint32_t)(k * ld + col) * 2u;
  }
}

// a W x BK (or BK x W) tile is W * BK / 512 chunks of 1 KB; wave w moves chunks w, w + NW, ...
template <int BK, int W, int NW>
__device__ __forceinline__ void issue_tile_loads(const char* __restrict__ g, uint32_t* off, char* __restrict__ lds, int wave) {
#pragma unroll
  for (int i = 0; i < W * BK / 512 / NW; i++) load16_to_lds(g, off[i], lds + (wave + NW * i) * 1024);
}

// fragment (8 k-values for row/col = lane % 32 of a 32-wide block) for k-step ks (16 k each)
template <int BK, int W, bool KS>
__device__ __forceinline__ bf16x8 read_frag(const char* __restrict__ lds, int base, int blk, int ks, int lane) {
  if (!KS) {
    constexpr int PR = BK / 8;
    constexpr int SH = BK == 64 ? 1 : 2;
    const int r = base + blk * 32 + (lane & 31);
    const int p = ks * 2 + (lane >> 5);
    const int q = p ^ ((r >> SH) & (PR - 1));
    return *(const bf16x8*)(lds + r * (2 * BK) + q * 16);
  } else {
    constexpr int RB = W * 2;
    const int k = ks * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
    const int c = base + blk * 32 + ((lane >> 4) & 1) * 16 + 4 * (lane & 3);
    const int a0 = k * RB + (((c >> 5) ^ granule_swizzle<W>(k)) << 6) + ((c * 2) & 63);
    bf16x4 lo = lds_read_tr4(lds + a0);
    bf16x4 hi = lds_read_tr4(lds + a0 + 4 * RB);
    return cat4(lo, hi);
  }
}

// fragment (8 k-values for row/col = lane % 16 of a 16-wide block) for k-step ks (32 k each)
template <int BK, int W, bool KS>
__device__ __forceinline__ bf16x8 read_frag32(const char* __restrict__ lds, int base, int blk, int ks, int lane) {
  if (!KS) {
    constexpr int PR = BK / 8;
    constexpr int SH = BK == 64 ? 1 : 2;
    const int r = base + blk * 16 + (lane & 15);
    const int p = ks * 4 + (lane >> 4);
    const int q = p ^ ((r >> SH) & (PR - 1));
    return *(const bf16x8*)(lds + r * (2 * BK) + q * 16);
  } else {
    constexpr int RB = W * 2;
    const int k = ks * 32 + (lane >> 4) * 8 + ((lane & 15) >> 2);
    const int c = base + blk * 16 + 4 * (lane & 3);
    const int a0 = k * RB + (((c >> 4) ^ granule32_swizzle<W>(k)) << 5) + ((c * 2) & 31);
    bf16x4 lo = lds_read_tr4(lds + a0);
    bf16x4 hi = lds_read_tr4(lds + a0 + 4 * RB);
    return cat4(lo, hi);
  }
}

// Fragments of one 32-wide k-step for the wave's sub-tile.
template <int BK, int BM, int BN, int WGM, int WGN, bool AKS, bool BKS>
struct Frags32 {
  static constexpr int TM = BM / WGM / 16, TN = BN / WGN / 16;
  bf16x8 a[TM], b[TN];
  __device__ __forceinline__ void load(const char* __restrict__ cA, const char* __restrict__ cB, int ks, int wm, int wn, int lane) {
#pragma unroll
    for (int t = 0; t < TM; t++) a[t] = read_frag32<BK, BM, AKS>(cA, wm * (BM / WGM), t, ks, lane);
#pragma unroll
    for (int t = 0; t < TN; t++) b[t] = read_frag32<BK, BN, BKS>(cB, wn * (BN / WGN), t, ks, lane);
  }
};

// Fragments of one 16-wide k-step for the wave's sub-tile.
template <int BK, int BM, int BN, int WGM, int WGN, bool AKS, bool BKS>
struct Frags {
  static constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
  bf16x8 a[TM], b[TN];
  __device__ __forceinline__ void load(const char* __restrict__ cA, const char* __restrict__ cB, int ks, int wm, int wn, int lane) {
#pragma unroll
    for (int t = 0; t < TM; t++) a[t] = read_frag<BK, BM, AKS>(cA, wm * (BM / WGM), t, ks, lane);
#pragma unroll
    for (int t = 0; t < TN; t++) b[t] = read_frag<BK, BN, BKS>(cB, wn * (BN / WGN), t, ks, lane);
  }
};

// Scheduling hint for one k-step: between consecutive MFMAs (NM of them) place
// the NV global->LDS loads and the NR LDS reads issued for later steps, the LDS
// reads within the first three quarters so their latency is covered by the rest.
// Masks: 0x020 = vector memory read, 0x100 = LDS read, 0x008 = MFMA.
template <int I, int NM, int NR, int NV, int SPAN = (NM * 3 / 4 > 0 ? NM * 3 / 4 : 1)>
__device__ __forceinline__ void interleave() {
  if constexpr (I < NM) {
    constexpr int v = (I + 1) * NV / NM - I * NV / NM;
    constexpr int r = I < SPAN ? (I + 1) * NR / SPAN - I * NR / SPAN : 0;
    if constexpr (v > 0) __builtin_amdgcn_sched_group_barrier(0x020, v, 0);
    if constexpr (r > 0) __builtin_amdgcn_sched_group_barrier(0x100, r, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    interleave<I + 1, NM, NR, NV, SPAN>();
  }
}

template <int BK, int BM, int BN, int WGM, int WGN, bool AKS, bool BKS>
__device__ __forceinline__ void mma_step(const Frags<BK, BM, BN, WGM, WGN, AKS, BKS>& f, f32x16 (&acc)[BM / WGM / 32][BN / WGN / 32]) {
  constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
#pragma unroll
  for (int tm = 0; tm < TM; tm++)
#pragma unroll
    for (int tn = 0; tn < TN; tn++)
      acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[tn], f.a[tm], acc[tm][tn], 0, 0, 0);
}

// The 16 x 16 x 32 instruction does the flops of the 32 x 32 x 16 one at less power, which is what bounds a loop that keeps the matrix
// pipelines busy: register-resident on random operands 2.06 against 1.78 PFLOP/s (2.44 both on zeros).  In the loops below, with
// the same bytes through LDS: 8192^3 NT 847 -> 811 us, 2048 x 5120 x 20480 394 -> 372, 2048^3 (128 x 128 tiles) 23.2 -> 20.5.
// As assembly, because the compiler's form has a destination of its own: with all 256 accumulation registers taken it
// moves 12 .. 60 of 64 accumulators to other registers and back in every k-step.  What the compiler then does not know of is
// kept here: an accumulator is used again one k-step (16 or more matrix instructions) later, and read 16 wait states
// after the loops (gemm_tile); operands come from LDS reads, which it does wait for.
__device__ __forceinline__ void mma16(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}

// One 32-wide k-step as a fixed sequence of slots: a matrix instruction on the fragments f each, and before it what falls on the slot
// of the NV loads (load(i)) and of the reads of the next step's fragments fn, which take the first three quarters (in the first
// 3, 4 or 8 eighths 1.005, 1.004 and 1.014 times as long, geometric mean over 56 products).  The loads of a short step, and those
// of the weight gradient, whose operands come from far away, go out in its first half: 4096 x 1024 x 4096 36.3 -> 35.0 us (NT), 2048^3
// 22.9 -> 22.1 (NN), 4096^3 111.8 -> 109.9 (TN); evenly they are 1 % better in the larger forward and input-gradient steps.
// In the weight gradient's short steps (TN, up to 32 matrix instructions) the reads, two to a fragment, take all slots but the last two: beside the loads
// the first three quarters made a wave that is alone on its SIMD wait for them.  Launches of up to a tile per CU, against the 32x32x16 loop that was
// here before (geometric means, three boxes): 128 x 256 and 256 x 128 1.04 -> 0.98 .. 1.00, 128 x 128 1.03 -> 1.01; 3840 x 1152 x 5120 51.8 us there, 57.1 -> 53.6 here.
template <int BK, int BM, int BN, int WGM, int WGN, bool AKS, bool BKS, int NV, class L>
__device__ __forceinline__ void k_step(const L& load, const char* __restrict__ nA, const char* __restrict__ nB, int ks,
                                       const Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& f, Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& fn,
                                       f32x4 (&acc)[BM / WGM / 16][BN / WGN / 16], int wm, int wn, int lane) {
  constexpr int TM = BM / WGM / 16, TN = BN / WGN / 16, NM = TM * TN, NF = TM + TN, SPAN = AKS && BKS && NM <= 32 ? NM - 2 : NM * 3 / 4;
  constexpr int VSPAN = (AKS && BKS) || NM <= 16 ? NM / 2 : NM;
#pragma unroll
  for (int i = 0; i < NM; i++) {
#pragma unroll
    for (int v = i * NV / VSPAN; v < (i + 1) * NV / VSPAN && v < NV; v++) load(v);
#pragma unroll
    for (int r = i * NF / SPAN; r < (i + 1) * NF / SPAN && r < NF; r++) {
      if (r < TN) fn.b[r] = read_frag32<BK, BN, BKS>(nB, wn * (BN / WGN), r, ks, lane);
      else fn.a[r - TN] = read_frag32<BK, BM, AKS>(nA, wm * (BM / WGM), r - TN, ks, lane);
    }
    mma16(acc[i / TN][i % TN], f.a[i / TN], f.b[i % TN]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

namespace k64 {
constexpr int BK = 64;  // k-extent of one operand tile in LDS (128 bytes per row of a k-contiguous operand: whole cache lines)
// DEPTH: k-blocks between the start of the second operand's loads and the wait for them (the first operand's: half a block more), for
// which the ring has DEPTH + 1 buffers for tiles of the first and DEPTH for those of the second.
//  256 x 256 tiles: 2, all of a CU's 160 KB.  128 x 256 and 256 x 128: 3, the same.
//  128 x 128: 2 where two blocks share a CU (80 KB).  In a launch of at most 256 blocks, which have a CU each, 3 (112 KB): a k-block
//    is 512 clocks of MFMA, and with 2 the loop waited for operands that come from HBM.  4096 x 1024 x 4096 49.4 -> 39.7 us from HBM,
//    33.7 -> 32.9 from the memory-side cache (NN); 2048^3 28.1 -> 23.0 and 20.8 -> 19.3 (NT); 4 is no better (40.3, 23.4).  Beside a
//    second stream (GemmArgs::beside) it keeps that stream's blocks off the CUs: BERT-Large stage with a group of 1, 1892 -> 1992 us.
template <int BM, int BN, int DEPTH, bool BF>
constexpr int ring_bytes() { return ((DEPTH + 1) * (BF ? BN : BM) + DEPTH * (BF ? BM : BN)) * 2 * BK; }

// The pipeline.  F is the operand whose tiles go first, S the other one (see b_first); the tiles of k-block j are F_j and S_j.
// A k-block is two k-steps of 32; fragments are double-buffered in registers (f0, f1), the fragments
// of a k-step being read from LDS under the MFMAs of the step before.  So all fragments of k-block j are in registers at its
// middle: there the one barrier per k-block frees its two buffers, and, after a wait that counts the wave's own loads down to the
// tiles issued after S_{j+1}, says that k-block j+1 has landed for the whole block.  The second half of k-block j starts the loads of
// S_{j + DEPTH} into the buffer of S_j, the first half those of F_{j + DEPTH} into that of F_{j-1}.
// The two halves are separate functions so that within each the buffer written is not one of the buffers read:
// the restrict qualifiers then tell the compiler that LDS reads never wait for the loads in flight.

// F has the longer way to go.  The weights (B of the forward and input-gradient products) stream from HBM while
// the activations were just written and mostly sit in the caches, so B goes first, unless its tiles are the larger ones, of which
// the ring has no room for one more.
template <int BM, int BN, bool AKS>
constexpr bool b_first() { return !AKS && BN <= BM; }

// First k-step of k-block j (f0 holds its fragments): starts the loads of F_{j + DEPTH} and reads the
// fragments of the second one.
template <int BM, int BN, int WGM, int WGN, bool AKS, bool BKS>
__device__ __forceinline__ void half_even(const char* gF, uint32_t* offF, char* __restrict__ fill, const char* __restrict__ cA,
                                          const char* __restrict__ cB, const Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& f0,
                                          Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& f1, f32x4 (&acc)[BM / WGM / 16][BN / WGN / 16],
                                          int wave, int wm, int wn, int lane) {
  constexpr int NW = WGM * WGN, WF = b_first<BM, BN, AKS>() ? BN : BM;
  k_step<BK, BM, BN, WGM, WGN, AKS, BKS, WF / 8 / NW>([&](int i) { load16_to_lds(gF, offF[i], fill + (wave + NW * i) * 1024); }, cA, cB, 1, f0, f1,
                                                      acc, wm, wn, lane);
}

// Second k-step of k-block j: waits for k-block j+1 (nA, nB), starts the loads of S_{j + DEPTH} into the buffer of S_j, whose
// fragments all waves hold by now, and reads the first fragments of k-block j+1.
template <int BM, int BN, int WGM, int WGN, bool AKS, bool BKS, int DEPTH>
__device__ __forceinline__ void half_odd(const char* gS, uint32_t* offS, char* __restrict__ fill, const char* __restrict__ nA,
                                         const char* __restrict__ nB, Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& f0,
                                         const Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& f1, f32x4 (&acc)[BM / WGM / 16][BN / WGN / 16],
                                         int wave, int wm, int wn, int lane) {
  constexpr int NW = WGM * WGN, WF = b_first<BM, BN, AKS>() ? BN : BM, WS = b_first<BM, BN, AKS>() ? BM : BN;
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(((DEPTH - 1) * WF + (DEPTH - 2) * WS) / 8 / NW));
  __builtin_amdgcn_s_barrier();
  k_step<BK, BM, BN, WGM, WGN, AKS, BKS, WS / 8 / NW>([&](int i) { load16_to_lds(gS, offS[i], fill + (wave + NW * i) * 1024); }, nA, nB, 0, f1, f0,
                                                      acc, wm, wn, lane);
}

}  // namespace k64

namespace k32 {
constexpr int BK = 32;  // k-extent of one LDS stage (64 bytes of bf16)
constexpr int NS = 4;   // stages in the LDS ring: loads run 3 stages ahead of the MFMAs

// One stage (32 of k) of the pipeline; on entry f holds its fragments.  Waits until the next stage (nA, nB) has landed for the
// whole block (own loads by count: two later stages may stay in flight; then the barrier), starts the loads of the stage four
// ahead into this stage's slot (fA, fB), which every wave has read out, and reads the next stage's fragments into fn under the
// MFMAs.  The restrict qualifiers tell the compiler that the two slots are distinct, so LDS reads never wait for the loads in flight.
template <int BM, int BN, int WGM, int WGN, bool AKS, bool BKS>
__device__ __forceinline__ void ring_step(const char* gA, const char* gB, uint32_t* offA, uint32_t* offB,
                                          char* __restrict__ fA, char* __restrict__ fB, const char* __restrict__ nA, const char* __restrict__ nB,
                                          const Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& f, Frags32<BK, BM, BN, WGM, WGN, AKS, BKS>& fn,
                                          f32x4 (&acc)[BM / WGM / 16][BN / WGN / 16], int wave, int wm, int wn, int lane) {
  constexpr int NW = WGM * WGN, LA = BM / 16 / NW, LPS = (BM + BN) / 16 / NW;  // loads per stage per wave
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(2 * LPS));
  __builtin_amdgcn_s_barrier();
  k_step<BK, BM, BN, WGM, WGN, AKS, BKS, LPS>(
      [&](int i) {
        if (i < LA) load16_to_lds(gA, offA[i], fA + (wave + NW * i) * 1024);
        else load16_to_lds(gB, offB[i - LA], fB + (wave + NW * (i - LA)) * 1024);
      },
      nA, nB, 0, f, fn, acc, wm, wn, lane);
}

}  // namespace k32

namespace ksplit {
// The pipeline of the tiles whose waves share a sub-tile and split the k axis: of the four k-steps of a 64-wide
// k-block, wave wk takes 4 / WGK.  The partial sums meet in the epilogue's staging strips.
//  64 x 64 with four shares and 64 x 128 with two are for outputs of fewer than 256 tiles of 128 x 128.  Such a launch
//    lasts as long as one block's chain of k-blocks; these have four (two) times the blocks, and a chain a quarter as
//    long.  256 x 256 x 1024: 9.3 -> 5.5 us, 1024 x 1024 x 2048: 21.6 -> 8.8, 2048 x 1024 x 2048: 21.6 -> 13.2 (NT).
//  128 x 128 with four shares: every wave owns the whole tile, so a k-block costs 32 KB of fragment reads instead of
//    the 64 KB of four 64 x 64 sub-tiles.  Beside 512 clocks of MFMA the CU's path to and from the LDS was busy ~950
//    (reads at 128 B per clock, the 32 KB fill at 1.7 times its bytes), now ~690; what bounds it then is the rate at
//    which the loads arrive (64 B per clock and CU).  2048 x 2048 x 8192: 76 -> 61 us (NT; against the 32x32x16 loop:
//    the present one has closed the gap, see kWholeCuMinK, and the tile is there for its shorter sums).  The epilogue moves four
//    times the partial sums (3 us): at k = 2048 the two are level, and where two blocks of the 64 x 64 sub-tiles share
//    a CU (more than 256 tiles) those are faster; in the weight gradient, whose transposing reads are half as long,
//    there is no gain (67 against 67 us), so it is not built there.
constexpr int BK = 64;
template <int BM, int BN> constexpr int stage_bytes() { return (BM + BN) * 2 * BK; }
// ring depth: all of a CU's 160 KB for the 128 x 128 tile, half of it for the small ones (two blocks share a CU): 5, 3 and 5 stages
template <int BM, int BN> constexpr int stages() { return (BM * BN < 128 * 128 ? 81920 : 163840) / stage_bytes<BM, BN>(); }

// Second (or only) part of a k-block: the block's slot is free (its fragments are in registers, the barrier is
// passed), so the loads of the stage NS ahead go there while the next stage's first fragments are read.  The two
// slots are distinct: the restrict qualifiers keep the LDS reads from waiting for the loads in flight.
template <int BM, int BN, int WGM, int WGN, bool AKS, bool BKS>
__device__ __forceinline__ void last_step(const char* pA, const char* pB, uint32_t* offA, uint32_t* offB, char* __restrict__ fill,
                                          const char* __restrict__ next, int ks, const Frags<BK, BM, BN, WGM, WGN, AKS, BKS>& f,
                                          Frags<BK, BM, BN, WGM, WGN, AKS, BKS>& fn, f32x16 (&acc)[BM / WGM / 32][BN / WGN / 32], int wave,
                                          int wm, int wn, int lane) {
  constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32, NW = 4;
  constexpr int NR = TM * (AKS ? 2 : 1) + TN * (BKS ? 2 : 1), NM = TM * TN, LPS = (BM + BN) / 8 / NW;
  issue_tile_loads<BK, BM, NW>(pA, offA, fill, wave);
  issue_tile_loads<BK, BN, NW>(pB, offB, fill + BM * 2 * BK, wave);
  fn.load(next, next + BM * 2 * BK, ks, wm, wn, lane);
  mma_step<BK, BM, BN, WGM, WGN, AKS, BKS>(f, acc);
  interleave<0, NM, NR, LPS, NM / 2>();
}

// First part of a two-step k-block
template <int BM, int BN, int WGM, int WGN, bool AKS, bool BKS>
__device__ __forceinline__ void first_step(const char* __restrict__ cur, int ks, const Frags<BK, BM, BN, WGM, WGN, AKS, BKS>& f,
                                           Frags<BK, BM, BN, WGM, WGN, AKS, BKS>& fn, f32x16 (&acc)[BM / WGM / 32][BN / WGN / 32], int wm,
                                           int wn, int lane) {
  constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32;
  constexpr int NR = TM * (AKS ? 2 : 1) + TN * (BKS ? 2 : 1), NM = TM * TN;
  fn.load(cur, cur + BM * 2 * BK, ks, wm, wn, lane);
  mma_step<BK, BM, BN, WGM, WGN, AKS, BKS>(f, acc);
  interleave<0, NM, NR, 0, NM / 2>();
}

}  // namespace ksplit

// One tile of a product: block `block` of the (M / BM) (N / BN) k_shares that cover it.
template <int BM, int BN, int WGM, int WGN, int WGK, bool AKS, bool BKS, int EPI, int DEPTH = 2>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, int block) {
  constexpr int TM = BM / WGM / 32, TN = BN / WGN / 32, NW = WGM * WGN * WGK;
  static_assert(NW == 4, "four waves per block");
  constexpr bool SPLIT = WGK > 1;                // which pipeline
  constexpr bool K32 = !SPLIT && AKS && BKS;
  // EPI_SWIGLU: the B tile gathers GW gate columns and their GW up columns per wave (see loader_src_offset); the
  // launch runs over N = 2 F tile columns that stand for F logical ones.
  constexpr bool SWIGLU = EPI == EPI_SWIGLU;
  constexpr int GW = SWIGLU ? BN / WGN / 2 : 0;
  static_assert(!SWIGLU || (!AKS && BKS), "the fused SwiGLU epilogue belongs to the forward layout");
  constexpr int RING = SPLIT ? ksplit::stages<BM, BN>() * ksplit::stage_bytes<BM, BN>() : K32 ? k32::NS * (BM + BN) * 64
                           : k64::ring_bytes<BM, BN, DEPTH, k64::b_first<BM, BN, AKS>()>();
  // the epilogue reuses the ring as staging space
  __shared__ __attribute__((aligned(1024))) char ring[RING];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps LDS bases in scalar registers
  const int wmn = wave / WGK, wk = wave % WGK;   // output sub-tile, share of the k axis
  const int wm = wmn / WGN, wn = wmn % WGN;

  // block -> tile: consecutive logical tiles share an XCD (blocks are dealt to the
  // 8 XCDs round-robin), and run down groups of about 4 tile-rows (raster_rows) so that the 32 tiles in
  // flight on one XCD reuse the same operand panels in its L2.
  // With the k axis shared by blocks (kernels.h) the shares follow each other: an XCD then works on one share's operands.
  constexpr bool KSHARES = AKS && BKS && EPI == EPI_F32_SET;
  const int shares = KSHARES ? g.k_shares : 1;
  const int tiles_m = g.M / BM, tiles_n = g.N / BN, out_tiles = tiles_m * tiles_n, ntiles = out_tiles * shares;
  // (Where the count is not a multiple of 8 the first ntiles % 8 XCDs take one tile more.)
  int logical = block;
  if (g.xcd_remap) logical = (block & 7) * (ntiles >> 3) + min(block & 7, ntiles & 7) + (block >> 3);
  const int share = KSHARES ? logical / out_tiles : 0;
  if (KSHARES) logical -= share * out_tiles;
  const int GROUP = g.group;
  const int per_group = GROUP * tiles_n;
  const int gid = logical / per_group;
  const int first_m = gid * GROUP;
  const int gsize = min(tiles_m - first_m, GROUP);
  const int in_group = logical - gid * per_group;
  const int m0 = (first_m + in_group % gsize) * BM;
  const int n0 = (in_group / gsize) * BN;

  const char* gA = (const char*)((const bf16*)g.A + (AKS ? (size_t)m0 : (size_t)m0 * g.lda));
  const char* gB = (const char*)((const bf16*)g.B + (BKS ? (size_t)(SWIGLU ? n0 / 2 : n0) : (size_t)n0 * g.ldb));
  // The block's part of the k axis: all of it, or share `share`, a whole number of its pieces (of its k-blocks where
  // it is one piece).
  const int kext = KSHARES ? g.K / shares : g.K;
  const int pieces = (AKS && BKS) ? (KSHARES && g.n_seg > 1 ? g.n_seg / shares : max(g.n_seg, 1)) : 1;
  const int piece0 = KSHARES && g.n_seg > 1 ? share * pieces : 0;
  if constexpr (KSHARES) {
    const size_t k0 = g.n_seg > 1 ? 0 : (size_t)share * kext;
    gA = (const char*)((const bf16*)g.segA[piece0] + m0 + k0 * g.lda);
    gB = (const char*)((const bf16*)g.segB[piece0] + n0 + k0 * g.ldb);
  }
  // SPLIT: blocks of 32 x 32, otherwise of 16 x 16
  using Acc = std::conditional_t<SPLIT, f32x16, f32x4>;
  constexpr int AB = SPLIT ? 32 : 16;
  Acc acc[BM / WGM / AB][BN / WGN / AB];
#pragma unroll
  for (int i = 0; i < BM / WGM / AB; i++)
#pragma unroll
    for (int j = 0; j < BN / WGN / AB; j++)
#pragma unroll
      for (int r = 0; r < AB * AB / 64; r++) acc[i][j][r] = 0.f;

  if constexpr (SPLIT) {
    using namespace ksplit;
    constexpr int STAGE = stage_bytes<BM, BN>(), NS = stages<BM, BN>(), KPW = 4 / WGK, LA = BM / 8 / NW, LB = BN / 8 / NW, LPS = LA + LB;
    const size_t stepA = (AKS ? (size_t)BK * g.lda : (size_t)BK) * 2;  // bytes per k-block
    const size_t stepB = (BKS ? (size_t)BK * g.ldb : (size_t)BK) * 2;
    uint32_t offA[LA], offB[LB];
#pragma unroll
    for (int i = 0; i < LA; i++) offA[i] = loader_src_offset<BK, BM, AKS, true>(wave + NW * i, lane, g.lda);
#pragma unroll
    for (int i = 0; i < LB; i++) offB[i] = loader_src_offset<BK, BN, BKS, true>(wave + NW * i, lane, g.ldb, GW, g.swiglu_F);
    // The stage to be fetched next: pA, pB, moved on by scalar selects (a branch per stage would cut the loop into
    // basic blocks).  Past the last stage it stays there: that stage is fetched again into dead slots, which keeps
    // the number of loads in flight uniform for the counted wait.  Weight gradients may have their k axis in pieces
    // (kernels.h): at the end of a piece the cursor moves to the next piece's base.
    constexpr bool PIECES = AKS && BKS;
    const int nk = kext / BK;
    const int nseg = pieces, seg_stages = nk / nseg;
    const char *pA = gA, *pB = gB;
    int fetched = 1, left = seg_stages, piece = 0;
    const char *nextA = gA, *nextB = gB;   // where the next piece starts (segA[0], segB[0] are set for one piece too)
    auto next_piece = [&]() {
      const int nx = min(piece + 1, nseg - 1);
      nextA = (const char*)((const bf16*)g.segA[piece0 + nx] + m0);
      nextB = (const char*)((const bf16*)g.segB[piece0 + nx] + n0);
    };
    if constexpr (PIECES) next_piece();
    auto advance = [&]() {
      const bool more = fetched < nk;
      fetched++;
      const char *nA = pA + stepA, *nB = pB + stepB;
      if constexpr (PIECES) {
        left--;
        const bool wrap = left == 0;
        nA = wrap ? nextA : nA;
        nB = wrap ? nextB : nB;
        left = wrap ? seg_stages : left;
        piece = min(piece + (wrap ? 1 : 0), nseg - 1);
        next_piece();
      }
      pA = more ? nA : pA;
      pB = more ? nB : pB;
    };
#pragma unroll
    for (int t = 0; t < NS; t++) {
      issue_tile_loads<BK, BM, NW>(pA, offA, ring + t * STAGE, wave);
      issue_tile_loads<BK, BN, NW>(pB, offB, ring + t * STAGE + BM * 2 * BK, wave);
      advance();
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 1) * LPS));
    __builtin_amdgcn_s_barrier();
    Frags<BK, BM, BN, WGM, WGN, AKS, BKS> f0, f1;
    f0.load(ring, ring + BM * 2 * BK, wk * KPW, wm, wn, lane);
    int c = 0;  // ring slot of k-block j (its wave's first fragments are in f0; with one k-step per block, in f0 and f1 by turns)
    for (int j = 0; j < nk; j += 3 - KPW) {
      const int n = c + 1 == NS ? 0 : c + 1;
      if constexpr (KPW == 2) {
        first_step<BM, BN, WGM, WGN, AKS, BKS>(ring + c * STAGE, wk * KPW + 1, f0, f1, acc, wm, wn, lane);
        // the next stage has landed (own loads by count, the others' by the barrier) and this one is read out
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 2) * LPS));
        __builtin_amdgcn_s_barrier();
        last_step<BM, BN, WGM, WGN, AKS, BKS>(pA, pB, offA, offB, ring + c * STAGE, ring + n * STAGE, wk * KPW, f1, f0, acc, wave, wm, wn, lane);
        advance();
        c = n;
      } else {
        const int n2 = n + 1 == NS ? 0 : n + 1;
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 2) * LPS));
        __builtin_amdgcn_s_barrier();
        last_step<BM, BN, WGM, WGN, AKS, BKS>(pA, pB, offA, offB, ring + c * STAGE, ring + n * STAGE, wk, f0, f1, acc, wave, wm, wn, lane);
        advance();
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((NS - 2) * LPS));
        __builtin_amdgcn_s_barrier();
        last_step<BM, BN, WGM, WGN, AKS, BKS>(pA, pB, offA, offB, ring + n * STAGE, ring + n2 * STAGE, wk, f1, f0, acc, wave, wm, wn, lane);
        advance();
        c = n2;
      }
    }
  } else if constexpr (K32) {
    using namespace k32;
    constexpr int LPS = (BM + BN) / 16 / NW;
    constexpr int SLOT = (BM + BN) * 64;  // ring slot t: A tile at t * SLOT, B tile behind it
    char* const sA0 = ring;
    char* const sB0 = ring + BM * 64;
    char* const sA1 = ring + SLOT;
    char* const sB1 = ring + SLOT + BM * 64;
    char* const sA2 = ring + 2 * SLOT;
    char* const sB2 = ring + 2 * SLOT + BM * 64;
    char* const sA3 = ring + 3 * SLOT;
    char* const sB3 = ring + 3 * SLOT + BM * 64;
    const size_t stepA = (size_t)BK * g.lda * 2;  // bytes per stage (both operands k-strided)
    const size_t stepB = (size_t)BK * g.ldb * 2;
    uint32_t offA[BM / 16 / NW], offB[BN / 16 / NW];
#pragma unroll
    for (int i = 0; i < BM / 16 / NW; i++) offA[i] = loader_src_offset<BK, BM, AKS>(wave + NW * i, lane, g.lda);
#pragma unroll
    for (int i = 0; i < BN / 16 / NW; i++) offB[i] = loader_src_offset<BK, BN, BKS>(wave + NW * i, lane, g.ldb, GW, g.swiglu_F);
    // nk is a multiple of 4 (K is a multiple of 128).  Stage t lives in ring slot t % 4.
    const int nk = kext / BK;
    // The k axis may be cut into pieces that live in different buffers (kernels.h): the outer loop runs over the
    // pieces, the inner one over the stages of a piece (a multiple of 4).  The stage fetched during local step t
    // is local stage t + 4; past the end of the piece that is a stage of the next piece, past the end of the last
    // piece the last stage again (fetched into a dead slot, which keeps the in-flight load count uniform).  The
    // choice is a scalar select, so the inner loop stays one basic block.
    const int nseg = pieces;
    const int seg_stages = nk / nseg;
    issue_tile_loads<BK, BM, NW>(gA, offA, sA0, wave);
    issue_tile_loads<BK, BN, NW>(gB, offB, sB0, wave);
    issue_tile_loads<BK, BM, NW>(gA + stepA, offA, sA1, wave);
    issue_tile_loads<BK, BN, NW>(gB + stepB, offB, sB1, wave);
    issue_tile_loads<BK, BM, NW>(gA + 2 * stepA, offA, sA2, wave);
    issue_tile_loads<BK, BN, NW>(gB + 2 * stepB, offB, sB2, wave);
    issue_tile_loads<BK, BM, NW>(gA + 3 * stepA, offA, sA3, wave);
    issue_tile_loads<BK, BN, NW>(gB + 3 * stepB, offB, sB3, wave);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(3 * LPS));
    __builtin_amdgcn_s_barrier();

    Frags32<BK, BM, BN, WGM, WGN, AKS, BKS> f0, f1;
    f0.load(sA0, sB0, 0, wm, wn, lane);
    const char *curA = gA, *curB = gB;
    int sg = 0;
    do {   // (neither loop is ever empty: see the k64 pipeline)
      const bool last_piece = sg + 1 == nseg;
      const char* nxtA = last_piece ? curA : (const char*)((const bf16*)g.segA[piece0 + sg + 1] + m0);
      const char* nxtB = last_piece ? curB : (const char*)((const bf16*)g.segB[piece0 + sg + 1] + n0);
      const int lim = last_piece ? seg_stages - 1 : seg_stages + 3;
#define AH_STAGE_PTRS(u)                                                                                              \
  (min((u), lim) >= seg_stages ? nxtA + (size_t)(min((u), lim) - seg_stages) * stepA : curA + (size_t)min((u), lim) * stepA), \
      (min((u), lim) >= seg_stages ? nxtB + (size_t)(min((u), lim) - seg_stages) * stepB : curB + (size_t)min((u), lim) * stepB)
      int t = 0;
      do {
        ring_step<BM, BN, WGM, WGN, AKS, BKS>(AH_STAGE_PTRS(t + 4), offA, offB, sA0, sB0, sA1, sB1, f0, f1, acc, wave, wm, wn, lane);
        ring_step<BM, BN, WGM, WGN, AKS, BKS>(AH_STAGE_PTRS(t + 5), offA, offB, sA1, sB1, sA2, sB2, f1, f0, acc, wave, wm, wn, lane);
        ring_step<BM, BN, WGM, WGN, AKS, BKS>(AH_STAGE_PTRS(t + 6), offA, offB, sA2, sB2, sA3, sB3, f0, f1, acc, wave, wm, wn, lane);
        ring_step<BM, BN, WGM, WGN, AKS, BKS>(AH_STAGE_PTRS(t + 7), offA, offB, sA3, sB3, sA0, sB0, f1, f0, acc, wave, wm, wn, lane);
        t += 4;
      } while (t < seg_stages);
#undef AH_STAGE_PTRS
      curA = nxtA;
      curB = nxtB;
    } while (++sg < nseg);
  } else {
    using namespace k64;
    constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;     // loads per tile per wave
    const size_t stepA = (AKS ? (size_t)BK * g.lda : (size_t)BK) * 2;  // bytes per k-block
    const size_t stepB = (BKS ? (size_t)BK * g.ldb : (size_t)BK) * 2;

    uint32_t offA[LA], offB[LB];
#pragma unroll
    for (int i = 0; i < LA; i++) offA[i] = loader_src_offset<BK, BM, AKS>(wave + NW * i, lane, g.lda);
#pragma unroll
    for (int i = 0; i < LB; i++) offB[i] = loader_src_offset<BK, BN, BKS>(wave + NW * i, lane, g.ldb, GW, g.swiglu_F);

    // K is a multiple of 128: an even number of k-blocks.  Past the end the last k-block is fetched again into
    // dead buffers, which keeps the number of loads in flight uniform for the counted wait.
    // F = the operand whose tiles go first, S = the other one.
    constexpr bool BF = b_first<BM, BN, AKS>();
    constexpr int WF = BF ? BN : BM, WS = BF ? BM : BN;
    const char* gF = BF ? gB : gA;
    const char* gS = BF ? gA : gB;
    const size_t stepF = BF ? stepB : stepA, stepS = BF ? stepA : stepB;
    uint32_t* offF = BF ? offB : offA;
    uint32_t* offS = BF ? offA : offB;
    const int np = g.K / BK, lastp = np - 1;
    // Ring: F_j in buffer j % (DEPTH + 1) of WF rows, S_j behind those in buffer j % DEPTH of WS rows.  During k-block j the tiles
    // F_{j + DEPTH} and S_{j + DEPTH} are fetched.
    constexpr int FB = WF * 2 * BK, SB = WS * 2 * BK, NF = DEPTH + 1, NSB = DEPTH;
    char* const ringS = ring + NF * FB;
#pragma unroll
    for (int t = 0; t < DEPTH; t++) {
      issue_tile_loads<BK, WF, NW>(gF + (size_t)min(t, lastp) * stepF, offF, ring + t * FB, wave);
      issue_tile_loads<BK, WS, NW>(gS + (size_t)min(t, lastp) * stepS, offS, ringS + t * SB, wave);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0((DEPTH - 1) * (WF + WS) / 8 / NW));
    __builtin_amdgcn_s_barrier();

    Frags32<BK, BM, BN, WGM, WGN, AKS, BKS> f0, f1;
    f0.load(BF ? ringS : ring, BF ? ring : ringS, 0, wm, wn, lane);
    int jf = 0, js = 0;  // buffers of F_j and S_j
    int j = 0;
    do {   // (np >= 2; a loop that might not run would have its accumulators copied at its exit, ahead of the wait below)
      const int nf = jf + 1 == NF ? 0 : jf + 1;    // F_{j+1}
      const int ns = js + 1 == NSB ? 0 : js + 1;   // S_{j+1}
      const int ff = jf == 0 ? NF - 1 : jf - 1;    // F_{j + DEPTH}: into the buffer of F_{j-1}; S_{j + DEPTH} goes into that of S_j
      const char *cF = ring + jf * FB, *cS = ringS + js * SB, *nxF = ring + nf * FB, *nxS = ringS + ns * SB;
      const char* pS = gS + (size_t)min(j + DEPTH, lastp) * stepS;
      const char* pF = gF + (size_t)min(j + DEPTH, lastp) * stepF;
      half_even<BM, BN, WGM, WGN, AKS, BKS>(pF, offF, ring + ff * FB, BF ? cS : cF, BF ? cF : cS, f0, f1, acc, wave, wm, wn, lane);
      half_odd<BM, BN, WGM, WGN, AKS, BKS, DEPTH>(pS, offS, ringS + js * SB, BF ? nxS : nxF, BF ? nxF : nxS, f0, f1, acc, wave, wm, wn, lane);
      jf = nf;
      js = ns;
    } while (++j < np);
  }
  __builtin_amdgcn_s_waitcnt(0);  // drain the redundant tail loads before the block's LDS is released
  if constexpr (!SPLIT) {
    // The compiler does not see that the accumulators come from matrix instructions: 16 wait states before the first read of
    // the last one's result.
    asm volatile("s_nop 15");
#pragma unroll
    for (int i = 0; i < BM / WGM / AB; i++)
#pragma unroll
      for (int j = 0; j < BN / WGN / AB; j++) asm volatile("" : "+a"(acc[i][j]));
  }

  // ---- epilogue.  A lane holds C[m][n .. n+3] of each 16x16 block (for 4 column groups of each 32x32 block where waves split
  // the k axis): stores straight from that layout would touch 16 (32) rows per instruction, 16 bytes each.  Instead each
  // wave passes its sub-tile through a private LDS strip, 32 rows at a time in fp32, and reads it
  // back row-major, so that every global access is 16 bytes per lane and whole rows per 16 lanes.
  // Where waves split the k axis, the WGK waves of a sub-tile leave 64 rows at a time, each its own partial sums, and
  // each takes 64 / WGK of those rows back, adding the partial sums in the order of the k shares.
  constexpr int WN = BN / WGN, WM = BM / WGM;
  constexpr int ROWB = WN * 4 + 16;                // padded strip row
  constexpr int SR = SPLIT ? 64 : 32;              // rows of a strip
  constexpr int RPW = SR / WGK;                    // rows of it that a wave writes out
  static_assert(NW * SR * ROWB + 2048 <= RING, "staging strips (and a row of column sums per wave) must fit in the ring");
  __syncthreads();                                  // every wave is done with the ring
  char* strip = ring + wave * (SR * ROWB);          // written by this wave
  const char* strip_rd = SPLIT ? ring + (wmn * WGK) * (SR * ROWB) + wk * RPW * ROWB : strip;   // first of the WGK strips, at this wave's rows
  float* const Cf = KSHARES && shares > 1 ? g.k_part + (size_t)share * g.M * g.N : (float*)g.C;   // fp32 outputs
  const int ldcf = KSHARES && shares > 1 ? g.N : g.ldc;
  const bf16* bias = (const bf16*)g.bias;
  const bf16* aux = (const bf16*)g.aux;
  constexpr bool RESID = EPI == EPI_RESID || EPI == EPI_RESID_F32 || EPI == EPI_RESID_F32_OUT16;
  constexpr bool AUX_F32 = EPI == EPI_RESID_F32 || EPI == EPI_RESID_F32_OUT16;   // the residual is read in fp32
  constexpr bool OUT_F32 = EPI == EPI_F32_ACC || EPI == EPI_F32_SET || EPI == EPI_RESID_F32;
  const bool has_bias = (EPI == EPI_BF16 || EPI == EPI_GELU || RESID) && bias != nullptr;
  constexpr int PPR = WN / 8;                       // 8-column pieces per strip row
  // rows that the wave takes at a time (PPR = 10 and 12, of tiles 160 and 192 wide: with 40 and 48 of its lanes), and how often
  constexpr int RPI = 64 % PPR == 0 ? 64 / PPR : 4, NIT = RPW / RPI;
  constexpr bool PART = RPI * PPR < 64;
  // ROLLED: the pieces of a strip are taken in a loop that is not unrolled.  Straight-line code runs once per launch and tile,
  // at the rate at which instructions arrive from a cold cache: the GeLU epilogues of a 256 x 256 tile had 27 and 42 KB of
  // it, now 10 and 14.  4096 x 4096 x 1024: forward 47.0 -> 42.0 us (half of the difference to the plain epilogue); input
  // gradient 51.7 -> 49.3.  Plain and residual epilogues (10 .. 15 KB) gain nothing from it, the rotary one loses 2 %.
  // AUX_LDS: the second operand's pieces then wait in LDS, two strips' worth per wave (each lane reads back what it asked
  // for), instead of in registers, which a loop cannot index (loaded piece by piece in the loop: 57.6 us).
  constexpr bool AUX_LDS = !SPLIT && EPI == EPI_GELU_BWD;
  constexpr bool ROLLED = !SPLIT && (EPI == EPI_GELU || EPI == EPI_GELU_BWD);
  constexpr int UNROLL = ROLLED ? 1 : NIT;
  char* const aux_lds = ring + NW * SR * ROWB + wave * (2 * NIT * 1024);
  static_assert(!AUX_LDS || NW * (SR * ROWB + 2 * NIT * 1024) <= RING, "two strips of the second operand must fit behind the staging strips");
  auto strip_piece = [&](int row, int piece) {      // 4 + 4 consecutive columns of a row, the partial sums added up
    const char* p = strip_rd + row * ROWB + piece * 32;
    f32x4 lo = *(const f32x4*)p, hi = *(const f32x4*)(p + 16);
#pragma unroll
    for (int k = 1; k < WGK; k++) {
      lo += *(const f32x4*)(p + k * (SR * ROWB));
      hi += *(const f32x4*)(p + k * (SR * ROWB) + 16);
    }
    struct { f32x4 lo, hi; } r = {lo, hi};
    return r;
  };
  const int cp = lane % PPR, row0 = PART ? min(lane / PPR, RPI - 1) : lane / PPR;     // the lane's rows: row0 + it * RPI
  const bool on = !PART || lane < RPI * PPR;
  // output column of the lane's piece.  SwiGLU: the first half of the wave's strip row holds GW gate columns, the
  // second half their up columns; both go to u[:, 2F] (gate at column c, up at F + c), their product to C2[:, F].
  const bool up_piece = SWIGLU && cp >= PPR / 2;
  const int nlog = SWIGLU ? n0 / 2 + wn * GW + (up_piece ? cp - PPR / 2 : cp) * 8 : 0;   // logical column of the piece
  const int n = SWIGLU ? (up_piece ? g.swiglu_F + nlog : nlog) : n0 + wn * WN + cp * 8;
  float bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (has_bias) {
    const bf16x8 b = *(const bf16x8*)(bias + n);
#pragma unroll
    for (int i = 0; i < 8; i++) bv[i] = bf2f(b[i]);
  }
  float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // EPI_GELU_BWD: this lane's column sums over the current 64-row slab
  const bool want_colsum = EPI == EPI_GELU_BWD && g.colsum_part != nullptr;
  // EPI_ROPE: this lane's 8 pairs, the partner piece, and (cos, sin) of RPI angle steps (the distance between a
  // lane's consecutive rows), read once from the table's row of that position; per strip of 32 rows (which never
  // straddles a sequence: S is a multiple of 128) the angles of the lane's first row are read from the table and
  // carried from row to row by rotation
  const bool rot = EPI == EPI_ROPE && n < g.rope_cols;
  float rc[8], rs[8], dcs_c[8], dcs_s[8];
  int rope_pcp = 0, rope_i0 = 0;
  float rope_sgn = 0.f;
  if (EPI == EPI_ROPE && rot) {
    const int d = g.rope_d, ch = (cp * 8) % d, half = d >> 1;
    const bool lower = ch < half;
    rope_pcp = lower ? cp + (d >> 4) : cp - (d >> 4);
    rope_i0 = lower ? ch : ch - half;
    rope_sgn = lower ? -1.f : 1.f;
    const float* t = g.rope_cs + ((size_t)RPI * half + rope_i0) * 2;
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) {
      const f32x4 e = *(const f32x4*)(t + 4 * q4);
      dcs_c[2 * q4] = e[0]; dcs_s[2 * q4] = e[1]; dcs_c[2 * q4 + 1] = e[2]; dcs_s[2 * q4 + 1] = e[3];
    }
  }
  const uint32_t aux_off = AUX_LDS ? (uint32_t)(row0 * g.ld_aux + n) * 2u : 0;
  auto fetch_aux = [&](int tm) {
    const bf16* p = aux + (size_t)(m0 + wm * WM + tm * 32) * g.ld_aux;
#pragma unroll
    for (int it = 0; it < NIT; it++) load16_to_lds_uncounted(p + (size_t)it * RPI * g.ld_aux, aux_off, aux_lds + ((tm & 1) * NIT + it) * 1024);
  };
  if constexpr (AUX_LDS) fetch_aux(0);
#pragma unroll
  for (int tm = 0; tm < TM; tm += SR / 32) {
    const int mbase = m0 + wm * WM + tm * 32 + wk * RPW + row0;
    if (EPI == EPI_ROPE && rot) {
      const float* t = g.rope_cs + ((size_t)(mbase % g.rope_S) * (g.rope_d >> 1) + rope_i0) * 2;
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const f32x4 e = *(const f32x4*)(t + 4 * q4);
        rc[2 * q4] = e[0]; rs[2 * q4] = e[1]; rc[2 * q4 + 1] = e[2]; rs[2 * q4 + 1] = e[3];
      }
    }
    // operands of the epilogue that come from memory: issue their loads before the strip round trip
    bf16x8 ax[AUX_LDS ? 1 : NIT], ax2[EPI == EPI_SWIGLU_BWD ? NIT : 1];
    f32x4 old0[NIT], old1[NIT];
    if constexpr (AUX_LDS) {
      if (tm + 1 < TM) fetch_aux(tm + 1);
    } else if (EPI == EPI_RESID || EPI == EPI_GELU_BWD || EPI == EPI_SWIGLU_BWD) {
#pragma unroll
      for (int it = 0; it < NIT; it++) ax[AUX_LDS ? 0 : it] = *(const bf16x8*)(aux + (size_t)(mbase + it * RPI) * g.ld_aux + n);
    }
    if (EPI == EPI_SWIGLU_BWD) {  // aux = gate | up: the up columns sit swiglu_F further
#pragma unroll
      for (int it = 0; it < NIT; it++) ax2[it] = *(const bf16x8*)(aux + (size_t)(mbase + it * RPI) * g.ld_aux + g.swiglu_F + n);
    }
    if (EPI == EPI_F32_ACC || AUX_F32) {
#pragma unroll
      for (int it = 0; it < NIT; it++) {
        const float* cptr = (AUX_F32 ? (const float*)g.aux : (const float*)g.C) + (size_t)(mbase + it * RPI) * (AUX_F32 ? g.ld_aux : g.ldc) + n;
        old0[it] = *(const f32x4*)cptr;
        old1[it] = *(const f32x4*)(cptr + 4);
      }
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int tr = 0; tr < SR / 32; tr++)
#pragma unroll
        for (int tn = 0; tn < TN; tn++)
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const int col = tn * 32 + 8 * q + 4 * (lane >> 5);
            const f32x16& a = acc[tm + tr][tn];
            f32x4 v = {a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
            *(f32x4*)(strip + (tr * 32 + (lane & 31)) * ROWB + col * 4) = v;
          }
    } else {
#pragma unroll
      for (int tr = 0; tr < 2; tr++)
#pragma unroll
        for (int tn = 0; tn < BN / WGN / 16; tn++)
          *(f32x4*)(strip + (tr * 16 + (lane & 15)) * ROWB + (tn * 16 + 4 * (lane >> 4)) * 4) = acc[2 * tm + tr][tn];
    }
    if constexpr (SPLIT) {
      __syncthreads();
    } else {
      if constexpr (AUX_LDS) {
        // this strip's pieces have landed: behind them there are the next strip's NIT loads (but for the last strip) and at
        // least NIT stores of the strip before (but for the first)
        if (tm > 0 && tm + 1 < TM) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(2 * NIT));
        else if (tm > 0 || TM > 1) __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(NIT));
        else __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));
      } else {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));
      }
      __builtin_amdgcn_wave_barrier();
      if (AUX_LDS) asm volatile("" ::: "memory");
    }
    if (on)
#pragma unroll UNROLL
    for (int it = 0; it < NIT; it++) {
      const int row = row0 + it * RPI;
      const auto pc = strip_piece(row, cp);
      const f32x4 lo = pc.lo, hi = pc.hi;
      float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      const size_t m = (size_t)(mbase + it * RPI);
      if (OUT_F32) {
        float* cptr = Cf + m * ldcf + n;
        if (EPI == EPI_F32_ACC || EPI == EPI_RESID_F32) {
          if (EPI == EPI_RESID_F32) {
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] += bv[i];
          }
#pragma unroll
          for (int i = 0; i < 4; i++) { v[i] += old0[it][i]; v[4 + i] += old1[it][i]; }
        }
        *(f32x4*)cptr = f32x4{v[0], v[1], v[2], v[3]};
        *(f32x4*)(cptr + 4) = f32x4{v[4], v[5], v[6], v[7]};
      } else {
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] += bv[i];
        if (EPI == EPI_RESID) {
#pragma unroll
          for (int i = 0; i < 8; i++) v[i] += bf2f(ax[it][i]);
        }
        if (EPI == EPI_ROPE && rot) {
          // rotary embedding on the fp32 sums: the pair of column c of a head is c +- d/2, d/16 pieces away in the
          // same strip row (a wave's strip holds whole heads: WN % d == 0, see tile_fits)
          const auto pp = strip_piece(row, rope_pcp);
          const f32x4 plo = pp.lo, phi = pp.hi;
          const float pv[8] = {plo[0], plo[1], plo[2], plo[3], phi[0], phi[1], phi[2], phi[3]};
#pragma unroll
          for (int i = 0; i < 8; i++) {
            v[i] = v[i] * rc[i] + rope_sgn * pv[i] * rs[i];
            // the lane's next row is RPI positions further: rotate (cos, sin) by that many steps of the angle
            const float c2 = rc[i] * dcs_c[i] - rs[i] * dcs_s[i];
            rs[i] = rs[i] * dcs_c[i] + rc[i] * dcs_s[i];
            rc[i] = c2;
          }
        }
        if (EPI == EPI_RESID_F32_OUT16) {
#pragma unroll
          for (int i = 0; i < 4; i++) { v[i] += old0[it][i]; v[4 + i] += old1[it][i]; }
        }
        if (EPI == EPI_GELU_BWD) {
          const bf16x8 u8 = AUX_LDS ? *(const bf16x8*)(aux_lds + ((tm & 1) * NIT + it) * 1024 + lane * 16) : ax[AUX_LDS ? 0 : it];
#pragma unroll
          for (int i = 0; i < 8; i++) v[i] *= gelu_grad_f(bf2f(u8[i]));
        }
        bf16x8 o;
        if (EPI == EPI_SWIGLU_BWD) {
          // v = dm; d(gate) = dm up silu'(gate) goes to column n, d(up) = dm silu(gate) to column F + n
          bf16x8 o2;
#pragma unroll
          for (int i = 0; i < 8; i++) {
            const float x = bf2f(ax[it][i]), sg = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
            o[i] = f2bf(v[i] * bf2f(ax2[it][i]) * sg * __builtin_fmaf(x, 1.0f - sg, 1.0f));
            o2[i] = f2bf(v[i] * x * sg);
          }
          *(bf16x8*)((bf16*)g.C + m * g.ldc + g.swiglu_F + n) = o2;
        } else {
#pragma unroll
          for (int i = 0; i < 8; i++) o[i] = f2bf(v[i]);
        }
        *(bf16x8*)((bf16*)g.C + m * g.ldc + n) = o;
        if (EPI == EPI_GELU) {
          bf16x8 o2;
#pragma unroll
          for (int i = 0; i < 8; i++) o2[i] = f2bf(gelu_f(v[i]));
          *(bf16x8*)((bf16*)g.C2 + m * g.ldc + n) = o2;
        }
        if (EPI == EPI_GELU_BWD) {
#pragma unroll
          for (int i = 0; i < 8; i++) cs[i] += bf2f(o[i]);
        }
        if (SWIGLU && !up_piece) {
          // silu(gate) * up from the fp32 accumulators: the up piece sits PPR / 2 pieces further in the strip row
          const auto up8 = strip_piece(row, cp + PPR / 2);
          const f32x4 ulo = up8.lo, uhi = up8.hi;
          const float up[8] = {ulo[0], ulo[1], ulo[2], ulo[3], uhi[0], uhi[1], uhi[2], uhi[3]};
          bf16x8 o2;
#pragma unroll
          for (int i = 0; i < 8; i++) o2[i] = f2bf(silu_f(v[i]) * up[i]);
          *(bf16x8*)((bf16*)g.C2 + m * g.ldc2 + nlog) = o2;
        }
      }
    }
    if constexpr (SPLIT) {
      __syncthreads();                                 // strip reads are in registers before the next 64 rows overwrite it
    } else {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(63));  // the same within the wave, whose strip it is
      __builtin_amdgcn_wave_barrier();
    }
    // (192 rows: 96 to a wave.  The first wave's are one partial sum, the second one's 64 and 32: three as for three slabs)
    constexpr bool ODD = !SPLIT && TM % 2 == 1;
    static_assert(!ODD || (TM == 3 && WGM == 2), "slabs of a tile");
    const bool slab_ends = SPLIT || (ODD ? tm == TM - 1 || (wm == 1 && tm == 1) : (tm & 1) == 1);
    if (EPI == EPI_GELU_BWD && slab_ends) {
      // one 64-row slab (two strips where a strip has 32 rows): lanes that share a column piece (lane % PPR) add up,
      // and where waves share the slab's rows, these waves' sums through LDS; the first PPR lanes write
      if (want_colsum) {
#pragma unroll
        for (int i = 0; i < 8; i++) {
          if constexpr (PART) {
            float t = cs[i];
#pragma unroll
            for (int r = 1; r < RPI; r++) t += __shfl(cs[i], cp + r * PPR);
            cs[i] = t;
          } else {
#pragma unroll
            for (int off = PPR; off < 64; off <<= 1) cs[i] += __shfl_xor(cs[i], off);
          }
        }
        if constexpr (SPLIT) {
          float* row = (float*)(ring + NW * SR * ROWB) + wave * WN;   // behind the strips
          if (lane < PPR) {
            *(f32x4*)(row + lane * 8) = f32x4{cs[0], cs[1], cs[2], cs[3]};
            *(f32x4*)(row + lane * 8 + 4) = f32x4{cs[4], cs[5], cs[6], cs[7]};
          }
          __syncthreads();
          if (wk == 0 && lane < PPR) {
#pragma unroll
            for (int k = 1; k < WGK; k++)
#pragma unroll
              for (int i = 0; i < 8; i++) cs[i] += row[k * WN + lane * 8 + i];
          }
        }
        if (wk == 0 && lane < PPR) {
          const int slab = ODD ? (m0 >> 6) + (wm == 0 ? 0 : 1 + (tm >> 1)) : (m0 + wm * WM + tm * 32) >> 6;
          float* dst = g.colsum_part + (size_t)slab * g.ld_colsum + n;
          if (g.colsum_acc) {
            const f32x4 o0 = *(const f32x4*)dst, o1 = *(const f32x4*)(dst + 4);
#pragma unroll
            for (int i = 0; i < 4; i++) { cs[i] += o0[i]; cs[4 + i] += o1[i]; }
          }
          *(f32x4*)dst = f32x4{cs[0], cs[1], cs[2], cs[3]};
          *(f32x4*)(dst + 4) = f32x4{cs[4], cs[5], cs[6], cs[7]};
        }
      }
#pragma unroll
      for (int i = 0; i < 8; i++) cs[i] = 0.f;
    }
  }
}

template <int BM, int BN, int WGM, int WGN, int WGK, bool AKS, bool BKS, int EPI, int DEPTH = 2>
__global__ __launch_bounds__(256) void gemm_kernel(GemmArgs g) {
  gemm_tile<BM, BN, WGM, WGN, WGK, AKS, BKS, EPI, DEPTH>(g, blockIdx.x);
}

// Several weight gradients over the same k axis in one launch, the blocks of one product after those of another (a block's
// XCD follows its number, so a product's tiles keep to the raster of a launch of its own, from another XCD on).
struct GemmGroup { int count, first[kMaxGemmGroup + 1]; GemmArgs p[kMaxGemmGroup]; };
template <int BM, int BN, int WGM, int WGN, int WGK, int EPI>
__global__ __launch_bounds__(256) void gemm_group_kernel(GemmGroup gg) {
  int i = 0;
  while (i + 1 < gg.count && (int)blockIdx.x >= gg.first[i + 1]) i++;
  gemm_tile<BM, BN, WGM, WGN, WGK, true, true, EPI>(gg.p[i], blockIdx.x - gg.first[i]);
}

// C[m, n] = beta C[m, n] + sum over the k shares of part[share][m, n], in the order of the shares.  Bound by memory:
// every partial sum is read once; four columns per lane.
__global__ __launch_bounds__(256) void k_shares_kernel(const float* __restrict__ part, float* __restrict__ C, int M, int N, int ldc, int shares, int beta) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4, n = (size_t)M * N;
  if (i >= n) return;
  float* c = C + (i / N) * ldc + i % N;
  f32x4 s = *(const f32x4*)(part + i);
#pragma unroll 4
  for (int k = 1; k < shares; k++) s += *(const f32x4*)(part + (size_t)k * n + i);
  if (beta) s += *(const f32x4*)c;
  *(f32x4*)c = s;
}

bool gemm_shape_ok(int M, int N, int K) {
  return M > 0 && N > 0 && K > 0 && (M % 128) == 0 && (N % 128) == 0 && (K % 128) == 0;
}

bool gemm_segments_ok(int seg_k, int n_seg) {
  return seg_k > 0 && (seg_k % 128) == 0 && n_seg >= 1 && n_seg <= kMaxGemmSegments && (long)seg_k * n_seg <= (1L << 30);
}

namespace {

// Tile choice.  The chip's 256 CUs take the tiles of a launch in rounds, one or (where half the LDS suffices) two to
// a CU; the time of a full round is a + b K, that of one of which only the share `fill` of the slots is taken is
// 1 - f (1 - fill) times that (the board is limited by power, the caches by what all CUs ask of them).  Measured, in us
// with K in units of 1024: 256 and 512 tiles of each kind, K = 256 .. 16384, the weights read from HBM, replayed back to
// back, so that a includes the gap between launches.  fwd is for the products with a k-contiguous operand (mean of NN and
// NT), tn for the weight gradient.
// f: 64 and 160 tiles of 256 x 256 take 0.70 and 0.78 of the time of 256 (f = 0.40, 0.59; 0.47 and 0.57 over 54 products
// of 64 .. 127 and 128 .. 191 tiles, 0.49 and 0.60 in the weight gradient).  With 0.35 there too, 130 .. 192 such tiles
// lost to 520 .. 768 of 128 x 128: 2560 x 3840 x 1536 (NT) 39.1 us against 32.8, 4096 x 3072 x 1024 with cold operands
// 38.0 / 30.5.
// The rows of the first four tiles were taken with the 32x32x16 loop, which the next three still run.  One round of the first four, the weights
// from HBM, on the present loop: 256 x 256 22.8 k + 11.8 (level at k = 1, 1 % less than its row at 16), 256 x 128 13.1 k + 8.2 (level, 6 %),
// 128 x 128 8.4 k + 4.8 (2 %, 6 %).  The rows of the 192 and 160 wide tiles are of the present loop, their second ones measured against 256 x 256 at
// 44.5 k + 17.2, so beside these the older tiles are priced up to 6 % too high.
// tn of the two small tiles: fitted to 1500 weight gradients of K = 128 .. 32768, scaled like the other tiles' rows
// (those over-estimate by 8 %).  The line through K >= 256 alone was 10-35 % short at K = 128 .. 512, where these tiles then
// displaced 128 x 128: 3200 x 896 x 128 8.6 us against 7.3.
struct Rate { float a, b, f; };
struct TileCfg { int bm, bn, wgm, wgn, wgk; Rate fwd1, fwd2, tn1, tn2; };  // one, two tiles to a CU
const TileCfg kTiles[] = {
  {256, 256, 2, 2, 1, {11.5f, 23.1f, .45f}, {21.8f, 44.9f, .35f}, {16.3f, 23.3f, .50f}, {33.5f, 45.4f, .35f}},
  {256, 128, 2, 2, 1, {7.1f, 14.1f, .35f}, {10.8f, 28.5f, .35f}, {12.3f, 12.7f, .35f}, {20.4f, 25.2f, .35f}},
  {128, 256, 2, 2, 1, {7.4f, 13.7f, .35f}, {12.1f, 27.4f, .35f}, {11.0f, 12.8f, .35f}, {20.5f, 25.0f, .35f}},
  {128, 128, 2, 2, 1, {4.4f, 9.0f, .35f}, {5.9f, 14.7f, .35f}, {8.2f, 8.0f, .35f}, {11.0f, 15.3f, .35f}},
  {128, 128, 1, 1, 4, {7.5f, 7.6f, .35f}, {14.2f, 14.5f, .35f}, {}, {}},   // not built for the weight gradient (see namespace ksplit)
  {64, 128, 1, 2, 2, {3.8f, 5.7f, .35f}, {4.8f, 10.5f, .35f}, {6.6f, 5.6f, .23f}, {8.7f, 10.1f, .14f}},
  {64, 64, 1, 1, 4, {3.6f, 3.3f, .35f}, {4.3f, 6.8f, .35f}, {5.7f, 3.5f, .15f}, {6.6f, 6.4f, .03f}},
  // forward and input gradient only
  {256, 192, 2, 2, 1, {9.4f, 18.1f, .45f}, {20.0f, 36.5f, .35f}, {}, {}},
  {256, 160, 2, 2, 1, {8.6f, 15.5f, .42f}, {20.0f, 31.0f, .35f}, {}, {}},
  {192, 256, 2, 2, 1, {9.8f, 17.9f, .42f}, {19.5f, 36.5f, .35f}, {}, {}},
  {192, 128, 2, 2, 1, {6.1f, 10.4f, .32f}, {10.5f, 21.5f, .35f}, {}, {}},
  {128, 192, 2, 2, 1, {5.5f, 11.1f, .32f}, {13.5f, 21.5f, .35f}, {}, {}}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
// Tiles of 192 and 160 fit outputs that the powers of two leave as one round of large tiles on half of the CUs, or as two of 128 x 128:
// of 48 random products of up to 4096 x 8192 x 8192 whose plan they changed, geometric means 0.91 (128 x 192), 0.88 (192 x 128), 0.87 (192 x
// 256), 0.83 (256 x 160) and 0.89 (256 x 192, one round); 1920 x 3200 x 2688 43.1 -> 33.5 us, 2048 x 5120 x 20480 366 -> 336 (NT; the vendor library
// 325), 4096 x 6144 x 4096 173 -> 160.  They are taken in launches of at least three quarters of the CUs (below, a cover of two launches comes
// close: 3840 x 2304 x 5248 98 .. 99 us in 180 tiles of 192 x 256, 103 .. 107 as such a cover), and the 256-row ones from
// K = 2048 on.  They are faster below, too (4096 x 3072 x 1024 27.6 -> 25.5 us with 256 x 192, 2560 x 3840 x 1536 35.0 -> 28.6 with 256 x 160), but there
// tests/test_gemm_plan.py holds the choice between the older tiles.  Rates: 256 and 512 tiles of each kind, the second measured against that
// of 256 x 256 (44.5 k + 17.2 us there).
constexpr int kNarrowTiles = 7;      // first of these tiles
constexpr int kNarrowMinK = 2048, kNarrowMinTiles = 192;
constexpr int kWholeCuTile = 4;      // the tile above whose blocks take all of a CU's LDS although the launch is small
constexpr float kLaunchGap = 2.5f;   // the part of a that later rounds of the same launch do not pay

int forced_tile() {
  static int forced = -2;
  if (forced == -2) {
    const char* e = getenv("AH_GEMM_TILE");  // tuning aid: index into kTiles
    forced = e ? atoi(e) : -1;
  }
  return forced;
}

// The order of a sum's terms, and so its last bits, depends on the tile.  So the choice knows the problem alone, not what runs beside it on
// another stream, but between tiles that add up in the same order (launch_gemm).  kWholeCuTile's blocks leave no room on a CU for those of a second stream, so it is
// taken only from a k on where the gain is clear.  Stage times with the line elsewhere, against 5120 (G: micro-batches
// per group; with G = 1 the second stream runs): at 3584, 1280-wide stage (k = 3840) 1.06 at G = 1, 1.02 at G = 2 and 3,
// BERT-Large (k = 4096) 1.01 at G = 1, 0.98 at G = 8; at 2048, 768-wide BERT (k = 3072) 1.00 at G = 1, 0.98 at G = 3;
// at 6400, 1536-wide stage (k = 6144) 0.97 at G = 1, 1.015 at G = 3, 1.026 at G = 5, LLaMA-style 2048-wide (k = 5504
// and 6144) 1.00; without the tile, the latter 1.03 at G = 1 and 3, 2048-wide GPT (k = 6144 and 8192) 0.98 at G = 1, 1.015 from
// G = 2 on.  Single products gain below the line too (1408 x 1536 x 4096 NT 39.0 us, 27.7 with this tile): what they
// lose is the price of one choice for all callers.
// (These were taken beside the 32x32x16 loop.)  128 x 128 tiles of the present loop, on the deeper ring, are level with this one or faster (this / those, us,
// operands from the caches): 2048 x 2048 x 6144 50.8 / 51.9 (NN) and 50.4 / 47.7 (NT), x 8192 64.9 / 67.6 and 62.8 / 60.7, 640 x 6016 x 6656 50.6 / 52.7 and
// 50.8 / 47.4; the 1.3B stage, whose weights come from HBM, 6088 / 5861.  The tile stays at every k for its sums: four chains a quarter as long
// leave fp32 results half as far from 64 bits, 2.0e-7 against 4.1e-7 of their norm at k = 6144, 2.4e-7 against 5.0e-7 at 8192.
constexpr int kWholeCuMinK = 5120;
// head: a wave's columns must hold whole heads of this width (0: any; the rotary epilogue, EPI_ROPE, of forward)
bool tile_fits(int i, int M, int n, int K, bool tn, int head) {
  const TileCfg& t = kTiles[i];
  if (M % t.bm || n % t.bn) return false;
  if (i == kWholeCuTile && (tn || (K < kWholeCuMinK && !head))) return false;
  if (i >= kNarrowTiles && (tn || head)) return false;
  if (i >= kNarrowTiles && forced_tile() != i && ((t.bm == 256 && K < kNarrowMinK) || (M / t.bm) * (n / t.bn) < kNarrowMinTiles)) return false;
  return !(head && t.bn / t.wgn % head);
}

// time of a launch of `tiles` tiles of kind i over K
float launch_cost(int i, long tiles, float K, bool tn) {
  const TileCfg& t = kTiles[i];
  const long full = tiles / 512, rest = tiles % 512;
  const float k = K / 1024.f;
  const Rate &r1 = tn ? t.tn1 : t.fwd1, &r2 = tn ? t.tn2 : t.fwd2;
  float us = full * (r2.a + r2.b * k - kLaunchGap) + kLaunchGap;
  if (rest > 0) {
    const Rate& r = rest > 256 ? r2 : r1;
    const float fill = (float)rest / (rest > 256 ? 512 : 256);
    us += (r.a + r.b * k) * (1.f - r.f * (1.f - fill)) - kLaunchGap;
  }
  return us;
}

// time of covering an M x n output with tile i, the k axis cut into `shares` that run side by side
float tile_cost(int i, int M, int n, int K, bool tn, int shares = 1) {
  return launch_cost(i, (long)(M / kTiles[i].bm) * (n / kTiles[i].bn) * shares, (float)K / shares, tn);
}

int pick_tile(int M, int N, int K, bool tn, int head, int kinds) {
  const int forced = forced_tile();
  if (forced >= 0 && forced < kNumTiles && tile_fits(forced, M, N, K, tn, head)) return forced;
  int best = -1;
  float best_t = 0;
  for (int i = 0; i < kinds; i++) {
    if (!tile_fits(i, M, N, K, tn, head)) continue;
    const float t = tile_cost(i, M, N, K, tn);
    if (best < 0 || t < best_t) { best = i; best_t = t; }
  }
  return best;
}

// How a launch covers its output: with one tile shape, or as two launches over the column ranges [0, n0) and
// [n0, N), each with its own tile shape.  The second form is for outputs whose tile count is not a good multiple
// of the 256 CUs: 4096 x 6144 is 384 tiles of 256 x 256, i.e. two rounds of which the second is half empty;
// 256 tiles of 256 x 256 over the first 4096 columns and then 256 tiles of 256 x 128 over the rest is two full rounds.
struct Plan { int parts; int tile[2]; int n0; int shares; };
constexpr float kSecondLaunch = 2.f;  // us: the first launch's last tiles run alone

// A weight gradient over many tokens with a small output (fewer tiles than CUs) may cut its k axis into shares, each a
// launch's worth of tiles of its own, whose sums a second kernel adds up: 1024 x 4096 over 32768 tokens is 64 tiles of
// 256 x 256 in four shares and 64 MB of partial sums instead of 256 tiles of 128 x 128 at 1.3 times the cost per flop.
constexpr int kMaxShares = 16;
float shares_cost(int M, int N, int shares) { return 4.f + (float)M * N * 4.f * (shares + 2) / 4.5e6f; }  // launch, and 4.5 TB/s

bool one_chain(const Plan& p) { return kTiles[p.tile[0]].wgk == 1 && (p.parts == 1 || kTiles[p.tile[1]].wgk == 1); }

Plan make_plan(int M, int N, int K, bool tn, int n_seg, size_t part_floats, int head, int kinds) {
  Plan p = {1, {pick_tile(M, N, K, tn, head, kinds), -1}, N, 1};
  if (p.tile[0] < 0 || forced_tile() >= 0) return p;
  // Tiles of 192 and 160 add up a sum in one chain.  Where the plan without them takes the sums of some columns in parts (15 % of the
  // products that would change to them), it stays although it is slower, because one chain is further from 64 bits (fp32 results, of their
  // norm): 2304 x 2048 x 9088 in parts 2.6e-7 and 109.8 us, in tiles of 192 x 128 5.3e-7 and 94.4; 3456 x 3328 x 10240 5.0e-7 and 220 / 5.8e-7 and 187.
  if (p.tile[0] >= kNarrowTiles) {
    const Plan older = make_plan(M, N, K, tn, n_seg, part_floats, head, kNarrowTiles);
    if (!one_chain(older)) return older;
  }
  if (getenv("AH_GEMM_NOSPLIT")) return p;
  float best = 0.96f * tile_cost(p.tile[0], M, N, K, tn);  // the model's accuracy: a second launch has to promise more
  for (int s = 2; tn && s <= kMaxShares && (size_t)M * N * s <= part_floats; s++) {
    if (n_seg > 1 ? n_seg % s : K % (128 * s)) continue;
    for (int i = 0; i < kNumTiles; i++) {
      if (!tile_fits(i, M, N, K, tn, head)) continue;
      const float t = tile_cost(i, M, N, K, tn, s) + shares_cost(M, N, s);
      if (t < best) { best = t; p = {1, {i, -1}, N, s}; }
    }
  }
  for (int n0 = 128; n0 < N; n0 += 128)
    for (int i = 0; i < kNarrowTiles; i++) {
      if (!tile_fits(i, M, n0, K, tn, head)) continue;
      for (int j = 0; j < kNarrowTiles; j++) {
        if (j == i || !tile_fits(j, M, N - n0, K, tn, head)) continue;
        const float t = tile_cost(i, M, n0, K, tn) + tile_cost(j, M, N - n0, K, tn) + kSecondLaunch;
        if (t < best) { best = t; p = {2, {i, j}, n0, 1}; }
      }
    }
  return p;
}

float plan_cost(const Plan& p, int M, int N, int K, bool tn) {
  if (p.shares > 1) return tile_cost(p.tile[0], M, N, K, tn, p.shares) + shares_cost(M, N, p.shares);
  return p.parts == 1 ? tile_cost(p.tile[0], M, N, K, tn)
                      : tile_cost(p.tile[0], M, p.n0, K, tn) + tile_cost(p.tile[1], M, N - p.n0, K, tn) + kSecondLaunch;
}

// make_plan is a search over a few thousand candidates: remembered per problem
Plan cached_plan(int M, int N, int K, bool tn, int n_seg = 1, size_t part_floats = 0, int head = 0, int kinds = kNumTiles) {
  struct Entry { int M, N, K; bool tn; int n_seg; size_t part_floats; int head, kinds; Plan p; };
  static std::mutex mu;
  static std::vector<Entry> cache;
  std::lock_guard<std::mutex> lock(mu);
  for (const Entry& e : cache)
    if (e.M == M && e.N == N && e.K == K && e.tn == tn && e.n_seg == n_seg && e.part_floats == part_floats && e.head == head &&
        e.kinds == kinds)
      return e.p;
  const Plan p = make_plan(M, N, K, tn, n_seg, part_floats, head, kinds);
  if (cache.size() < 4096) cache.push_back({M, N, K, tn, n_seg, part_floats, head, kinds, p});
  return p;
}

// Tile rows per raster group.  Four: the 32 tiles an XCD has in flight then read 4 panels of A and 8 of B (8 and 4 have the
// same size but took 0.5 % longer on the 7B shard's layer, 1 % on the 13B and LLaMA-style layers; 2, 3, 5, 6 and 16 rows
// are no better there).  A last group of one or two rows would read the whole of B for itself: where that is a fair part
// of the output, the rows are spread evenly instead (forward and input gradients, geometric means over 18 .. 188 products
// against groups of four: 5 rows 0.965, 6 0.975, 9 0.978, 10 0.983; 640 x 4096 x 1152 14.8 -> 12.5 us, 1152 x 4096 x 1280 22.4 -> 20.2.  Weight gradients
// 0.990 .. 1.002; 7 and 11 rows 0.998 .. 1.004, 13 and more 0.993 .. 1.03, so those keep groups of four).
int raster_rows(int tiles_m) {
  if (tiles_m >= 12 || tiles_m % 4 == 0 || tiles_m % 4 == 3) return 4;
  const int groups = std::max(tiles_m / 4, 1);
  return (tiles_m + groups - 1) / groups;
}

template <int BM, int BN, int WGM, int WGN, int WGK, bool AKS, bool BKS, int EPI, int DEPTH = 2>
hipError_t run(GemmArgs a, hipStream_t s) {
  if (a.group <= 0) a.group = raster_rows(a.M / BM);
  dim3 grid((a.M / BM) * (a.N / BN) * (AKS && BKS && EPI == EPI_F32_SET ? a.k_shares : 1));
  hipLaunchKernelGGL((gemm_kernel<BM, BN, WGM, WGN, WGK, AKS, BKS, EPI, DEPTH>), grid, dim3(64 * WGM * WGN * WGK), 0, s, a);
  return hipGetLastError();
}

template <bool AKS, bool BKS, int EPI>
hipError_t run_tile(int t, const GemmArgs& a, hipStream_t s) {
  switch (t) {
    case 0: return run<256, 256, 2, 2, 1, AKS, BKS, EPI>(a, s);
    // (depth 3 of the forward and input-gradient tiles: see k64; the weight gradient's pipeline has no such choice)
    case 1: return run<256, 128, 2, 2, 1, AKS, BKS, EPI, 3>(a, s);
    case 2: return run<128, 256, 2, 2, 1, AKS, BKS, EPI, 3>(a, s);
    case 3:
      if constexpr (!(AKS && BKS)) {
        if (!a.beside && (a.M / 128) * (a.N / 128) <= 256) return run<128, 128, 2, 2, 1, AKS, BKS, EPI, 3>(a, s);
      }
      return run<128, 128, 2, 2, 1, AKS, BKS, EPI>(a, s);
    case kWholeCuTile:
      if constexpr (!(AKS && BKS)) return run<128, 128, 1, 1, 4, AKS, BKS, EPI>(a, s);
      else return hipErrorInvalidValue;
    case 5: return run<64, 128, 1, 2, 2, AKS, BKS, EPI>(a, s);
    case 7: case 8: case 9: case 10: case 11:
      if constexpr (!(AKS && BKS) && EPI != EPI_ROPE) {
        if (t == 7) return run<256, 192, 2, 2, 1, AKS, BKS, EPI>(a, s);
        if (t == 8) return run<256, 160, 2, 2, 1, AKS, BKS, EPI>(a, s);
        if (t == 9) return run<192, 256, 2, 2, 1, AKS, BKS, EPI>(a, s);
        if (t == 10) return run<192, 128, 2, 2, 1, AKS, BKS, EPI, 3>(a, s);
        return run<128, 192, 2, 2, 1, AKS, BKS, EPI, 3>(a, s);
      } else {
        return hipErrorInvalidValue;
      }
    default: return run<64, 64, 1, 1, 4, AKS, BKS, EPI>(a, s);
  }
}

}  // namespace

// The rotary kernel reads and writes the rotated columns once more (and rounds them once more); tiles whose waves hold
// whole heads, where the output would take others, cost more than that only on the smallest outputs (128-wide heads,
// fused against kernel, us a layer: 128 rows x 256 hidden 36.6 / 32.5, 384 x 640 46.3 / 41.5, 1024 x 1024 61.1 / 62.3,
// 4096 x 1024 116.8 / 126.1).
// Compared are the tiles that hold heads with the others of their kind.  Those of 192 and 160, which are not built with this epilogue,
// stay out: with them `any` is cheap enough that 93 of 2496 stages (128 .. 4096 rows x 256 .. 5120 hidden) would give up the rotation
// on the fp32 sums for a narrower tile and round q and k to 16 bits before it: at 512 rows x 4096 hidden a layer of 919 instead of 934 us whose
// y is 5.41e-3 instead of 5.06e-3 from 64 bits, at 1920 x 2048 635 / 649 us, 3.07e-3 / 3.05e-3.
bool gemm_rope_pays(int M, int N, int K, int d, int rope_cols) {
  if (!gemm_shape_ok(M, N, K) || d <= 0 || d % 16) return false;
  const Plan heads = cached_plan(M, N, K, false, 1, 0, d), any = cached_plan(M, N, K, false, 1, 0, 0, kNarrowTiles);
  if (heads.tile[0] < 0) return false;
  return plan_cost(heads, M, N, K, false) <= plan_cost(any, M, N, K, false) + 3.f + (float)M * rope_cols * 4.f / 4.5e6f;
}

bool gemm_plan(GemmLayout layout, int M, int N, int K, int n_seg, size_t part_floats, int head, GemmPlanInfo* out) {
  if (!gemm_shape_ok(M, N, K)) return false;
  const bool tn = layout == GEMM_TN;
  const Plan p = cached_plan(M, N, K, tn, tn ? n_seg : 1, tn ? part_floats : 0, head);
  if (p.tile[0] < 0) return false;
  *out = {p.parts, p.shares, {p.n0, N - p.n0}, {}, {}, {}, {}};
  for (int i = 0; i < p.parts; i++) {
    const TileCfg& t = kTiles[p.tile[i]];
    out->bm[i] = t.bm;
    out->bn[i] = t.bn;
    out->wgk[i] = t.wgk;
    out->raster[i] = raster_rows(M / t.bm);
  }
  return true;
}

GemmTime gemm_wgrad_time(int M, int N, int K, int n_seg, size_t part_floats) {
  if (!gemm_shape_ok(M, N, K)) return {};
  const Plan p = cached_plan(M, N, K, true, n_seg, part_floats);
  if (p.tile[0] < 0) return {};
  GemmTime t = {plan_cost(p, M, N, K, true), 0.f, 0.f};
  for (int i = 0; i < p.parts; i++) {
    const TileCfg& c = kTiles[p.tile[i]];
    const int n = p.parts == 1 ? N : i ? N - p.n0 : p.n0;
    const long tiles = (long)(M / c.bm) * (n / c.bn) * p.shares, rounds = (tiles + 255) / 256;
    const float us = t.us * n / N;
    if (c.bm * c.bn <= 128 * 128) t.room_us += us;    // (the 128 x 128 tile with four k shares is not built for this product)
    else t.idle_us += us * (1.f - (float)tiles / (256 * rounds));
  }
  return t;
}

size_t gemm_k_part_floats(int M, int N, int K, int n_seg) {
  if (!gemm_shape_ok(M, N, K)) return 0;
  const Plan p = cached_plan(M, N, K, true, n_seg, (size_t)M * N * kMaxShares);
  return p.shares > 1 ? (size_t)M * N * p.shares : 0;
}

namespace {

hipError_t dispatch(GemmLayout layout, GemmEpilogue epi, int t, const GemmArgs& a, hipStream_t s) {
  if (layout == GEMM_NN) {
    if (epi == EPI_BF16) return run_tile<false, true, EPI_BF16>(t, a, s);
    if (epi == EPI_GELU) return run_tile<false, true, EPI_GELU>(t, a, s);
    if (epi == EPI_RESID) return run_tile<false, true, EPI_RESID>(t, a, s);
    if (epi == EPI_RESID_F32) return run_tile<false, true, EPI_RESID_F32>(t, a, s);
    if (epi == EPI_RESID_F32_OUT16) return run_tile<false, true, EPI_RESID_F32_OUT16>(t, a, s);
    if (epi == EPI_SWIGLU) return run_tile<false, true, EPI_SWIGLU>(t, a, s);
    if (epi == EPI_ROPE) return run_tile<false, true, EPI_ROPE>(t, a, s);
  } else if (layout == GEMM_NT) {
    if (epi == EPI_BF16) return run_tile<false, false, EPI_BF16>(t, a, s);
    if (epi == EPI_GELU_BWD) return run_tile<false, false, EPI_GELU_BWD>(t, a, s);
    if (epi == EPI_SWIGLU_BWD) return run_tile<false, false, EPI_SWIGLU_BWD>(t, a, s);
  } else if (layout == GEMM_TN) {
    if (epi == EPI_F32_ACC) return a.beta ? run_tile<true, true, EPI_F32_ACC>(t, a, s) : run_tile<true, true, EPI_F32_SET>(t, a, s);
  }
  return hipErrorInvalidValue;
}

// the same problem restricted to output columns [c0, c0 + n)
GemmArgs column_range(GemmLayout layout, GemmEpilogue epi, const GemmArgs& a, int c0, int n) {
  GemmArgs b = a;
  b.N = n;
  if (epi == EPI_SWIGLU) {  // c0 tile columns stand for c0 / 2 logical ones of each of gate, up and the product
    b.B = (const bf16*)a.B + c0 / 2;
    b.C = (bf16*)a.C + c0 / 2;
    b.C2 = (bf16*)a.C2 + c0 / 2;
    return b;
  }
  const bool f32 = layout == GEMM_TN || epi == EPI_RESID_F32;
  const bool aux_f32 = epi == EPI_RESID_F32 || epi == EPI_RESID_F32_OUT16;
  b.C = f32 ? (void*)((float*)a.C + c0) : (void*)((bf16*)a.C + c0);
  if (a.C2) b.C2 = (bf16*)a.C2 + c0;
  if (a.bias) b.bias = (const bf16*)a.bias + c0;
  if (a.aux) b.aux = aux_f32 ? (const void*)((const float*)a.aux + c0) : (const void*)((const bf16*)a.aux + c0);
  if (a.colsum_part) b.colsum_part = a.colsum_part + c0;
  b.rope_cols = a.rope_cols - c0;  // the rotated columns are counted from the launch's first column
  if (layout == GEMM_NT) {
    b.B = (const bf16*)a.B + (size_t)c0 * a.ldb;  // B is [N, K]
  } else {
    b.B = (const bf16*)a.B + c0;                  // B is [K, N]
    for (int i = 0; i < std::max(a.n_seg, 1); i++) b.segB[i] = (const bf16*)a.segB[i] + c0;
  }
  return b;
}

}  // namespace

namespace {

// Checks a problem and sets what the kernels expect beside it.
bool complete(GemmLayout layout, GemmArgs& a) {
  static int grp = -1, remap = -1;
  if (grp < 0) { grp = getenv("AH_GEMM_GROUP") ? atoi(getenv("AH_GEMM_GROUP")) : 0; remap = getenv("AH_GEMM_NOREMAP") ? 0 : 1; }
  a.group = grp; a.xcd_remap = remap;
  if (!gemm_shape_ok(a.M, a.N, a.K)) return false;
  if (a.n_seg != 0) {  // pieces along k: weight-gradient layout only, and the pieces must add up to K
    if (layout != GEMM_TN || !gemm_segments_ok(a.seg_k, a.n_seg) || (long)a.seg_k * a.n_seg != a.K) return false;
    for (int i = 0; i < a.n_seg; i++)
      if (!a.segA[i] || !a.segB[i]) return false;
    a.A = a.segA[0];
    a.B = a.segB[0];
  } else {
    a.segA[0] = a.A;
    a.segB[0] = a.B;
  }
  a.k_shares = 1;
  return true;
}

template <int BM, int BN, int WGM, int WGN, int WGK>
hipError_t run_group(const GemmArgs* p, int n, hipStream_t s) {
  GemmGroup gg;
  gg.count = n;
  gg.first[0] = 0;
  for (int i = 0; i < n; i++) {
    gg.p[i] = p[i];
    if (gg.p[i].group <= 0) gg.p[i].group = raster_rows(p[i].M / BM);
    gg.first[i + 1] = gg.first[i] + (p[i].M / BM) * (p[i].N / BN);
  }
  const dim3 grid(gg.first[n]), block(64 * WGM * WGN * WGK);
  if (p[0].beta) hipLaunchKernelGGL((gemm_group_kernel<BM, BN, WGM, WGN, WGK, EPI_F32_ACC>), grid, block, 0, s, gg);
  else hipLaunchKernelGGL((gemm_group_kernel<BM, BN, WGM, WGN, WGK, EPI_F32_SET>), grid, block, 0, s, gg);
  return hipGetLastError();
}

}  // namespace

// The tile is one for all products: they share the k axis, so their tiles take the same time, and a launch of all of them
// is priced like one of a single product with as many.  A layer's four products together fill whole rounds where each by
// itself leaves CUs idle (BERT-Large: 16, 48, 64 and 64 tiles of 256 x 256), and small ones pay for one launch.  Stage steps, one by
// one / together: smallest 353.0 / 322.6 us, 5-head stage (pairs) 254.7 / 236.7, BERT-Large layer 3744 / 3651, 1.3B 6387 / 6274, 7B
// shard 17608 / 17453; over 40 random stages with groups of 2 .. 8 0.956 (geometric mean, worst 1.002), over 40 with pairs 0.903
// (0.978).
int gemm_group_tile(const GemmShape* p, int n, int K, int n_seg, size_t part_floats) {
  if (n < 2 || n > kMaxGemmGroup || forced_tile() >= 0 || getenv("AH_GEMM_SEPARATE")) return -1;  // (the variable: tuning and test aid)
  float separate = 0.f;
  for (int i = 0; i < n; i++) {
    if (!gemm_shape_ok(p[i].M, p[i].N, K)) return -1;
    separate += plan_cost(cached_plan(p[i].M, p[i].N, K, true, n_seg, part_floats), p[i].M, p[i].N, K, true);
  }
  int best = -1;
  float best_t = separate;
  for (int t = 0; t < kNumTiles; t++) {
    long tiles = 0;
    bool fits = true;
    for (int i = 0; i < n; i++) {
      fits = fits && tile_fits(t, p[i].M, p[i].N, K, true, 0);
      tiles += (long)(p[i].M / kTiles[t].bm) * (p[i].N / kTiles[t].bn);
    }
    if (!fits) continue;
    const float us = launch_cost(t, tiles, K, true);
    if (us < best_t) { best = t; best_t = us; }
  }
  return best;
}

hipError_t launch_gemm_group(int tile, const GemmArgs* p_in, int n, hipStream_t s) {
  if (n < 1 || n > kMaxGemmGroup) return hipErrorInvalidValue;
  GemmArgs p[kMaxGemmGroup];
  for (int i = 0; i < n; i++) {
    p[i] = p_in[i];
    if (!complete(GEMM_TN, p[i]) || p[i].K != p[0].K || p[i].beta != p[0].beta || tile < 0 || tile >= kNumTiles ||
        !tile_fits(tile, p[i].M, p[i].N, p[i].K, true, 0))
      return hipErrorInvalidValue;
  }
  switch (tile) {
    case 0: return run_group<256, 256, 2, 2, 1>(p, n, s);
    case 1: return run_group<256, 128, 2, 2, 1>(p, n, s);
    case 2: return run_group<128, 256, 2, 2, 1>(p, n, s);
    case 3: return run_group<128, 128, 2, 2, 1>(p, n, s);
    case 5: return run_group<64, 128, 1, 2, 2>(p, n, s);
    default: return run_group<64, 64, 1, 1, 4>(p, n, s);
  }
}

hipError_t launch_gemm(GemmLayout layout, GemmEpilogue epi, const GemmArgs& a_in, hipStream_t s) {
  GemmArgs a = a_in;
  if (!complete(layout, a)) return hipErrorInvalidValue;
  const bool tn = layout == GEMM_TN;
  Plan p = cached_plan(a.M, a.N, a.K, tn, std::max(a.n_seg, 1), tn && a.k_part ? a.k_part_floats : 0,
                       epi == EPI_ROPE ? a.rope_d : 0);
  // Beside a second stream's weight gradients the CUs that larger tiles leave idle are not lost: 13B layer 3478 -> 3360 us with the
  // older tiles there, 1536-wide LLaMA-style stage 1747 -> 1708.  They add up a sum in the same order (make_plan), which the column
  // sums of the GeLU derivative are not, so the bits do not depend on the streams.
  if (a.beside && p.tile[0] >= kNarrowTiles && !a.colsum_part) p = cached_plan(a.M, a.N, a.K, tn, 1, 0, 0, kNarrowTiles);
  if (p.tile[0] < 0) return hipErrorInvalidValue;
  if (p.shares > 1) {
    GemmArgs b = a;
    b.k_shares = p.shares;
    b.beta = 0;
    hipError_t e = dispatch(layout, epi, p.tile[0], b, s);
    if (e != hipSuccess) return e;
    const size_t n4 = (size_t)a.M * a.N / 4;
    hipLaunchKernelGGL(k_shares_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, a.k_part, (float*)a.C, a.M, a.N, a.ldc, p.shares, a.beta);
    return hipGetLastError();
  }
  if (p.parts == 1) return dispatch(layout, epi, p.tile[0], a, s);
  hipError_t e = dispatch(layout, epi, p.tile[0], column_range(layout, epi, a, 0, p.n0), s);
  if (e != hipSuccess) return e;
  return dispatch(layout, epi, p.tile[1], column_range(layout, epi, a, p.n0, a.N - p.n0), s);
}

}  // namespace ah
