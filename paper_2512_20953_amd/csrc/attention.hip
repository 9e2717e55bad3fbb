// Fused self-attention (causal or bidirectional) for gfx950, forward and backward, on the packed
// projection output qkv[T, 3*nh*d] ([Q | K | V], head-major).  No S x S matrix
// ever reaches HBM: scores are produced tile by tile with MFMA 32x32x16, the
// softmax runs in fp32 registers (base-2 exponent), and the backward pass
// rebuilds the probabilities from the saved log-sum-exp.
//
// All products are computed "transposed" (keys or head-dim along the MFMA row
// axis, one query or one key per lane), so that
//   - every per-row softmax quantity is a per-lane scalar, and
//   - an accumulator tile converts to the next product's bf16 operand in
//     place: the 8 values a lane holds for a 16-wide contraction step are the
//     operand's 8 slots; the other operand is fetched from LDS in the matching
//     slot order with the transposing LDS read.
// Tiles of 64 rows of K, V (or Q, dO) are staged through LDS by direct
// global->LDS loads into a ring of two to four slots, one to three tiles ahead, and are waited
// for by count, with one block barrier per tile.
//
// Backward is two deterministic kernels (no atomics): one block per 128
// queries accumulates dQ over the key tiles at or before it and leaves
// delta = rowsum(dO * O) of its queries behind, negated; one block per 128 keys then
// accumulates dK and dV over the query tiles at or after it (causal; without
// the mask both walk every tile of the sequence).
#include "common.h"
#include "kernels.h"
#include <cfloat>
#include <cstdlib>
#include <type_traits>

namespace ah {
namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr int NSLOT = 2;  // ring slots of the kernels that take one tile after the other, and of the 64-row forward kernel

// nothing is scheduled across this point
#define AH_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
// Issue priority of the wave among the waves of its SIMD: raised for the runs of matrix instructions, so that the
// other waves' vector work (softmax, masks, conversions) fills in behind them instead of delaying them.  Used by the unmasked
// 64-wide forward kernel, with / without: 8 x 16 x 512 12.6 / 13.4 us, 2 x 16 x 2048 38.2 / 40.6, 1 x 9 x 4096 56.7 / 68.2, 1 x 32 x 4096
// 141.5 / 145.5, 16 x 16 x 512 24.8 / 24.1; the kernels that run in slots gain nothing from it.
#define AH_PRIO(p) __builtin_amdgcn_s_setprio(p)

// All but the last n of the wave's loads have landed, for the whole block, and every wave is done with its LDS reads.  The
// empty statement keeps the compiler from moving LDS reads above the barrier: it does not know that the loads (which
// are assembly) write what they read.
#define AH_LANDED(n)                                  \
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(n));    \
  __builtin_amdgcn_s_barrier();                       \
  asm volatile("" ::: "memory")
#define AH_NEXT_TILE() AH_LANDED(0)

// LDS tile [64 rows][D] bf16.  16-byte piece p of row r is stored at piece
// swz(r, p): conflict-free both for 16-byte reads down a column of pieces (16 rows
// at a time must hit 16 different pieces of the 256 bytes that the banks span) and
// for the transposing reads of 4 rows x 64 bytes.  With D = 64 the banks hold two
// rows: rows 2i and 2i + 1 share a permutation, the eight values of i have eight
// different ones, and the low bit of i moves a piece to the other 64 bytes.
template <int D>
__device__ __forceinline__ int swz(int r, int p) {
  if (D == 128) return p ^ ((r & 3) << 2) ^ ((r >> 2) & 3);
  return p ^ ((r << 1) & 4) ^ ((r >> 2) & 3);
}

template <int D>
__device__ __forceinline__ uint32_t tile_src_offset(int chunk, int lane, int ld) {
  constexpr int RB = 2 * D;
  const int pos = chunk * 1024 + lane * 16;
  const int r = pos / RB, q = (pos % RB) >> 4;
  return (uint32_t)(r * ld + swz<D>(r, q) * 8) * 2u;  // bytes
}

// The loads into LDS as assembly: for the builtin the compiler assumes an access that may return out of order with LDS
// reads, and waits for all of a wave's LDS reads (lgkmcnt(0)) before the first use of any of them while such a load is in
// flight.  Nothing is returned to a register; the kernels wait for these loads by count before they pass a barrier.  M0 (the
// LDS address) is set in the same statement and named as overwritten.  Against the builtin, forward / backward:
// 2 x 16 x 2048 x 128 causal 51.1 / 163.2 -> 49.7 / 160.2 us, 2 x 16 x 2048 x 64 causal 29.5 / 86.4 -> 28.7 / 83.0 (same bits).
__device__ __forceinline__ void load4(const void* base, uint32_t off, void* lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_offset(lds)), "v"(off), "s"(base) : "memory", "m0");
}

template <int D>
__device__ __forceinline__ void issue_tile(const bf16* __restrict__ g, const uint32_t* off, char* lds, int wave) {
#pragma unroll
  for (int i = 0; i < D / 32; i++) load16_to_lds_uncounted(g, off[i], lds + (wave + 4 * i) * 1024);
}

// 32 rows
template <int D>
__device__ __forceinline__ void issue_half(const bf16* __restrict__ g, const uint32_t* off, char* lds, int wave) {
#pragma unroll
  for (int i = 0; i < D / 64; i++) load16_to_lds_uncounted(g, off[i], lds + (wave + 4 * i) * 1024);
}

// 8 consecutive head-dim values (k-step ks, half hf) of row r
template <int D>
__device__ __forceinline__ bf16x8 frag_rowmajor(const char* __restrict__ t, int r, int ks, int hf) {
  return *(const bf16x8*)(t + r * (2 * D) + swz<D>(r, 2 * ks + hf) * 16);
}

// column (dt*32 + lane%32) of rows rbase..rbase+3 and rbase+8..rbase+11
template <int D>
__device__ __forceinline__ bf16x8 frag_transposed(const char* __restrict__ t, int rbase, int dt, int lane) {
  const int r = rbase + ((lane & 15) >> 2);
  const int c = dt * 32 + ((lane >> 4) & 1) * 16 + 4 * (lane & 3);
  bf16x4 lo = lds_read_tr4(t + r * (2 * D) + swz<D>(r, c >> 3) * 16 + (c & 7) * 2);
  bf16x4 hi = lds_read_tr4(t + (r + 8) * (2 * D) + swz<D>(r + 8, c >> 3) * 16 + (c & 7) * 2);
  return cat4(lo, hi);
}

__device__ __forceinline__ bf16x8 pack8(const f32x16& a, int s2) {
  bf16x8 p;
#pragma unroll
  for (int j = 0; j < 8; j++) p[j] = f2bf(a[8 * s2 + j]);
  return p;
}

// max / sum of a value over the two lanes (l, l + 32) that share a query: one exchange of the halves of two registers
// instead of a trip through the LDS crossbar
__device__ __forceinline__ float half_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// A wave's result of 32 rows x D, val(dt, r) being the element of row lane % 32 and column dt * 32 + 8 (r / 4) + 4 (lane / 32) + r % 4,
// to 32 rows of the output.  It passes through a strip of LDS of the wave's own and leaves as whole rows, 16 bytes a lane: stored
// straight from the registers, an instruction writes 16 bytes to each of 32 rows (dK and dV of 128 keys: 4.5 us, now 1.45).
template <int D> constexpr int strip_bytes() { return 32 * 2 * D; }
template <int D, class F>
__device__ __forceinline__ void store_rows(const F& val, char* strip, bf16* __restrict__ dst, size_t ld, int lane) {
  constexpr int RB = 2 * D, PPR = D / 8, RPI = 64 / PPR;   // bytes of a row, 16-byte pieces of a row, rows per store
  auto at = [](int row, int piece) { return row * RB + ((piece ^ (D == 128 ? row : row >> 1)) & (PPR - 1)) * 16; };
  const int base = at(lane & 31, 0) + 8 * (lane >> 5);
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; i++) v[i] = f2bf(val(dt, 4 * g + i));
      *(bf16x4*)(strip + (base ^ ((4 * dt + g) * 16))) = v;
    }
  __builtin_amdgcn_wave_barrier();
  const int row = lane / PPR, piece = lane % PPR;
#pragma unroll
  for (int it = 0; it < 32 / RPI; it++) *(bf16x8*)(dst + (size_t)(row + it * RPI) * ld + piece * 8) = *(const bf16x8*)(strip + at(row + it * RPI, piece));
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Query block of a thread block under the causal mask (block qb walks 2*qb + 2 key tiles).  A launch that
// fits on the chip at once (two blocks per CU, 256 CUs) is placed statically, blocks i and i + grid/2 on
// the same CU, so the second half of the grid runs the light blocks in ascending order and every CU gets
// the same total; a larger launch is dispatched as CUs free up and simply goes heaviest first.
__device__ __forceinline__ int causal_query_block(int r, int nq) {
  if (gridDim.x > 512) return nq - 1 - r;
  const int half = (nq + 1) / 2;
  return r < half ? nq - 1 - r : r - half;
}

// =========================================================================== forward
template <int D>
struct FwdState {
  bf16x8 qf[D / 16];
  f32x16 oacc[D / 32];
  float m, l;
  __device__ __forceinline__ void load(const bf16* __restrict__ qrow, int hf) {
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) qf[ks] = *(const bf16x8*)(qrow + ks * 16 + hf * 8);
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) oacc[dt][r] = 0.f;
    m = -INFINITY;
    l = 0.f;
  }
  // the output rows of the wave's 32 queries (orow: the first) and the query's log-sum-exp
  __device__ __forceinline__ void store(char* strip, bf16* __restrict__ orow, size_t ldo, float* __restrict__ lse, int lane) const {
    const float sum = l + __shfl_xor(l, 32, 64);
    const float inv = 1.f / sum;
    store_rows<D>([&](int dt, int r) { return oacc[dt][r] * inv; }, strip, orow, ldo, lane);
    if (lane < 32) *lse = (m + __log2f(sum)) * LN2;
  }
};

// The running maximum is only raised when a new score exceeds it by more than this many powers of two:
// probabilities are then at most 2^8 instead of 1, which fp32 sums and the bf16 operand of the second
// product hold with unchanged relative accuracy, and the rescaling of the output accumulator -- the
// largest block of vector arithmetic in the loop -- runs on the first tile only in practice.
constexpr float RESCALE_SLACK = 8.f;

// ---- without the mask, head_dim 64: one tile after the other.  Three waves share a SIMD and all of them run to the end, so
// that they cover each other's waits; the steps below, whose first scores and last product stand alone, are level on long
// sequences there and lose on short ones (8 x 16 x 512: 17.2 against 18.0 us in a stage).
// One key tile of 64 for the wave's 32 queries.  LDS reads are issued a phase ahead of their use.
template <int D>
__device__ __forceinline__ void fwd_tile(const char* __restrict__ cK, const char* __restrict__ cV, FwdState<D>& st, float sc2,
                                         int lane) {
  constexpr int NK = D / 16, ND = D / 32;
  const int hf = lane >> 5;
  bf16x8 fk0[NK], fk1[NK];
#pragma unroll
  for (int ks = 0; ks < NK; ks++) fk0[ks] = frag_rowmajor<D>(cK, lane & 31, ks, hf);
  AH_SCHED_FENCE();
  f32x16 s0, s1;
#pragma unroll
  for (int r = 0; r < 16; r++) { s0[r] = 0.f; s1[r] = 0.f; }
  AH_PRIO(1);
#pragma unroll
  for (int ks = 0; ks < NK; ks++) s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk0[ks], st.qf[ks], s0, 0, 0, 0);
#pragma unroll
  for (int ks = 0; ks < NK; ks++) fk1[ks] = frag_rowmajor<D>(cK, 32 + (lane & 31), ks, hf);
  AH_SCHED_FENCE();
  bf16x8 v0[2][ND], v1[2][ND];
#pragma unroll
  for (int ks = 0; ks < NK; ks++) s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk1[ks], st.qf[ks], s1, 0, 0, 0);
#pragma unroll
  for (int s2 = 0; s2 < 2; s2++)
#pragma unroll
    for (int dt = 0; dt < ND; dt++) v0[s2][dt] = frag_transposed<D>(cV, 16 * s2 + 4 * hf, dt, lane);
  AH_PRIO(0);
  AH_SCHED_FENCE();
  float mx = fmaxf(s0[0], s1[0]);
#pragma unroll
  for (int r = 1; r < 16; r++) mx = fmaxf(fmaxf(mx, s0[r]), s1[r]);  // one three-way maximum each
  mx = half_max(mx) * sc2;
  if (__any(mx > st.m + RESCALE_SLACK)) {  // wave-uniform branch
    const float m_new = fmaxf(st.m, mx);
    const float alpha = fexp2(st.m - m_new);
    st.m = m_new;
    st.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < ND; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) st.oacc[dt][r] *= alpha;
  }
  const float nm = -st.m;
  float ls = 0.f;
#pragma unroll
  for (int r = 0; r < 16; r++) {
    s0[r] = fexp2(__builtin_fmaf(s0[r], sc2, nm));
    s1[r] = fexp2(__builtin_fmaf(s1[r], sc2, nm));
    ls += s0[r] + s1[r];
  }
  st.l += ls;
#pragma unroll
  for (int s2 = 0; s2 < 2; s2++)
#pragma unroll
    for (int dt = 0; dt < ND; dt++) v1[s2][dt] = frag_transposed<D>(cV, 32 + 16 * s2 + 4 * hf, dt, lane);
  AH_SCHED_FENCE();
  AH_PRIO(1);
#pragma unroll
  for (int s2 = 0; s2 < 2; s2++) {
    const bf16x8 pf = pack8(s0, s2);
#pragma unroll
    for (int dt = 0; dt < ND; dt++) st.oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v0[s2][dt], pf, st.oacc[dt], 0, 0, 0);
  }
#pragma unroll
  for (int s2 = 0; s2 < 2; s2++) {
    const bf16x8 pf = pack8(s1, s2);
#pragma unroll
    for (int dt = 0; dt < ND; dt++) st.oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v1[s2][dt], pf, st.oacc[dt], 0, 0, 0);
  }
  AH_PRIO(0);
  AH_SCHED_FENCE();
}

template <int D>
__global__ __launch_bounds__(256, 2) void attn_fwd_plain_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ o, float* __restrict__ lse,
                                                             int B, int S, int nh, float sc2) {
  constexpr int TILEB = 64 * 2 * D, STAGE = 2 * TILEB;  // ring slot = K tile then V tile
  __shared__ __attribute__((aligned(1024))) char ring[NSLOT * STAGE];
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: LDS bases stay scalar
  const int nbh = B * nh;
  const int qb = blockIdx.x / nbh, bh = blockIdx.x - qb * nbh;
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const int qw0 = qb * 128 + wave * 32, q = qw0 + (lane & 31);

  FwdState<D> st;
  st.load(qp + (size_t)q * ld, hf);
  uint32_t off[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) off[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);

  // Tile t lives in ring slot t % 2 and is loaded during step t - 1 (the last step loads the last tile again, into a dead
  // slot).  Two tiles per round (S / 64 is even), so that every LDS address is a constant away from a loop-invariant one.
  const int ntile = S / 64, last = ntile - 1;
  const size_t step = (size_t)64 * ld;
  char *const K0 = ring, *const V0 = ring + TILEB, *const K1 = ring + STAGE, *const V1 = ring + STAGE + TILEB;
  issue_tile<D>(kp, off, K0, wave);
  issue_tile<D>(vp, off, V0, wave);
  AH_NEXT_TILE();
  for (int j = 0; j < ntile; j += 2) {
    const size_t o1 = (size_t)(j + 1) * step, o2 = (size_t)min(j + 2, last) * step;
    issue_tile<D>(kp + o1, off, K1, wave);
    issue_tile<D>(vp + o1, off, V1, wave);
    fwd_tile<D>(K0, V0, st, sc2, lane);
    AH_NEXT_TILE();
    issue_tile<D>(kp + o2, off, K0, wave);
    issue_tile<D>(vp + o2, off, V0, wave);
    fwd_tile<D>(K1, V1, st, sc2, lane);
    AH_NEXT_TILE();
  }
  st.store(ring + wave * strip_bytes<D>(), o + ((size_t)b * S + qw0) * (nh * D) + head * D, nh * D, lse + ((size_t)b * nh + head) * S + q, lane);
}

// Byte offsets of a lane's fragments in a tile: row[ks] as frag_rowmajor, lo[dt] and hi[dt] as frag_transposed, for rows that
// start at a multiple of 16 (the permutation depends on the row's low four bits only), so that every other fragment is a
// compile-time distance away.
template <int D>
struct LaneOffs {
  int row[D / 16], lo[D / 32], hi[D / 32];
  __device__ __forceinline__ LaneOffs(int lane) {
    const int r = lane & 31, hf = lane >> 5, rt = 4 * hf + ((lane & 15) >> 2);
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) row[ks] = r * (2 * D) + swz<D>(r, 2 * ks + hf) * 16;
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) {
      const int c = dt * 32 + ((lane >> 4) & 1) * 16 + 4 * (lane & 3);
      lo[dt] = rt * (2 * D) + swz<D>(rt, c >> 3) * 16 + (c & 7) * 2;
      hi[dt] = (rt + 8) * (2 * D) + swz<D>(rt + 8, c >> 3) * 16 + (c & 7) * 2;
    }
  }
  __device__ __forceinline__ bf16x8 rows(const char* t, int rb, int ks) const { return *(const bf16x8*)(t + row[ks] + rb * (2 * D)); }
  __device__ __forceinline__ bf16x8 cols(const char* t, int rb, int dt) const {
    return cat4(lds_read_tr4(t + lo[dt] + rb * (2 * D)), lds_read_tr4(t + hi[dt] + rb * (2 * D)));
  }
};

// f(integral_constant<int, I>) for I .. N - 1, unrolled
template <int I, int N, class F>
__device__ __forceinline__ void unrolled(const F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<I + 1, N>(f);
  }
}

// scores of one key tile: s0, s1 = K Q^T
template <int D>
__device__ __forceinline__ void fwd_scores(const char* cK, const LaneOffs<D>& lo, const bf16x8 (&qf)[D / 16], f32x16& s0, f32x16& s1) {
#pragma unroll
  for (int r = 0; r < 16; r++) { s0[r] = 0.f; s1[r] = 0.f; }
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo.rows(cK, 0, ks), qf[ks], s0, 0, 0, 0);
    s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo.rows(cK, 32, ks), qf[ks], s1, 0, 0, 0);
  }
}

template <bool DIAG>
__device__ __forceinline__ float fwd_max(f32x16& s0, f32x16& s1, int lim) {
  if (DIAG) {
    // element r of half t is key k0 + t*32 + 8*(r/4) + 4*hf + r%4: masked iff that exceeds q (lim = q - k0 - 4 hf)
#pragma unroll
    for (int r = 0; r < 16; r++) {
      if (8 * (r >> 2) + (r & 3) > lim) s0[r] = -INFINITY;
      if (32 + 8 * (r >> 2) + (r & 3) > lim) s1[r] = -INFINITY;
    }
  }
  float mx = fmaxf(s0[0], s1[0]);
#pragma unroll
  for (int r = 1; r < 16; r++) mx = fmaxf(fmaxf(mx, s0[r]), s1[r]);  // one three-way maximum each
  return half_max(mx);
}

// ---- otherwise: a pipeline of steps.  A step takes the softmax of tile j (its scores in s0, s1, their maximum in mx), its product
// with V, and the scores of tile j + 1 (NEXT).  One probability (multiply-add, exponential, sum, half a conversion) fits under
// one matrix instruction (32 clocks; both units busy, 17 ns against 17 and 9 alone), so the step is a fixed sequence of
// slots: an LDS fragment requested AHEAD slots before its use, one matrix instruction, its share of the probabilities
// (all 32 before the products that need them), and the maximum of the new scores under the last products.  The fences
// keep the sequence as written.  A wave that is left alone on its SIMD, as the causal mask leaves the ones with the most
// keys, no longer does one thing at a time; with two, what is left to bound it is the CU's path from the LDS (320 KB of
// fragments and tiles a step at head_dim 128).  Against one phase after the other: 2 x 16 x 2048 x 128 causal 51.0 -> 46.3 us, without
// the mask 72.6 -> 69.8, 1 x 32 x 4096 x 128 causal 143.3 -> 138.3, 2 x 16 x 2048 x 64 causal 30.4 -> 27.9.  AHEAD 2 .. 7 and a raised
// issue priority change nothing; 64 queries per wave and one wave per SIMD (half the fragments) take 85 us for 69.8.
template <int D, bool NEXT, bool DIAG>
__device__ __forceinline__ void fwd_pipe(const char* nK, const char* cV, FwdState<D>& st, f32x16& s0, f32x16& s1, float& mx,
                                         const LaneOffs<D>& lo, int lim, float sc2) {
  constexpr int NK = D / 16, ND = D / 32;
  const float mxs = mx * sc2;
  if (__any(mxs > st.m + RESCALE_SLACK)) {  // wave-uniform branch
    const float m_new = fmaxf(st.m, mxs);
    const float alpha = fexp2(st.m - m_new);
    st.m = m_new;
    st.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < ND; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) st.oacc[dt][r] *= alpha;
  }
  const float nm = -st.m;
  constexpr int N1 = NEXT ? 2 * NK : 0, N2 = N1 + 2 * ND, NS = N2 + 2 * ND;  // slots: scores, then the halves of the product with V
  constexpr int SE = NEXT ? NS - ND - 2 : 0;                                 // slots over which the exponentials are spread
  static_assert(!NEXT || (15 * SE / 32 < N1 && 23 * SE / 32 < N2 && 31 * SE / 32 < NS - ND), "probabilities precede their products");
  constexpr int AHEAD = 4;                                                   // fragments requested before their use
  f32x16 t0, t1;
  bf16x8 fr[NS], pf[4];
  float ls[2] = {0.f, 0.f};
  auto fetch = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i < N1) fr[i] = lo.rows(nK, 32 * (i & 1), i >> 1);
    else if constexpr (i < NS) fr[i] = lo.cols(cV, 16 * ((i - N1) / ND), (i - N1) % ND);
  };
  auto element = [&](auto ic) {
    constexpr int e = decltype(ic)::value, r = e & 15;
    f32x16& s = e < 16 ? s0 : s1;
    s[r] = fexp2(__builtin_fmaf(s[r], sc2, nm));
    ls[e & 1] += s[r];
    if constexpr ((e & 7) == 7) pf[e >> 3] = pack8(s, (e >> 3) & 1);
  };
  if (NEXT) {
#pragma unroll
    for (int r = 0; r < 16; r++) { t0[r] = 0.f; t1[r] = 0.f; }
  } else {
    unrolled<0, 32>(element);
  }
  unrolled<0, AHEAD>(fetch);
  unrolled<0, NS>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    AH_SCHED_FENCE();
    fetch(std::integral_constant<int, i + AHEAD>{});
    if constexpr (i < N1) {
      f32x16& t = i & 1 ? t1 : t0;
      t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], st.qf[i >> 1], t, 0, 0, 0);
    } else {
      constexpr int dt = (i - N1) % ND;
      st.oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], pf[(i - N1) / ND], st.oacc[dt], 0, 0, 0);
    }
    AH_SCHED_FENCE();
    if constexpr (i < SE) unrolled<i * 32 / SE, (i + 1) * 32 / SE>(element);
    if constexpr (NEXT && i == NS - ND) mx = fwd_max<DIAG>(t0, t1, lim);
  });
  st.l += ls[0] + ls[1];
  if (NEXT) {
    s0 = t0;
    s1 = t1;
  }
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ o, float* __restrict__ lse,
                                                       int B, int S, int nh, float sc2) {
  constexpr int TILEB = 64 * 2 * D;
  __shared__ __attribute__((aligned(1024))) char ring[4 * TILEB];  // two K tiles, two V tiles
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: LDS bases stay scalar
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int qb = CAUSAL ? causal_query_block(rank, S / 128) : rank;
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const int qw0 = qb * 128 + wave * 32, q = qw0 + (lane & 31);

  uint32_t off[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) off[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);

  // Key tiles of 64 up to and including the diagonal (all of them without the mask), an even number.  K tile t lives in K slot
  // t % 2 and V tile t in V slot t % 2; step j reads K tile j + 1 and V tile j, while K tile j + 2 and V tile j + 1 arrive.  The
  // loop takes two steps per round, so that every LDS address is a constant away from a loop-invariant one; the steps
  // whose scores straddle the diagonal are peeled, so that the others have no mask in them.
  const int ntile = CAUSAL ? 2 * qb + 2 : S / 64, last = ntile - 1, nfull = CAUSAL ? ntile - 2 : ntile;
  const size_t step = (size_t)64 * ld;
  char *const K0 = ring, *const K1 = ring + TILEB, *const V0 = ring + 2 * TILEB, *const V1 = ring + 3 * TILEB;
  issue_tile<D>(kp, off, K0, wave);
  issue_tile<D>(vp, off, V0, wave);
  issue_tile<D>(kp + step, off, K1, wave);

  FwdState<D> st;
  st.load(qp + (size_t)q * ld, hf);
  const LaneOffs<D> lo(lane);
  f32x16 s0, s1;
  float mx;
  const int lim = q - 4 * hf;
  AH_NEXT_TILE();
  fwd_scores<D>(K0, lo, st.qf, s0, s1);
  if (CAUSAL && nfull == 0) mx = fwd_max<true>(s0, s1, lim);
  else mx = fwd_max<false>(s0, s1, lim);
  AH_NEXT_TILE();
  int j = 0;
#define AH_FWD_LOADS(cK, nV)                                             \
  issue_tile<D>(kp + (size_t)min(j + 2, last) * step, off, cK, wave);    \
  issue_tile<D>(vp + (size_t)(j + 1) * step, off, nV, wave)
  for (; j < nfull - 2; ) {
    AH_FWD_LOADS(K0, V1);
    fwd_pipe<D, true, false>(K1, V0, st, s0, s1, mx, lo, 0, sc2);
    AH_NEXT_TILE();
    j++;
    AH_FWD_LOADS(K1, V0);
    fwd_pipe<D, true, false>(K0, V1, st, s0, s1, mx, lo, 0, sc2);
    AH_NEXT_TILE();
    j++;
  }
  if (nfull > 0) {
    AH_FWD_LOADS(K0, V1);
    fwd_pipe<D, true, false>(K1, V0, st, s0, s1, mx, lo, 0, sc2);
    AH_NEXT_TILE();
    j++;
    if (CAUSAL) {
      AH_FWD_LOADS(K1, V0);
      fwd_pipe<D, true, true>(K0, V1, st, s0, s1, mx, lo, lim - (last - 1) * 64, sc2);
      AH_NEXT_TILE();
      j++;
    }
  }
  if (CAUSAL) {  // j == last - 1, an even tile
    issue_tile<D>(vp + (size_t)last * step, off, V1, wave);
    fwd_pipe<D, true, true>(K1, V0, st, s0, s1, mx, lo, lim - last * 64, sc2);
    AH_NEXT_TILE();
  }
  // (under the mask the first two waves see no key of the last tile: its scores are all masked)
  if (!CAUSAL || wave >= 2) fwd_pipe<D, false, false>(K0, V1, st, s0, s1, mx, lo, 0, sc2);
#undef AH_FWD_LOADS
  st.store(ring + wave * strip_bytes<D>(), o + ((size_t)b * S + qw0) * (nh * D) + head * D, nh * D, lse + ((size_t)b * nh + head) * S + q, lane);
}

// =========================================================================== forward for launches that cannot fill the chip
// With at most one 128-query block per CU a wave sits alone on its SIMD and the launch lasts as long as the block
// with the most key tiles.  Here a block takes 64 queries and its four waves split the work two ways: wave w
// owns queries 32 * (w & 1) .. + 31 and, of every 64-key tile, the keys 32 * (w >> 1) .. + 31.  There are twice as
// many blocks (two per CU, heavy ones paired with light ones) and every wave walks half the keys of its queries;
// the two partial results per query (running maximum, sum and output accumulator) meet in LDS at the end.
// The steps are those of the 128-row kernels, here and in the backward kernels but dQ at head_dim 64: 1 x 16 x 2048 x 128 causal, forward / dQ
// / dK,dV, 34.4 / 42.6 / 60.9 us one phase after the other, 32.7 / 41.0 / 57.0 now; 1 x 16 x 1024 x 64 causal, forward / dK,dV, 11.7 / 16.8
// and 11.0 / 15.3.
template <int D>
__device__ __forceinline__ void fwd_half_scores(const char* cK, const LaneOffs<D>& lo, const bf16x8 (&qf)[D / 16], f32x16& s) {
#pragma unroll
  for (int r = 0; r < 16; r++) s[r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo.rows(cK, 0, ks), qf[ks], s, 0, 0, 0);
}

// maximum over 32 keys; under the mask (lim = q - first key - 4 hf) of those the query sees
template <bool DIAG>
__device__ __forceinline__ float fwd_half_max(f32x16& s, int lim) {
  if (DIAG) {
#pragma unroll
    for (int r = 0; r < 16; r++)
      if (8 * (r >> 2) + (r & 3) > lim) s[r] = -INFINITY;
  }
  float mx = fmaxf(s[0], s[1]);
#pragma unroll
  for (int r = 2; r < 16; r += 2) mx = fmaxf(fmaxf(mx, s[r]), s[r + 1]);  // one three-way maximum each
  return half_max(mx);
}

// One step of the pipeline (see fwd_pipe) over 32 keys
template <int D, bool NEXT, bool DIAG>
__device__ __forceinline__ void fwd_half_step(const char* nK, const char* cV, FwdState<D>& st, f32x16& s, float& mx, const LaneOffs<D>& lo,
                                              int lim, float sc2) {
  constexpr int NK = D / 16, ND = D / 32;
  const float mxs = mx * sc2;
  if (__any(mxs > st.m + RESCALE_SLACK)) {  // wave-uniform branch
    const float m_new = fmaxf(st.m, mxs);
    const float alpha = fexp2(st.m - m_new);
    st.m = m_new;
    st.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < ND; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) st.oacc[dt][r] *= alpha;
  }
  const float nm = -st.m;
  constexpr int N1 = NEXT ? NK : 0, NS = N1 + 2 * ND;   // slots: scores, then the product with V
  constexpr int SE = NEXT ? N1 + ND - 1 : 0;            // slots over which the 16 probabilities are spread
  static_assert(!NEXT || (7 * SE / 16 < N1 && 15 * SE / 16 < N1 + ND), "probabilities precede their products");
  constexpr int AHEAD = 4;
  f32x16 t;
  bf16x8 fr[NS], pf[2];
  float ls = 0.f;
  auto fetch = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i < N1) fr[i] = lo.rows(nK, 0, i);
    else if constexpr (i < NS) fr[i] = lo.cols(cV, 16 * ((i - N1) / ND), (i - N1) % ND);
  };
  auto element = [&](auto ic) {
    constexpr int r = decltype(ic)::value;
    s[r] = fexp2(__builtin_fmaf(s[r], sc2, nm));
    ls += s[r];
    if constexpr ((r & 7) == 7) pf[r >> 3] = pack8(s, r >> 3);
  };
  if (NEXT) {
#pragma unroll
    for (int r = 0; r < 16; r++) t[r] = 0.f;
  } else {
    unrolled<0, 16>(element);
  }
  unrolled<0, AHEAD>(fetch);
  unrolled<0, NS>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    AH_SCHED_FENCE();
    fetch(std::integral_constant<int, i + AHEAD>{});
    if constexpr (i < N1) t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], st.qf[i], t, 0, 0, 0);
    else st.oacc[(i - N1) % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], pf[(i - N1) / ND], st.oacc[(i - N1) % ND], 0, 0, 0);
    AH_SCHED_FENCE();
    if constexpr (i < SE) unrolled<i * 16 / SE, (i + 1) * 16 / SE>(element);
    if constexpr (NEXT && i == NS - ND) mx = fwd_half_max<DIAG>(t, lim);
  });
  st.l += ls;
  if (NEXT) s = t;
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_fwd64_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ o, float* __restrict__ lse,
                                                         int B, int S, int nh, float sc2) {
  constexpr int TILEB = 64 * 2 * D, STAGE = 2 * TILEB, ND = D / 32;
  __shared__ __attribute__((aligned(1024))) char ring[NSLOT * STAGE];
  static_assert(2 * (ND * 16 + 2) * 64 * 4 <= NSLOT * STAGE, "the partial results of two waves fit in the ring");
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qt = wave & 1, kh = wave >> 1;
  const int nq = S / 64;
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int qb = CAUSAL ? causal_query_block(rank, nq) : rank;
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const int qw0 = qb * 64 + qt * 32, q = qw0 + (lane & 31);

  FwdState<D> st;
  st.load(qp + (size_t)q * ld, hf);

  uint32_t off[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) off[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);

  // Key tiles of 64 up to and including the one that holds the block's own keys, one step of the pipeline each (the wave's half of
  // it).  K tile t lives in K slot t % 2 and V tile t in V slot t % 2; step j reads K tile j + 1 and V tile j, while K tile
  // j + 2 and V tile j + 1 arrive.
  st.m = -FLT_MAX;   // finite: in the block's own tile a wave may see no key at all
  const int ntile = CAUSAL ? qb + 1 : nq, last = ntile - 1, k0 = 32 * kh;
  const size_t step = (size_t)64 * ld;
  auto load_k = [&](int t) { issue_tile<D>(kp + (size_t)min(t, last) * step, off, ring + (t & 1) * TILEB, wave); };
  auto load_v = [&](int t) { issue_tile<D>(vp + (size_t)min(t, last) * step, off, ring + (2 + (t & 1)) * TILEB, wave); };
  auto slot_k = [&](int t) { int x = (t & 1) * TILEB; asm("" : "+s"(x)); return (const char*)ring + x + k0 * (2 * D); };
  auto slot_v = [&](int t) { int x = (2 + (t & 1)) * TILEB; asm("" : "+s"(x)); return (const char*)ring + x + k0 * (2 * D); };
  load_k(0);
  load_v(0);
  load_k(1);
  const LaneOffs<D> lo(lane);
  f32x16 s;
  const int lim = q - k0 - 4 * hf;
  AH_NEXT_TILE();
  fwd_half_scores<D>(slot_k(0), lo, st.qf, s);
  float mx = CAUSAL && last == 0 ? fwd_half_max<true>(s, lim) : fwd_half_max<false>(s, 0);
  AH_NEXT_TILE();   // the first K tile's slot is loaded next
  int j = 0;
#define AH_FWD_STEP(MASK, limit)                                                              \
  load_k(j + 2);                                                                              \
  load_v(j + 1);                                                                              \
  fwd_half_step<D, true, MASK>(slot_k(j + 1), slot_v(j), st, s, mx, lo, limit, sc2);          \
  AH_NEXT_TILE();                                                                             \
  j++
#pragma unroll 1
  while (j < (CAUSAL ? last - 1 : last)) { AH_FWD_STEP(false, 0); }
  if (CAUSAL && last > 0) { AH_FWD_STEP(true, lim - last * 64); }
#undef AH_FWD_STEP
  // (a wave that sees no key of the block's own tile skips it: see the 128-row dK/dV kernel)
  if (!CAUSAL || qt >= kh) fwd_half_step<D, false, false>(slot_k(last), slot_v(last), st, s, mx, lo, 0, sc2);
  __syncthreads();

  // merge: the waves of the second key half leave (m, l, O) in LDS, lane by lane; the others fold them in
  float* mg = (float*)ring + (size_t)qt * (ND * 16 + 2) * 64;
  if (kh == 1) {
#pragma unroll
    for (int dt = 0; dt < ND; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) mg[(dt * 16 + r) * 64 + lane] = st.oacc[dt][r];
    mg[(ND * 16) * 64 + lane] = st.m;
    mg[(ND * 16 + 1) * 64 + lane] = st.l;
  }
  __syncthreads();
  if (kh == 1) return;
  const float m2 = mg[(ND * 16) * 64 + lane], l2 = mg[(ND * 16 + 1) * 64 + lane];
  const float m = fmaxf(st.m, m2);
  const float a1 = fexp2(st.m - m), a2 = fexp2(m2 - m);  // m2 = -FLT_MAX (nothing visible in that half) gives a2 = 0
  const float lsum = a1 * st.l + a2 * l2;
  const float l = lsum + __shfl_xor(lsum, 32, 64);
  const float inv = 1.f / l;
  bf16* op = o + ((size_t)b * S + q) * (nh * D) + head * D;
#pragma unroll
  for (int dt = 0; dt < ND; dt++)
#pragma unroll
    for (int g = 0; g < 4; g++) {
      bf16x4 v;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int r = 4 * g + i;
        v[i] = f2bf((a1 * st.oacc[dt][r] + a2 * mg[(dt * 16 + r) * 64 + lane]) * inv);
      }
      *(bf16x4*)(op + dt * 32 + 8 * g + 4 * hf) = v;
    }
  if (hf == 0) lse[((size_t)b * nh + head) * S + q] = (m + __log2f(l)) * LN2;
}

// =========================================================================== backward: dQ (one block per 128 queries)
// delta_q = sum_c dO[q, c] O[q, c] for the lane's query: the lane holds half of the row of dO as MFMA fragments
// (columns ks * 16 + hf * 8 ..), reads the same columns of O, and the two lanes of a query add their halves.
// The dQ kernels compute it for their own queries and leave it in `delta` for the dK/dV kernel, which runs after them.
template <int D>
__device__ __forceinline__ float row_delta(const bf16x8 (&dof)[D / 16], const bf16* __restrict__ orow, int hf) {
  float s = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    const bf16x8 ov = *(const bf16x8*)(orow + ks * 16 + hf * 8);
#pragma unroll
    for (int j = 0; j < 8; j++) s = __builtin_fmaf(bf2f(dof[ks][j]), bf2f(ov[j]), s);
  }
  return s + __shfl_xor(s, 32, 64);
}

template <int D>
struct DqState {
  bf16x8 qf[D / 16], dof[D / 16];
  f32x16 acc[D / 32];
  float lse2, delta;
  // token: the query's row of o and d_o; row: its place in lse and delta
  __device__ __forceinline__ void load(const bf16* __restrict__ qrow, const bf16* __restrict__ o, const bf16* __restrict__ d_o,
                                       const float* __restrict__ lse, float* __restrict__ dlt, size_t token, size_t row, int head, int nh,
                                       int hf, bool keep) {
    const size_t at = token * (nh * D) + head * D;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) {
      qf[ks] = *(const bf16x8*)(qrow + ks * 16 + hf * 8);
      dof[ks] = *(const bf16x8*)(d_o + at + ks * 16 + hf * 8);
    }
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[dt][r] = 0.f;
    lse2 = lse[row] * LOG2E;
    delta = row_delta<D>(dof, o + at, hf);
    if (hf == 0 && keep) dlt[row] = -delta;  // negated: what the dK/dV kernel starts dP from
  }
};

// ---- head_dim 128: a pipeline of steps over 32 keys, in slots as in the forward kernel (the 256 registers of a wave leave no room for
// 64): 2 x 16 x 2048 causal 79.7 -> 70.2 us, without the mask 99.9 -> 96.9 (one tile of 64 keys after the other, its fragments
// fetched where they were used).
// One step: dS of the keys whose scores S and dP - delta are in s, dp (K
// rows at cK), its product with K, and S and dP - delta of the next 32 keys (rows at nK, nV).
template <int D, bool MASK>
__device__ __forceinline__ void dq_step(const char* cK, const char* nK, const char* nV, DqState<D>& st, f32x16& s, f32x16& dp,
                                        const LaneOffs<D>& lo, int lim, float sc2) {
  constexpr int NK = D / 16, ND = D / 32;
  constexpr int N1 = 2 * NK, NS = N1 + 2 * ND;   // slots: S and dP by turns, then dQ
  constexpr int SE = NS - ND - 2;                // slots over which the 16 elements are spread
  static_assert(15 * SE / 16 < NS - ND && 7 * SE / 16 < N1, "dS precedes its product");
  constexpr int AHEAD = 4;
  f32x16 ns, ndp;
#pragma unroll
  for (int r = 0; r < 16; r++) { ns[r] = 0.f; ndp[r] = -st.delta; }   // the product dO V^T lands on -delta: dP - delta for free
  bf16x8 fr[NS], dsf[2];
  auto fetch = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i < N1) fr[i] = lo.rows(i & 1 ? nV : nK, 0, i >> 1);
    else if constexpr (i < NS) fr[i] = lo.cols(cK, 16 * ((i - N1) / ND), (i - N1) % ND);
  };
  auto element = [&](auto ic) {   // key 8 (r / 4) + 4 hf + r % 4 of the 32, the lane's query: masked iff beyond lim = q - first key - 4 hf
    constexpr int r = decltype(ic)::value;
    s[r] = fexp2(__builtin_fmaf(s[r], sc2, -st.lse2));
    if (MASK && 8 * (r >> 2) + (r & 3) > lim) s[r] = 0.f;
    s[r] *= dp[r];
    if constexpr ((r & 7) == 7) dsf[r >> 3] = pack8(s, r >> 3);
  };
  unrolled<0, AHEAD>(fetch);
  unrolled<0, NS>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    AH_SCHED_FENCE();
    fetch(std::integral_constant<int, i + AHEAD>{});
    if constexpr (i >= N1) st.acc[(i - N1) % ND] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], dsf[(i - N1) / ND], st.acc[(i - N1) % ND], 0, 0, 0);
    else if constexpr (i & 1) ndp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], st.dof[i >> 1], ndp, 0, 0, 0);
    else ns = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], st.qf[i >> 1], ns, 0, 0, 0);
    AH_SCHED_FENCE();
    if constexpr (i < SE) unrolled<i * 16 / SE, (i + 1) * 16 / SE>(element);
  });
  s = ns;
  dp = ndp;
}

// S and dP - delta of the first 32 keys of a pipeline
template <int D>
__device__ __forceinline__ void dq_scores(const char* cK, const char* cV, const DqState<D>& st, f32x16& s, f32x16& dp, const LaneOffs<D>& lo) {
#pragma unroll
  for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = -st.delta; }
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo.rows(cK, 0, ks), st.qf[ks], s, 0, 0, 0);
    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo.rows(cV, 0, ks), st.dof[ks], dp, 0, 0, 0);
  }
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_dq_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ o,
                                                      const bf16* __restrict__ d_o, const float* __restrict__ lse,
                                                      float* __restrict__ delta, bf16* __restrict__ dqkv, int B, int S, int nh,
                                                      float sc2, float scale) {
  constexpr int HALF = 32 * 2 * D;                                 // bytes of 32 rows
  __shared__ __attribute__((aligned(1024))) char ring[10 * HALF];  // six halves of K tiles, four of V tiles
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: LDS bases stay scalar
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int qb = CAUSAL ? causal_query_block(rank, S / 128) : rank;
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const int qw0 = qb * 128 + wave * 32, q = qw0 + (lane & 31);

  DqState<D> st;
  st.load(qp + (size_t)q * ld, o, d_o, lse, delta, (size_t)b * S + q, ((size_t)b * nh + head) * S + q, head, nh, hf, true);

  uint32_t off[D / 64];
#pragma unroll
  for (int i = 0; i < D / 64; i++) off[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);

  // Keys by 32 up to and including the diagonal (all of them without the mask), two steps per round.  Keys 32 h .. are in K
  // slot h % 6 and V slot h % 4: step h reads the columns of K half h and the rows of halves h + 1, so a round reads three halves
  // of K and two of V while the two after those arrive.  (Five K slots would do; either way two blocks share a CU.  Past the end the
  // last half is fetched again, into slots whose scores nobody uses.)
  const int nround = CAUSAL ? 2 * qb + 2 : S / 64, lasth = 2 * nround - 1;
  auto load = [&](int h) {
    const size_t row = (size_t)min(h, lasth) * 32 * ld;
    issue_half<D>(kp + row, off, ring + (h % 6) * HALF, wave);
    issue_half<D>(vp + row, off, ring + (6 + (h & 3)) * HALF, wave);
  };
  // (opaque to the compiler, which otherwise keeps every lane's address of every slot)
  auto slot_k = [&](int h) { int x = (h % 6) * HALF; asm("" : "+s"(x)); return (const char*)ring + x; };
  auto slot_v = [&](int h) { int x = (6 + (h & 3)) * HALF; asm("" : "+s"(x)); return (const char*)ring + x; };
  load(0);
  load(1);
  load(2);
  const LaneOffs<D> lo(lane);
  f32x16 s, dp;
  AH_NEXT_TILE();
  dq_scores<D>(slot_k(0), slot_v(0), st, s, dp, lo);
  AH_NEXT_TILE();   // every wave has read V half 0, whose slot the first round fills
  const int lim = q - 4 * hf;
#define AH_DQ_ROUND(MASK)                                                                                               \
  load(h + 3);                                                                                                          \
  load(h + 4);                                                                                                          \
  if (!MASK || h <= own) dq_step<D, MASK>(slot_k(h), slot_k(h + 1), slot_v(h + 1), st, s, dp, lo, lim - 32 * h, sc2);   \
  if (!MASK || h < own)                                                                                                 \
    dq_step<D, MASK>(slot_k(h + 1), slot_k(h + 2), slot_v(h + 2), st, s, dp, lo, lim - 32 * h - 32, sc2);               \
  AH_NEXT_TILE()
  const int own = 4 * qb + wave;   // the half with the wave's own positions; those after it are skipped (see the dK/dV kernel)
  int h = 0;
#pragma unroll 1
  for (; h < (CAUSAL ? 4 * qb : lasth); h += 2) { AH_DQ_ROUND(false); }
  if (CAUSAL) {  // the keys of the block's own queries
#pragma unroll 1
    for (; h < lasth; h += 2) { AH_DQ_ROUND(true); }
  }
#undef AH_DQ_ROUND

  store_rows<D>([&](int dt, int r) { return st.acc[dt][r] * scale; }, ring + wave * strip_bytes<D>(), dqkv + ((size_t)b * S + qw0) * ld + head * D, ld, lane);
}

// ---- head_dim 64: one tile of 64 keys after the other, LDS reads a phase ahead of their use.  Three waves fit a SIMD this way (168
// registers; the steps above take 181) and do better than two that overlap their own phases: 8 x 16 x 512 20.3 against
// 21.6 us, 2 x 16 x 2048 causal 35.2 / 38.1, 1 x 32 x 4096 causal 5 % more for the whole backward.
template <int D, bool DIAG>
__device__ __forceinline__ void dq_tile(const char* __restrict__ cK, const char* __restrict__ cV, DqState<D>& st, int k0, int q,
                                        float sc2, int lane) {
  constexpr int NK = D / 16, ND = D / 32;
  const int hf = lane >> 5;
  const int lim = q - k0 - 4 * hf;  // element r of half t is masked iff t*32 + 8*(r/4) + r%4 > lim
  bf16x8 fk[NK], fv[NK];
#pragma unroll
  for (int ks = 0; ks < NK; ks++) {
    fk[ks] = frag_rowmajor<D>(cK, lane & 31, ks, hf);
    fv[ks] = frag_rowmajor<D>(cV, lane & 31, ks, hf);
  }
#pragma unroll
  for (int t = 0; t < 2; t++) {
    AH_SCHED_FENCE();
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = -st.delta; }   // the product dO V^T lands on -delta: dP - delta for free
    bf16x8 kt[2][ND];
#pragma unroll
    for (int ks = 0; ks < NK; ks++) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[ks], st.qf[ks], s, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv[ks], st.dof[ks], dp, 0, 0, 0);
    }
#pragma unroll
    for (int s2 = 0; s2 < 2; s2++)
#pragma unroll
      for (int dt = 0; dt < ND; dt++) kt[s2][dt] = frag_transposed<D>(cK, t * 32 + 16 * s2 + 4 * hf, dt, lane);
    AH_SCHED_FENCE();
    const float nl = -st.lse2;
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] = fexp2(__builtin_fmaf(s[r], sc2, nl));
    if (DIAG) {
#pragma unroll
      for (int r = 0; r < 16; r++)
        if (t * 32 + 8 * (r >> 2) + (r & 3) > lim) s[r] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < 16; r++) s[r] *= dp[r];  // dS^T
    if (t == 0) {
#pragma unroll
      for (int ks = 0; ks < NK; ks++) {
        fk[ks] = frag_rowmajor<D>(cK, 32 + (lane & 31), ks, hf);
        fv[ks] = frag_rowmajor<D>(cV, 32 + (lane & 31), ks, hf);
      }
    }
    AH_SCHED_FENCE();
#pragma unroll
    for (int s2 = 0; s2 < 2; s2++) {
      const bf16x8 dsf = pack8(s, s2);
#pragma unroll
      for (int dt = 0; dt < ND; dt++) st.acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[s2][dt], dsf, st.acc[dt], 0, 0, 0);
    }
  }
  AH_SCHED_FENCE();
}

// MASK: the tile straddles the diagonal for some of the waves and lies behind it for others, which skip it
template <int D, bool MASK>
__device__ __forceinline__ void dq_tile_step(const bf16* gK, const bf16* gV, uint32_t* off, char* __restrict__ nK,
                                        char* __restrict__ nV, const char* __restrict__ cK, const char* __restrict__ cV,
                                        DqState<D>& st, int k0, int q, int qw0, float sc2, int wave, int lane) {
  issue_tile<D>(gK, off, nK, wave);
  issue_tile<D>(gV, off, nV, wave);
  if (MASK && k0 > qw0 + 31) return;
  dq_tile<D, MASK>(cK, cV, st, k0, q, sc2, lane);
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_dq_plain_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ o,
                                                      const bf16* __restrict__ d_o, const float* __restrict__ lse,
                                                      float* __restrict__ delta, bf16* __restrict__ dqkv, int B, int S, int nh,
                                                      float sc2, float scale) {
  constexpr int TILEB = 64 * 2 * D, STAGE = 2 * TILEB;  // ring slot = K tile then V tile
  __shared__ __attribute__((aligned(1024))) char ring[NSLOT * STAGE];
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: LDS bases stay scalar
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int qb = CAUSAL ? causal_query_block(rank, S / 128) : rank;
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const int qw0 = qb * 128 + wave * 32, q = qw0 + (lane & 31);

  DqState<D> st;
  st.load(qp + (size_t)q * ld, o, d_o, lse, delta, (size_t)b * S + q, ((size_t)b * nh + head) * S + q, head, nh, hf, true);

  uint32_t off[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) off[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);

  // Tile t lives in ring slot t % 2 and is loaded during step t - 1, two steps per round (the number of tiles is even); under the mask
  // the two tiles with the block's own positions are peeled, so that the others have no mask in them
  const int ntile = CAUSAL ? 2 * qb + 2 : S / 64, last = ntile - 1, nfull = CAUSAL ? ntile - 2 : ntile;
  const size_t step = (size_t)64 * ld;
  char *const K0 = ring, *const V0 = ring + TILEB, *const K1 = ring + STAGE, *const V1 = ring + STAGE + TILEB;
  issue_tile<D>(kp, off, K0, wave);
  issue_tile<D>(vp, off, V0, wave);
  AH_NEXT_TILE();
  for (int j = 0; j < nfull; j += 2) {
    const size_t o1 = (size_t)(j + 1) * step, o2 = (size_t)min(j + 2, last) * step;
    dq_tile_step<D, false>(kp + o1, vp + o1, off, K1, V1, K0, V0, st, j * 64, q, qw0, sc2, wave, lane);
    AH_NEXT_TILE();
    dq_tile_step<D, false>(kp + o2, vp + o2, off, K0, V0, K1, V1, st, (j + 1) * 64, q, qw0, sc2, wave, lane);
    AH_NEXT_TILE();
  }
  if (CAUSAL) {
    const size_t o1 = (size_t)last * step;
    int late = lane;  // opaque, so that the addresses of these two tiles are not computed and kept (spilled) before the loop
    asm volatile("" : "+v"(late));
    dq_tile_step<D, true>(kp + o1, vp + o1, off, K1, V1, K0, V0, st, (last - 1) * 64, q, qw0, sc2, wave, late);
    AH_NEXT_TILE();
    if (last * 64 <= qw0 + 31) dq_tile<D, true>(K1, V1, st, last * 64, q, sc2, late);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));  // drain the redundant tail loads

  // (the other waves may still read the second ring slot; the strips lie in the first)
  store_rows<D>([&](int dt, int r) { return st.acc[dt][r] * scale; }, ring + wave * strip_bytes<D>(), dqkv + ((size_t)b * S + qw0) * ld + head * D, ld, lane);
}

// =========================================================================== backward: dQ for launches that cannot fill the chip
// The split of attn_fwd64_kernel applied to dQ: 64 queries per block, wave w owns queries 32 * (w & 1) .. + 31 and
// keys 32 * (w >> 1) .. + 31 of every 64-key tile; the two partial dQ per query are added in LDS at the end.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_dq64_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ o,
                                                        const bf16* __restrict__ d_o, const float* __restrict__ lse,
                                                        float* __restrict__ delta, bf16* __restrict__ dqkv, int B, int S, int nh,
                                                        float sc2, float scale) {
  constexpr int TILEB = 64 * 2 * D, ND = D / 32;
  __shared__ __attribute__((aligned(1024))) char ring[5 * TILEB];   // three K tiles, two V tiles
  static_assert(2 * ND * 16 * 64 * 4 + 2 * strip_bytes<D>() <= 5 * TILEB, "the partial results and output strips of two waves fit in the ring");
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qt = wave & 1, kh = wave >> 1;
  const int nq = S / 64;
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int qb = CAUSAL ? causal_query_block(rank, nq) : rank;
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const int qw0 = qb * 64 + qt * 32, q = qw0 + (lane & 31);

  DqState<D> st;   // (both key halves' waves take delta, one writes it)
  st.load(qp + (size_t)q * ld, o, d_o, lse, delta, (size_t)b * S + q, ((size_t)b * nh + head) * S + q, head, nh, hf, kh == 0);

  uint32_t off[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) off[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);

  // One step of the pipeline per key tile (the wave's half of it).  K tile t lives in K slot t % 3 and V tile t in V slot t % 2: step j
  // reads the columns of K tile j and the rows of tiles j + 1, while tiles j + 2 arrive (past the end the last one again)
  const int ntile = CAUSAL ? qb + 1 : nq, last = ntile - 1, k0 = 32 * kh;
  auto load = [&](int t) {
    const size_t row = (size_t)min(t, last) * 64 * ld;
    issue_tile<D>(kp + row, off, ring + (t % 3) * TILEB, wave);
    issue_tile<D>(vp + row, off, ring + (3 + (t & 1)) * TILEB, wave);
  };
  auto slot_k = [&](int t) { int x = (t % 3) * TILEB; asm("" : "+s"(x)); return (const char*)ring + x + k0 * (2 * D); };
  auto slot_v = [&](int t) { int x = (3 + (t & 1)) * TILEB; asm("" : "+s"(x)); return (const char*)ring + x + k0 * (2 * D); };
  load(0);
  load(1);
  const LaneOffs<D> lo(lane);
  f32x16 s, dp;
  AH_NEXT_TILE();
  dq_scores<D>(slot_k(0), slot_v(0), st, s, dp, lo);
  AH_NEXT_TILE();   // the first V tile's slot is loaded next
#pragma unroll 1
  for (int j = 0; j < last; j++) {
    load(j + 2);
    dq_step<D, false>(slot_k(j), slot_k(j + 1), slot_v(j + 1), st, s, dp, lo, 0, sc2);
    AH_NEXT_TILE();
  }
  // the last tile, under the mask that of the block's own queries (a wave whose keys all lie after its queries skips it: see
  // the 128-row dK/dV kernel; the next scores are nobody's)
  if (!CAUSAL || qt >= kh) dq_step<D, CAUSAL>(slot_k(last), slot_k(last), slot_v(last), st, s, dp, lo, q - 64 * last - k0 - 4 * hf, sc2);
  __syncthreads();

  float* mg = (float*)ring + (size_t)qt * ND * 16 * 64;
  if (kh == 1) {
#pragma unroll
    for (int dt = 0; dt < ND; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) mg[(dt * 16 + r) * 64 + lane] = st.acc[dt][r];
  }
  __syncthreads();
  if (kh == 1) return;
  store_rows<D>([&](int dt, int r) { return (st.acc[dt][r] + mg[(dt * 16 + r) * 64 + lane]) * scale; }, ring + 5 * TILEB - (2 - qt) * strip_bytes<D>(),
                dqkv + ((size_t)b * S + qw0) * ld + head * D, ld, lane);
}

// ---- head_dim 64: one tile after the other, as in the 128-row kernel of this width (168 registers, the steps take 184).  The whole backward,
// in steps / this way: 1 x 16 x 1024 causal 26.9 / 26.2 us, without the mask 27.1 / 26.4, 1 x 8 x 4096 causal 91.4 / 89.1, 4 x
// 16 x 512 28.6 / 28.1, 1 x 16 x 256 causal 13.1 / 12.9 (same bits).
__device__ __forceinline__ void dq_half_tile(const char* __restrict__ cK, const char* __restrict__ cV, DqState<64>& st, int kh, int lim,
                                             bool diag, float sc2, int lane) {
  constexpr int D = 64, NK = D / 16, ND = D / 32;
  const int hf = lane >> 5;
  bf16x8 fk[NK], fv[NK];
#pragma unroll
  for (int ks = 0; ks < NK; ks++) {
    fk[ks] = frag_rowmajor<D>(cK, 32 * kh + (lane & 31), ks, hf);
    fv[ks] = frag_rowmajor<D>(cV, 32 * kh + (lane & 31), ks, hf);
  }
  AH_SCHED_FENCE();
  f32x16 s, dp;
#pragma unroll
  for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = -st.delta; }   // dP - delta for free
#pragma unroll
  for (int ks = 0; ks < NK; ks++) {
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[ks], st.qf[ks], s, 0, 0, 0);
    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv[ks], st.dof[ks], dp, 0, 0, 0);
  }
  bf16x8 kt[2][ND];
#pragma unroll
  for (int s2 = 0; s2 < 2; s2++)
#pragma unroll
    for (int dt = 0; dt < ND; dt++) kt[s2][dt] = frag_transposed<D>(cK, 32 * kh + 16 * s2 + 4 * hf, dt, lane);
  AH_SCHED_FENCE();
  const float nl = -st.lse2;
#pragma unroll
  for (int r = 0; r < 16; r++) s[r] = fexp2(__builtin_fmaf(s[r], sc2, nl));
  if (diag) {  // wave-uniform; element r is masked iff 8 * (r / 4) + r % 4 > lim
#pragma unroll
    for (int r = 0; r < 16; r++)
      if (8 * (r >> 2) + (r & 3) > lim) s[r] = 0.f;
  }
#pragma unroll
  for (int r = 0; r < 16; r++) s[r] *= dp[r];  // dS^T
  AH_SCHED_FENCE();
#pragma unroll
  for (int s2 = 0; s2 < 2; s2++) {
    const bf16x8 dsf = pack8(s, s2);
#pragma unroll
    for (int dt = 0; dt < ND; dt++) st.acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[s2][dt], dsf, st.acc[dt], 0, 0, 0);
  }
  AH_SCHED_FENCE();
}

template <bool CAUSAL>
__global__ __launch_bounds__(256, 2) void attn_dq64_plain_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ o,
                                                        const bf16* __restrict__ d_o, const float* __restrict__ lse,
                                                        float* __restrict__ delta, bf16* __restrict__ dqkv, int B, int S, int nh,
                                                        float sc2, float scale) {
  constexpr int D = 64, TILEB = 64 * 2 * D, STAGE = 2 * TILEB, ND = D / 32;
  __shared__ __attribute__((aligned(1024))) char ring[NSLOT * STAGE];   // ring slot = K tile then V tile
  static_assert(2 * ND * 16 * 64 * 4 + 2 * strip_bytes<D>() <= NSLOT * STAGE, "the partial results and output strips of two waves fit in the ring");
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qt = wave & 1, kh = wave >> 1;
  const int nq = S / 64;
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int qb = CAUSAL ? causal_query_block(rank, nq) : rank;
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const int qw0 = qb * 64 + qt * 32, q = qw0 + (lane & 31);

  DqState<D> st;   // (both key halves' waves take delta, one writes it)
  st.load(qp + (size_t)q * ld, o, d_o, lse, delta, (size_t)b * S + q, ((size_t)b * nh + head) * S + q, head, nh, hf, kh == 0);

  uint32_t off[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++) off[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);

  // tile t lives in ring slot t % 2 and is loaded during tile t - 1 (the last one again during the last, into a dead slot)
  const int ntile = CAUSAL ? qb + 1 : nq, last = ntile - 1;
  const size_t step = (size_t)64 * ld;
  issue_tile<D>(kp, off, ring, wave);
  issue_tile<D>(vp, off, ring + TILEB, wave);
  AH_NEXT_TILE();
  for (int j = 0; j < ntile; j++) {
    const size_t o2 = (size_t)min(j + 1, last) * step;
    char* fill = ring + ((j + 1) & 1) * STAGE;
    const char* cur = ring + (j & 1) * STAGE;
    issue_tile<D>(kp + o2, off, fill, wave);
    issue_tile<D>(vp + o2, off, fill + TILEB, wave);
    // in the block's own tile the wave's keys lie before (kh < qt), on (kh == qt) or after (kh > qt: skipped) its queries
    const bool own = CAUSAL && j == last;
    if (!(own && kh > qt)) dq_half_tile(cur, cur + TILEB, st, kh, q - j * 64 - 32 * kh - 4 * hf, own && kh == qt, sc2, lane);
    AH_NEXT_TILE();
  }

  float* mg = (float*)ring + (size_t)qt * ND * 16 * 64;
  if (kh == 1) {
#pragma unroll
    for (int dt = 0; dt < ND; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) mg[(dt * 16 + r) * 64 + lane] = st.acc[dt][r];
  }
  __syncthreads();
  if (kh == 1) return;
  store_rows<D>([&](int dt, int r) { return (st.acc[dt][r] + mg[(dt * 16 + r) * 64 + lane]) * scale; }, ring + NSLOT * STAGE - (2 - qt) * strip_bytes<D>(),
                dqkv + ((size_t)b * S + qw0) * ld + head * D, ld, lane);
}

// =========================================================================== backward: dK, dV (one block per 128 keys)
template <int D>
struct DkvState {
  bf16x8 kf[D / 16], vf[D / 16];
  f32x16 dk[D / 32], dv[D / 32];
};

// One step of the pipeline over 32 queries: the probabilities and dS of the 32 queries whose scores S and dP - delta are in s, dp (rows
// t .. t + 31 of the tile at cur), their products with dO and Q, and S and dP - delta of the next 32 (rows tn .. of the tile at nxt).
// A fixed sequence of slots as in the forward kernel: under each matrix instruction of the next scores one probability and
// one element of dS, and a fragment requested AHEAD slots before its use.  With head_dim 128 a wave has its SIMD to itself
// (K, V and the accumulators of dK and dV are 192 registers), so what it does not overlap, nobody does.  One phase after
// the other a tile of 64 queries took 2.9 us, now 2.2; 64 matrix instructions alone take 1.15, with their LDS reads, the
// loads and one barrier 1.7 .. 1.9.  dK/dV at 2 x 16 x 2048 x 128 causal 108.5 -> 103.7 us, without the mask 156.3 -> 147.2, 1 x 32 x
// 4096 x 128 causal 339 -> 331 (same bits).
template <int D, bool MASK>
__device__ __forceinline__ void dkv_step(const char* cur, int t, const char* nxt, int tn, DkvState<D>& st, f32x16& s, f32x16& dp,
                                         const LaneOffs<D>& lo, int lim, float sc2, int hf) {
  constexpr int NK = D / 16, ND = D / 32, TILEB = 64 * 2 * D;
  constexpr int N1 = 2 * NK, NS = N1 + 4 * ND;   // slots: S and dP by turns, then dV and dK by turns
  constexpr int SE = NS - 2 * ND - 2;            // slots over which the 16 probabilities are spread
  static_assert(15 * SE / 16 < NS - 2 * ND && 7 * SE / 16 < N1, "probabilities precede their products");
  constexpr int AHEAD = 5;
  const float* stat = (const float*)(cur + 2 * TILEB) + t + 4 * hf;        // log-sum-exps; 64 further on the -deltas
  const float* nstat = (const float*)(nxt + 2 * TILEB) + 64 + tn + 4 * hf;
  f32x16 ns, ndp;
  f32x4 l4[4];
#pragma unroll
  for (int g = 0; g < 4; g++) {
    const f32x4 d4 = *(const f32x4*)(nstat + 8 * g);   // the product dO V^T lands on -delta: dP - delta without a subtraction
#pragma unroll
    for (int i = 0; i < 4; i++) { ns[4 * g + i] = 0.f; ndp[4 * g + i] = d4[i]; }
    l4[g] = *(const f32x4*)(stat + 8 * g);
  }
  bf16x8 fr[NS], pf[2], dsf[2];
  const char *const nQ = nxt + tn * (2 * D), *const nO = nQ + TILEB, *const cQ = cur + t * (2 * D), *const cO = cQ + TILEB;
  auto fetch = [&](auto ic) {
    constexpr int i = decltype(ic)::value;
    if constexpr (i < N1) fr[i] = lo.rows(i & 1 ? nO : nQ, 0, i >> 1);
    else if constexpr (i < NS) fr[i] = lo.cols((i - N1) & 1 ? cQ : cO, 16 * ((i - N1) / (2 * ND)), ((i - N1) >> 1) % ND);
  };
  auto element = [&](auto ic) {   // the lane's query t + 8 (r / 4) + 4 hf + r % 4 of the tile, its own key
    constexpr int r = decltype(ic)::value;
    s[r] = fexp2(__builtin_fmaf(s[r], sc2, -l4[r >> 2][r & 3] * LOG2E));
    if (MASK && 8 * (r >> 2) + (r & 3) < lim) s[r] = 0.f;
    dp[r] *= s[r];
    if constexpr ((r & 7) == 7) { pf[r >> 3] = pack8(s, r >> 3); dsf[r >> 3] = pack8(dp, r >> 3); }
  };
  unrolled<0, AHEAD>(fetch);
  unrolled<0, NS>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    AH_SCHED_FENCE();
    fetch(std::integral_constant<int, i + AHEAD>{});
    if constexpr (i < N1) {
      if constexpr (i & 1) ndp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], st.vf[i >> 1], ndp, 0, 0, 0);
      else ns = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], st.kf[i >> 1], ns, 0, 0, 0);
    } else {
      constexpr int s2 = (i - N1) / (2 * ND), dt = ((i - N1) >> 1) % ND;
      if constexpr ((i - N1) & 1) st.dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], dsf[s2], st.dk[dt], 0, 0, 0);
      else st.dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i], pf[s2], st.dv[dt], 0, 0, 0);
    }
    AH_SCHED_FENCE();
    if constexpr (i < SE) unrolled<i * 16 / SE, (i + 1) * 16 / SE>(element);
  });
  s = ns;
  dp = ndp;
}

// S and dP - delta of the first 32 queries of a pipeline: rows t .. of the tile at cur
template <int D>
__device__ __forceinline__ void dkv_scores(const char* cur, int t, const DkvState<D>& st, f32x16& s, f32x16& dp, const LaneOffs<D>& lo, int hf) {
  constexpr int TILEB = 64 * 2 * D;
  const float* nstat = (const float*)(cur + 2 * TILEB) + 64 + t + 4 * hf;
#pragma unroll
  for (int r = 0; r < 16; r++) { s[r] = 0.f; dp[r] = nstat[8 * (r >> 2) + (r & 3)]; }
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo.rows(cur + t * (2 * D), 0, ks), st.kf[ks], s, 0, 0, 0);
    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo.rows(cur + TILEB + t * (2 * D), 0, ks), st.vf[ks], dp, 0, 0, 0);
  }
}

// ring slot of the dK/dV kernel: Q tile, dO tile, then 64 log-sum-exps, 64 deltas and 512 spare bytes
template <int D>
__device__ __forceinline__ void dkv_issue(const bf16* gQ, const bf16* gO, const float* gL, const float* gD, uint32_t* offq,
                                          uint32_t* offo, uint32_t& offs, char* __restrict__ slot, int wave) {
  constexpr int TILEB = 64 * 2 * D;
  issue_tile<D>(gQ, offq, slot, wave);
  issue_tile<D>(gO, offo, slot + TILEB, wave);
  // one 4-byte load per lane: waves 0 and 1 bring the statistics, waves 2 and 3 repeat them into the
  // spare bytes so that every wave has the same number of loads in flight
  load4((wave & 1) ? gD : gL, offs, slot + 2 * TILEB + wave * 256);
}

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_dkv_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ d_o,
                                                       const float* __restrict__ lse, const float* __restrict__ delta,
                                                       bf16* __restrict__ dqkv, int B, int S, int nh, float sc2, float scale) {
  constexpr int TILEB = 64 * 2 * D, STAGE = 2 * TILEB + 1024;
  __shared__ __attribute__((aligned(1024))) char ring[3 * STAGE];
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: LDS bases stay scalar
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int kb = rank;  // key block 0 sees every query tile: heaviest first
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D, ldo = nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const bf16* dop = d_o + (size_t)b * S * ldo + head * D;
  const int kw0 = kb * 128 + wave * 32, key = kw0 + (lane & 31);
  const float* lse_row = lse + ((size_t)b * nh + head) * S;
  const float* delta_row = delta + ((size_t)b * nh + head) * S;

  DkvState<D> st;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    st.kf[ks] = *(const bf16x8*)(kp + (size_t)key * ld + ks * 16 + hf * 8);
    st.vf[ks] = *(const bf16x8*)(vp + (size_t)key * ld + ks * 16 + hf * 8);
  }
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) { st.dk[dt][r] = 0.f; st.dv[dt][r] = 0.f; }

  uint32_t offq[D / 32], offo[D / 32], offs = lane * 4;  // byte offsets of the lane's loads (offs: the 4-byte statistics)
#pragma unroll
  for (int i = 0; i < D / 32; i++) {
    offq[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);
    offo[i] = tile_src_offset<D>(wave + 4 * i, lane, ldo);
  }

  // Query tiles of 64 from the diagonal on (from 0 without the mask), two steps each.  Tile t lives in ring slot t % 3: the second
  // step of a tile reads the next one's first rows, while the one after that arrives.  (Past the end the last tile is
  // fetched again, into a slot whose scores nobody uses.)
  const int j0 = CAUSAL ? 2 * kb : 0, ntile = S / 64 - j0, last = ntile - 1;
  qp += (size_t)j0 * 64 * ld;
  dop += (size_t)j0 * 64 * ldo;
  lse_row += j0 * 64;
  delta_row += j0 * 64;
  auto load = [&](int t, char* slot) {
    t = min(t, last);
    dkv_issue<D>(qp + (size_t)t * 64 * ld, dop + (size_t)t * 64 * ldo, lse_row + t * 64, delta_row + t * 64, offq, offo, offs, slot, wave);
  };
  const LaneOffs<D> lo(lane);
  char *cur = ring, *nxt = ring + STAGE, *fill = ring + 2 * STAGE;
  load(0, cur);
  load(1, nxt);
  f32x16 s, dp;
  AH_NEXT_TILE();
  const int lim = key - j0 * 64 - 4 * hf;   // under the mask the lane's key sees no query before lim
#define AH_DKV_STEPS(MASK)                                                            \
  dkv_step<D, MASK>(cur, 0, cur, 32, st, s, dp, lo, lim - j * 64, sc2, hf);           \
  dkv_step<D, MASK>(cur, 32, nxt, 0, st, s, dp, lo, lim - j * 64 - 32, sc2, hf)
#define AH_DKV_NEXT()                                                                 \
  AH_NEXT_TILE();                                                                     \
  { char* const c = cur; cur = nxt; nxt = fill; fill = c; }                           \
  j++
#define AH_DKV_TILE(MASK)                                                             \
  load(j + 2, fill);                                                                  \
  AH_DKV_STEPS(MASK);                                                                 \
  AH_DKV_NEXT()
  int j = 0;
  if (CAUSAL) {
    // The block's own positions.  The first of their two tiles holds only queries before the keys of the last two waves, which
    // skip it: a probability of zero times what is not finite would reach their results.  (By steps of 32 queries, the
    // accumulators move out of the ordinary registers: 67.9 -> 70.6 us for the whole backward at 16 x 20 x 256 x 128.)
    load(2, fill);
    dkv_scores<D>(wave < 2 ? cur : nxt, 0, st, s, dp, lo, hf);
    if (wave < 2) { AH_DKV_STEPS(true); }
    AH_DKV_NEXT();
    AH_DKV_TILE(true);
  } else {
    dkv_scores<D>(cur, 0, st, s, dp, lo, hf);
  }
#pragma unroll 1
  while (j < ntile) { AH_DKV_TILE(false); }
#undef AH_DKV_TILE
#undef AH_DKV_NEXT
#undef AH_DKV_STEPS

  char* strip = ring + wave * strip_bytes<D>();
  bf16* out = dqkv + ((size_t)b * S + kw0) * ld + nh * D + head * D;
  store_rows<D>([&](int dt, int r) { return st.dk[dt][r] * scale; }, strip, out, ld, lane);
  store_rows<D>([&](int dt, int r) { return st.dv[dt][r]; }, strip, out + nh * D, ld, lane);
}

// =========================================================================== backward: dK, dV for launches that cannot fill the chip
// 64 keys per block instead of 128 (twice the blocks, dispatched heaviest first, so that the CUs even out): wave w
// owns keys 32 * (w & 1) .. + 31 of the block and, of every 64-query tile, the queries 32 * (w >> 1) .. + 31; the two
// partial dK, dV per key are added in LDS at the end.
template <int D, bool CAUSAL>
__global__ __launch_bounds__(256) void attn_dkv64_kernel(const bf16* __restrict__ qkv, const bf16* __restrict__ d_o,
                                                         const float* __restrict__ lse, const float* __restrict__ delta,
                                                         bf16* __restrict__ dqkv, int B, int S, int nh, float sc2, float scale) {
  constexpr int TILEB = 64 * 2 * D, STAGE = 2 * TILEB + 1024, LPS = 2 * (D / 32) + 1, ND = D / 32;
  __shared__ __attribute__((aligned(1024))) char ring[4 * STAGE];
  static_assert(2 * 2 * ND * 16 * 64 * 4 + 2 * strip_bytes<D>() <= 4 * STAGE, "the partial results and output strips of two waves fit in the ring");
  const int lane = threadIdx.x & 63, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kt = wave & 1, qh = wave >> 1;
  const int nkb = S / 64;
  const int nbh = B * nh;
  const int rank = blockIdx.x / nbh, bh = blockIdx.x - rank * nbh;   // all heads of one block of rows, then the next
  const int kb = rank;  // key block 0 sees every query tile: heaviest first
  const int b = bh / nh, head = bh - b * nh;
  const int ld = 3 * nh * D, ldo = nh * D;
  const bf16* qp = qkv + (size_t)b * S * ld + head * D;
  const bf16* kp = qp + nh * D;
  const bf16* vp = qp + 2 * nh * D;
  const bf16* dop = d_o + (size_t)b * S * ldo + head * D;
  const int kw0 = kb * 64 + kt * 32, key = kw0 + (lane & 31);
  const float* lse_row = lse + ((size_t)b * nh + head) * S;
  const float* delta_row = delta + ((size_t)b * nh + head) * S;

  DkvState<D> st;
#pragma unroll
  for (int ks = 0; ks < D / 16; ks++) {
    st.kf[ks] = *(const bf16x8*)(kp + (size_t)key * ld + ks * 16 + hf * 8);
    st.vf[ks] = *(const bf16x8*)(vp + (size_t)key * ld + ks * 16 + hf * 8);
  }
#pragma unroll
  for (int dt = 0; dt < ND; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) { st.dk[dt][r] = 0.f; st.dv[dt][r] = 0.f; }

  uint32_t offq[D / 32], offo[D / 32], offs = lane * 4;  // byte offsets of the lane's loads (offs: the 4-byte statistics)
#pragma unroll
  for (int i = 0; i < D / 32; i++) {
    offq[i] = tile_src_offset<D>(wave + 4 * i, lane, ld);
    offo[i] = tile_src_offset<D>(wave + 4 * i, lane, ldo);
  }

  // Query tiles of 64 from the one that holds the block's own positions on (from 0 without the mask), one step of the pipeline
  // each (the wave's half of it).  Tile t lives in ring slot t % 4; loads run three tiles ahead and are waited for by count, past
  // the end the last tile is fetched again (a uniform number of loads in flight)
  const int j0 = CAUSAL ? kb : 0, ntile = S / 64 - j0, last = ntile - 1;
  qp += (size_t)j0 * 64 * ld;
  dop += (size_t)j0 * 64 * ldo;
  lse_row += j0 * 64;
  delta_row += j0 * 64;
  auto load = [&](int t) {
    char* slot = ring + (t & 3) * STAGE;
    t = min(t, last);
    dkv_issue<D>(qp + (size_t)t * 64 * ld, dop + (size_t)t * 64 * ldo, lse_row + t * 64, delta_row + t * 64, offq, offo, offs, slot, wave);
  };
  load(0);
  load(1);
  load(2);
  const LaneOffs<D> lo(lane);
  f32x16 s, dp;
  const int t0 = 32 * qh;
  AH_LANDED(LPS);   // tiles 0 and 1
  const bool skip = CAUSAL && qh < kt;   // the wave's queries of the block's own tile all lie before its keys (see the 128-row kernel)
  dkv_scores<D>(skip ? ring + STAGE : ring, t0, st, s, dp, lo, hf);
  auto slot = [&](int t) { int x = (t & 3) * STAGE; asm("" : "+s"(x)); return (const char*)ring + x; };
  const int lim = key - j0 * 64 - t0 - 4 * hf;
  load(3);
  if (!skip) dkv_step<D, CAUSAL>(slot(0), t0, slot(1), t0, st, s, dp, lo, lim, sc2, hf);
  AH_LANDED(LPS);
#pragma unroll 1
  for (int j = 1; j < ntile; j++) {
    load(j + 3);
    dkv_step<D, false>(slot(j), t0, slot(j + 1), t0, st, s, dp, lo, 0, sc2, hf);
    AH_LANDED(LPS);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(0));  // drain the redundant tail loads
  __syncthreads();

  float* mg = (float*)ring + (size_t)kt * 2 * ND * 16 * 64;
  if (qh == 1) {
#pragma unroll
    for (int dt = 0; dt < ND; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        mg[(dt * 16 + r) * 64 + lane] = st.dk[dt][r];
        mg[((ND + dt) * 16 + r) * 64 + lane] = st.dv[dt][r];
      }
  }
  __syncthreads();
  if (qh == 1) return;
  char* strip = ring + 4 * STAGE - (2 - kt) * strip_bytes<D>();
  bf16* out = dqkv + ((size_t)b * S + kw0) * ld + nh * D + head * D;
  store_rows<D>([&](int dt, int r) { return (st.dk[dt][r] + mg[(dt * 16 + r) * 64 + lane]) * scale; }, strip, out, ld, lane);
  store_rows<D>([&](int dt, int r) { return st.dv[dt][r] + mg[((ND + dt) * 16 + r) * 64 + lane]; }, strip, out + nh * D, ld, lane);
}

}  // namespace

// Launches of at most this many 128-row blocks (one per CU) take the 64-row kernels, which split every block's work
// between wave pairs: twice the blocks, so that the CUs even out under the causal mask and a SIMD has two waves
// (gpt1p3b stage, 1 x 16 heads x 2048: forward 48 -> 36 us, backward 144 -> 114 us); larger launches fill the chip
// with 128-row blocks and are 8 % faster with them.
static int small_grid_blocks() {
  static const int v = getenv("AH_ATTN_SMALL_GRID") ? atoi(getenv("AH_ATTN_SMALL_GRID")) : 256;  // tuning aid
  return v;
}

static bool attn_shape_ok(int B, int S, int nh, int d) { return B > 0 && nh > 0 && S > 0 && S % 128 == 0 && (d == 64 || d == 128); }

template <int D, bool CAUSAL>
static void launch_fwd_t(dim3 grid, hipStream_t s, const void* qkv, void* o, float* lse, int B, int S, int nh, float sc2) {
  if ((int)grid.x <= small_grid_blocks())  // at most one 128-query block per CU: 64-query blocks with the keys split between wave pairs
    hipLaunchKernelGGL((attn_fwd64_kernel<D, CAUSAL>), dim3(2 * grid.x), dim3(256), 0, s, (const bf16*)qkv, (bf16*)o, lse, B, S, nh, sc2);
  else if constexpr (D == 64 && !CAUSAL)
    hipLaunchKernelGGL((attn_fwd_plain_kernel<D>), grid, dim3(256), 0, s, (const bf16*)qkv, (bf16*)o, lse, B, S, nh, sc2);
  else
    hipLaunchKernelGGL((attn_fwd_kernel<D, CAUSAL>), grid, dim3(256), 0, s, (const bf16*)qkv, (bf16*)o, lse, B, S, nh, sc2);
}

hipError_t launch_attention_fwd(const void* qkv, void* o, float* lse, int B, int S, int nh, int d, bool causal, hipStream_t s) {
  if (!attn_shape_ok(B, S, nh, d)) return hipErrorInvalidValue;
  const float sc2 = LOG2E / sqrtf((float)d);
  const dim3 grid(B * nh * (S / 128));
  if (d == 128) {
    if (causal) launch_fwd_t<128, true>(grid, s, qkv, o, lse, B, S, nh, sc2);
    else launch_fwd_t<128, false>(grid, s, qkv, o, lse, B, S, nh, sc2);
  } else {
    if (causal) launch_fwd_t<64, true>(grid, s, qkv, o, lse, B, S, nh, sc2);
    else launch_fwd_t<64, false>(grid, s, qkv, o, lse, B, S, nh, sc2);
  }
  return hipGetLastError();
}

// dQ first: it leaves the row sums delta = rowsum(dO * O) of its queries behind for the dK/dV kernel
template <int D, bool CAUSAL>
static void launch_bwd_t(dim3 grid, hipStream_t s, const void* qkv, const void* o, const float* lse, const void* d_o,
                         void* dqkv, float* delta, int B, int S, int nh, float sc2, float scale) {
  const bool small = (int)grid.x <= small_grid_blocks();  // at most one 128-row block per CU: 64-row blocks, each split between wave pairs
  if (small) grid.x *= 2;
  auto dq = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, (const bf16*)qkv, (const bf16*)o, (const bf16*)d_o, lse, delta, (bf16*)dqkv, B, S, nh, sc2, scale);
  };
  if constexpr (D == 64) {
    if (small) dq(attn_dq64_plain_kernel<CAUSAL>);
    else dq(attn_dq_plain_kernel<D, CAUSAL>);
  } else {
    if (small) dq(attn_dq64_kernel<D, CAUSAL>);
    else dq(attn_dq_kernel<D, CAUSAL>);
  }
  auto dkv = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, (const bf16*)qkv, (const bf16*)d_o, lse, delta, (bf16*)dqkv, B, S, nh, sc2, scale);
  };
  if (small) dkv(attn_dkv64_kernel<D, CAUSAL>);
  else dkv(attn_dkv_kernel<D, CAUSAL>);
}

hipError_t launch_attention_bwd(const void* qkv, const void* o, const float* lse, const void* d_o, void* dqkv, float* delta,
                                int B, int S, int nh, int d, bool causal, hipStream_t s) {
  if (!attn_shape_ok(B, S, nh, d)) return hipErrorInvalidValue;
  const float scale = 1.f / sqrtf((float)d), sc2 = LOG2E * scale;
  const dim3 grid(B * nh * (S / 128));
  if (d == 128) {
    if (causal) launch_bwd_t<128, true>(grid, s, qkv, o, lse, d_o, dqkv, delta, B, S, nh, sc2, scale);
    else launch_bwd_t<128, false>(grid, s, qkv, o, lse, d_o, dqkv, delta, B, S, nh, sc2, scale);
  } else {
    if (causal) launch_bwd_t<64, true>(grid, s, qkv, o, lse, d_o, dqkv, delta, B, S, nh, sc2, scale);
    else launch_bwd_t<64, false>(grid, s, qkv, o, lse, d_o, dqkv, delta, B, S, nh, sc2, scale);
  }
  return hipGetLastError();
}

}  // namespace ah
