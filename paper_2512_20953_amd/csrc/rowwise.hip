// Row-wise and element-wise kernels of the decoder layer: LayerNorm / RMSNorm
// forward and backward (fused with the residual add and the column sums that
// give the gains', offsets' and biases' gradients), column sums, rotary
// embedding.  All are bound by HBM bandwidth: every tensor is read and
// written once, 16 bytes per lane, statistics and sums in fp32.
#include "common.h"
#include "kernels.h"
#include <cstdlib>

namespace ah {

namespace {

constexpr int NT = 256;      // threads per block
// MAXC (template): 16-byte chunks per thread per row, ceil(hidden / 2048), at most 8 (hidden <= 16384)

__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();  // red may still be read from the previous call
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// Eight consecutive values of a tensor of the residual stream, which is bf16 or (residual_fp32) fp32.
template <bool F32> struct XVec;
template <> struct XVec<false> {
  bf16x8 v;
  __device__ __forceinline__ void load(const void* base, size_t elem) { v = *(const bf16x8*)((const bf16*)base + elem); }
  __device__ __forceinline__ float get(int j) const { return bf2f(v[j]); }
};
template <> struct XVec<true> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const void* base, size_t elem) {
    a = *(const f32x4*)((const float*)base + elem);
    b = *(const f32x4*)((const float*)base + elem + 4);
  }
  __device__ __forceinline__ float get(int j) const { return j < 4 ? a[j] : b[j - 4]; }
};

// The stage's input is kept for backward: its first norm, which reads it, leaves the copy, in bf16 or widened to the fp32 stream
// (4096 x 4096: 20.4 us, where a copy of 13.0 us preceded a norm of 14.8).  Instances of their own: with the choice made at
// run time a 4096-wide row takes eight more registers, and one wave fits a SIMD instead of two (bound to two, the instance
// that copies spills four).  With the same in the norm backward: 5-head stage 237.1 -> 234.9 us, smallest 321.6 -> 319.2, 1.3B
// 6052 -> 6024, 7B shard 17561 -> 17438, LLaMA-style 5962 -> 5943.
enum Keep { KEEP_NONE, KEEP_BF16, KEEP_F32 };
template <Keep KEEP, bool XF32>
__device__ __forceinline__ void keep_input(void* to, size_t elem, const XVec<XF32>& t) {
  static_assert(KEEP == KEEP_NONE || !XF32, "an fp32 input is there already");
  if constexpr (KEEP == KEEP_BF16) {
    *(bf16x8*)((bf16*)to + elem) = t.v;
  } else if constexpr (KEEP == KEEP_F32) {
    float* p = (float*)to + elem;
    *(f32x4*)p = f32x4{t.get(0), t.get(1), t.get(2), t.get(3)};
    *(f32x4*)(p + 4) = f32x4{t.get(4), t.get(5), t.get(6), t.get(7)};
  }
}

// ---------------------------------------------------------------- norm forward: one block per row
template <bool RMS, int MAXC, bool XF32, Keep KEEP>
__global__ __launch_bounds__(NT) void norm_fwd_kernel(const void* __restrict__ x, const bf16* __restrict__ gamma,
                                                      const bf16* __restrict__ beta, bf16* __restrict__ a,
                                                      float* __restrict__ stats, int h, float eps, void* __restrict__ keep) {
  __shared__ float red[8];
  const int row = blockIdx.x, nchunk = h >> 3;
  float v[MAXC][8];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = threadIdx.x + i * NT;
    if (c < nchunk) {
      XVec<XF32> t;
      t.load(x, (size_t)row * h + c * 8);
      keep_input<KEEP>(keep, (size_t)row * h + c * 8, t);
#pragma unroll
      for (int j = 0; j < 8; j++) { v[i][j] = t.get(j); s += RMS ? v[i][j] * v[i][j] : v[i][j]; }
    }
  }
  float mean = 0.f, rstd;
  if (RMS) {
    rstd = rsqrtf(block_sum(s, red) / h + eps);
  } else {
    mean = block_sum(s, red) / h;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < MAXC; i++)
      if (threadIdx.x + i * NT < nchunk)
#pragma unroll
        for (int j = 0; j < 8; j++) { float d = v[i][j] - mean; q += d * d; }
    rstd = rsqrtf(block_sum(q, red) / h + eps);
  }
  if (threadIdx.x == 0) { stats[2 * row] = mean; stats[2 * row + 1] = rstd; }
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = threadIdx.x + i * NT;
    if (c < nchunk) {
      bf16x8 g = *(const bf16x8*)(gamma + c * 8), o;
      bf16x8 b;
      if (!RMS) b = *(const bf16x8*)(beta + c * 8);
#pragma unroll
      for (int j = 0; j < 8; j++) {
        float r = (v[i][j] - mean) * rstd * bf2f(g[j]);
        if (!RMS) r += bf2f(b[j]);
        o[j] = f2bf(r);
      }
      *(bf16x8*)(a + (size_t)row * h + c * 8) = o;
    }
  }
}

// ---------------------------------------------------------------- norm forward, rows up to 8192 wide: one wave per row
// A wave keeps a whole row in registers (MAXI chunks of 8 values per lane), so both statistics are wave
// reductions with no block barrier, and it walks rows w, w + (waves in the grid), ... with the next row's loads
// issued before the current one is reduced: loads, arithmetic and stores of different rows overlap inside a wave
// as well as across the waves of a CU.  The gain and offset stay packed in registers for all rows.
template <bool RMS, int MAXI, bool XF32, Keep KEEP>
__global__ __launch_bounds__(NT, MAXI == 8 && KEEP == KEEP_BF16 ? 2 : 1) void norm_fwd_wave_kernel(const void* __restrict__ x, const bf16* __restrict__ gamma,
                                                           const bf16* __restrict__ beta, bf16* __restrict__ a,
                                                           float* __restrict__ stats, int T, int h, float eps, void* __restrict__ keep) {
  const int lane = threadIdx.x & 63, nchunk = h >> 3;
  const int nw = gridDim.x * (NT / 64);
  int row = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  if (row >= T) return;
  const float inv_h = 1.f / h;
  bf16x8 gam[MAXI], bet[RMS ? 1 : MAXI];
  XVec<XF32> cur[MAXI], nxt[MAXI];
#pragma unroll
  for (int i = 0; i < MAXI; i++) {
    const int c = lane + 64 * i;
    if (c < nchunk) {
      gam[i] = *(const bf16x8*)(gamma + c * 8);
      if (!RMS) bet[i] = *(const bf16x8*)(beta + c * 8);
      cur[i].load(x, (size_t)row * h + c * 8);
    }
  }
  for (; row < T; row += nw) {
    const int nr = row + nw;
    if (nr < T) {
#pragma unroll
      for (int i = 0; i < MAXI; i++)
        if (lane + 64 * i < nchunk) nxt[i].load(x, (size_t)nr * h + (lane + 64 * i) * 8);
    }
    if constexpr (KEEP != KEEP_NONE) {
#pragma unroll
      for (int i = 0; i < MAXI; i++)
        if (lane + 64 * i < nchunk) keep_input<KEEP>(keep, (size_t)row * h + (lane + 64 * i) * 8, cur[i]);
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MAXI; i++)
      if (lane + 64 * i < nchunk)
#pragma unroll
        for (int j = 0; j < 8; j++) { const float v = cur[i].get(j); s += RMS ? v * v : v; }
    s = wave_sum(s);
    float mean = 0.f, rstd;
    if (RMS) {
      rstd = rsqrtf(s * inv_h + eps);
    } else {
      mean = s * inv_h;
      float q = 0.f;
#pragma unroll
      for (int i = 0; i < MAXI; i++)
        if (lane + 64 * i < nchunk)
#pragma unroll
          for (int j = 0; j < 8; j++) { const float d = cur[i].get(j) - mean; q += d * d; }
      rstd = rsqrtf(wave_sum(q) * inv_h + eps);
    }
    if (lane == 0) { stats[2 * row] = mean; stats[2 * row + 1] = rstd; }
#pragma unroll
    for (int i = 0; i < MAXI; i++) {
      const int c = lane + 64 * i;
      if (c < nchunk) {
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 8; j++) {
          float r = (cur[i].get(j) - mean) * rstd * bf2f(gam[i][j]);
          if (!RMS) r += bf2f(bet[i][j]);
          o[j] = f2bf(r);
        }
        *(bf16x8*)(a + (size_t)row * h + c * 8) = o;
      }
    }
#pragma unroll
    for (int i = 0; i < MAXI; i++) cur[i] = nxt[i];
  }
}

// ---------------------------------------------------------------- column sums
// Partial sums: part[nblk][n], a row for each slab of 64 rows.  Four waves take 512 columns (16 bytes per lane, one
// contiguous kilobyte per row) of a slab, each every fourth row; their sums meet in LDS.
// The sums of dqkv are wanted once per layer and micro-batch.  In small stages, where a launch between two others costs more than
// the sums, the first norm's backward takes them along in blocks behind its own (ColsumJob; the line is in layer_backward).
constexpr int CS_ROWS = 64;  // rows per slab
__device__ __forceinline__ void colsum_slab(const bf16* __restrict__ m, int T, int n, float* __restrict__ part, int acc, int cols, int slab,
                                            float (*red)[512], int wave) {
  const int lane = threadIdx.x & 63, col = cols * 512 + lane * 8;
  const int r0 = slab * CS_ROWS, r1 = min(T, r0 + CS_ROWS);   // (no rows behind the last slab)
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (col < n) {
#pragma unroll 8
    for (int r = r0 + wave; r < r1; r += 4) {
      bf16x8 t = *(const bf16x8*)(m + (size_t)r * n + col);
#pragma unroll
      for (int j = 0; j < 8; j++) s[j] += bf2f(t[j]);
    }
  }
  float* p = part + (size_t)slab * n + col;
  const bool last = wave == 0 && col < n && r0 < T;
  f32x4 old[2] = {};                 // the earlier micro-batches' sums, requested before the waves' sums meet
  if (last && acc) { old[0] = *(const f32x4*)p; old[1] = *(const f32x4*)(p + 4); }
  if (wave > 0) {
#pragma unroll
    for (int q = 0; q < 2; q++) *(f32x4*)&red[wave - 1][lane * 8 + 4 * q] = f32x4{s[4 * q], s[4 * q + 1], s[4 * q + 2], s[4 * q + 3]};
  }
  __syncthreads();
  if (last) {
#pragma unroll
    for (int q = 0; q < 2; q++) {
      f32x4 v = f32x4{s[4 * q], s[4 * q + 1], s[4 * q + 2], s[4 * q + 3]};
#pragma unroll
      for (int w = 0; w < 3; w++) v += *(const f32x4*)&red[w][lane * 8 + 4 * q];
      *(f32x4*)(p + 4 * q) = acc ? old[q] + v : v;
    }
  }
}
__global__ __launch_bounds__(NT) void colsum_partial_kernel(ColsumJob c, int T) {
  __shared__ __attribute__((aligned(16))) float red[3][512];
  colsum_slab((const bf16*)c.m, T, c.n, c.part, c.acc, blockIdx.x, blockIdx.y, red, threadIdx.x >> 6);
}
// Block `block` of those behind a norm backward's own: eight waves, two slabs.
constexpr int kColsumLds = 2 * 3 * 512;   // floats
int colsum_tail(const ColsumJob* c, int T) { return c ? (c->n + 511) / 512 * ((ah::colsum_blocks(T) + 1) / 2) : 0; }
__device__ __forceinline__ void colsum_tail_block(const ColsumJob& c, int T, int block, float* red) {
  const int wide = (c.n + 511) / 512, wave = threadIdx.x >> 6, half = wave >> 2;
  colsum_slab((const bf16*)c.m, T, c.n, c.part, c.acc, block % wide, block / wide * 2 + half, (float(*)[512])(red + half * 3 * 512), wave & 3);
}

// ---------------------------------------------------------------- norm backward
// keep, optional: a copy of dres (the stage's output gradient, which a group's weight gradients need after the call; 4096 x 4096:
// 30.5 us with and 30.4 without, a copy kernel 13.0).
// Block b handles rows b, b + nblk, b + 2*nblk, ... (so that the blocks, which advance together, read one
// contiguous stretch of memory at a time and spread over all HBM channels); a thread keeps its columns for
// all of them, so the three column sums accumulate in registers and leave the block once.  512 threads (two waves per
// SIMD), rows in batches of RB; the loads of the next batch are issued before the current one is
// reduced, so that memory latency, the block reduction and the arithmetic overlap.
constexpr int NTB = 512;  // threads per block of the norm backward; MAXC here = ceil(hidden / 4096)

template <bool RMS, int MAXC, bool XF32, bool JOB>
__global__ __launch_bounds__(NTB) void norm_bwd_kernel(const bf16* __restrict__ da, const void* __restrict__ x,
                                                       const float* __restrict__ stats, const bf16* __restrict__ gamma,
                                                       const bf16* __restrict__ dres, bf16* __restrict__ dx,
                                                       float* __restrict__ part, int T, int h, int rpb, int acc, bf16* __restrict__ keep, int nblk_job, ColsumJob job) {
  const int nblk = JOB ? nblk_job : gridDim.x;
  constexpr int RB = MAXC <= 1 ? 2 : 1;  // rows per batch: two keep a 4096-wide row kernel at 125 registers (36.8 us; four rows 39.6, one 38.4)
  constexpr int NWV = NTB / 64;
  constexpr bool PIPE = MAXC <= 2;  // wider rows (hidden > 8192) leave no registers for a second batch, and spill a few
  __shared__ float red[2][NWV][2 * RB];                     // double-buffered: one block barrier per batch
  if constexpr (JOB) {
    __shared__ __attribute__((aligned(16))) float job_red[kColsumLds];
    if ((int)blockIdx.x >= nblk) return colsum_tail_block(job, T, blockIdx.x - nblk, job_red);
  }
  const int nchunk = h >> 3;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float inv_h = 1.f / h;
  // the gain stays packed (bf16x8 per chunk: a quarter of the registers of a float copy; rows wider than 8192 need the room)
  bf16x8 gam[MAXC];
  float s_g[MAXC][8], s_b[MAXC][8], s_r[MAXC][8];
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = threadIdx.x + i * NTB;
    if (c < nchunk) {
      gam[i] = *(const bf16x8*)(gamma + c * 8);
#pragma unroll
      for (int j = 0; j < 8; j++) { s_g[i][j] = 0.f; s_b[i][j] = 0.f; s_r[i][j] = 0.f; }
    }
  }
  // the block's rows are j * nblk + blockIdx.x for j in [r0, r1)
  const int r0 = 0, r1 = (T - (int)blockIdx.x + nblk - 1) / nblk;
  XVec<XF32> tx[RB][MAXC];
  bf16x8 td[RB][MAXC], tr[RB][MAXC];   // current batch
  XVec<XF32> nx[PIPE ? RB : 1][PIPE ? MAXC : 1];
  bf16x8 nd[PIPE ? RB : 1][PIPE ? MAXC : 1], nr[PIPE ? RB : 1][PIPE ? MAXC : 1];  // next batch
  float mean[RB], rstd[RB], nmean[PIPE ? RB : 1], nrstd[PIPE ? RB : 1];
  // a short last batch repeats its last row; the copies are computed but neither summed nor stored
  auto fetch = [&](int rb, auto& fx, auto& fd, auto& fr, auto& fm, auto& fs) {
#pragma unroll
    for (int k = 0; k < RB; k++) {
      const int row = min(rb + k, r1 - 1) * nblk + blockIdx.x;
#pragma unroll
      for (int i = 0; i < MAXC; i++) {
        const int c = threadIdx.x + i * NTB;
        if (c < nchunk) {
          fx[k][i].load(x, (size_t)row * h + c * 8);
          fd[k][i] = *(const bf16x8*)(da + (size_t)row * h + c * 8);
          fr[k][i] = *(const bf16x8*)(dres + (size_t)row * h + c * 8);
        }
      }
      fm[k] = RMS ? 0.f : stats[2 * row];
      fs[k] = stats[2 * row + 1];
    }
  };
  if (PIPE && r0 < r1) fetch(r0, tx, td, tr, mean, rstd);
  int buf = 0;
  for (int rb = r0; rb < r1; rb += RB, buf ^= 1) {
    if constexpr (PIPE) {
      if (rb + RB < r1) fetch(rb + RB, nx, nd, nr, nmean, nrstd);
    } else {
      fetch(rb, tx, td, tr, mean, rstd);
    }
    float sums[2 * RB];
#pragma unroll
    for (int k = 0; k < RB; k++) {
      const bool live = rb + k < r1;
      const float nm = -mean[k] * rstd[k];
      float sw = 0.f, swx = 0.f;
#pragma unroll
      for (int i = 0; i < MAXC; i++) {
        if (threadIdx.x + i * NTB < nchunk) {
#pragma unroll
          for (int j = 0; j < 8; j++) {
            const float d = bf2f(td[k][i][j]);
            const float xh = __builtin_fmaf(tx[k][i].get(j), rstd[k], nm);
            const float w = d * bf2f(gam[i][j]);
            sw += w;
            swx = __builtin_fmaf(w, xh, swx);
            if (live) { s_g[i][j] = __builtin_fmaf(d, xh, s_g[i][j]); s_b[i][j] += d; }
          }
        }
      }
      sums[2 * k] = wave_sum(sw);
      sums[2 * k + 1] = wave_sum(swx);
    }
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < 2 * RB; k++) red[buf][wave][k] = sums[k];
    }
    __syncthreads();  // the other half of red was last read before the previous barrier
#pragma unroll
    for (int k = 0; k < RB; k++) {
      if (rb + k >= r1) break;
      const int row = (rb + k) * nblk + blockIdx.x;
      float c1 = 0.f, c2 = 0.f;
#pragma unroll
      for (int w8 = 0; w8 < NWV; w8++) { c1 += red[buf][w8][2 * k]; c2 += red[buf][w8][2 * k + 1]; }
      c1 = RMS ? 0.f : c1 * inv_h;
      c2 *= inv_h;
      const float nm = -mean[k] * rstd[k];
#pragma unroll
      for (int i = 0; i < MAXC; i++) {
        const int c = threadIdx.x + i * NTB;
        if (c < nchunk) {
          bf16x8 o;
#pragma unroll
          for (int j = 0; j < 8; j++) {
            const float r = bf2f(tr[k][i][j]);
            const float xh = __builtin_fmaf(tx[k][i].get(j), rstd[k], nm);
            const float w = bf2f(td[k][i][j]) * bf2f(gam[i][j]);
            s_r[i][j] += r;
            o[j] = f2bf(r + rstd[k] * (w - c1 - xh * c2));
          }
          *(bf16x8*)(dx + (size_t)row * h + c * 8) = o;
          if (keep) *(bf16x8*)(keep + (size_t)row * h + c * 8) = tr[k][i];
        }
      }
    }
    if constexpr (PIPE) {
#pragma unroll
      for (int k = 0; k < RB; k++) {
        mean[k] = nmean[k];
        rstd[k] = nrstd[k];
#pragma unroll
        for (int i = 0; i < MAXC; i++) { tx[k][i] = nx[k][i]; td[k][i] = nd[k][i]; tr[k][i] = nr[k][i]; }
      }
    }
  }
  // The earlier micro-batches' sums are requested all at once: added value by value, each load waits behind the store
  // before it (4096 x 4096: 35.6 -> 31.3 us, 2048 x 2048: 17.5 -> 13.6).
#pragma unroll
  for (int i = 0; i < MAXC; i++) {
    const int c = threadIdx.x + i * NTB;
    if (c < nchunk) {
      f32x4 v[3][2], old[3][2];
#pragma unroll
      for (int q = 0; q < 2; q++) {
        const int j = 4 * q;
        v[0][q] = f32x4{s_g[i][j], s_g[i][j + 1], s_g[i][j + 2], s_g[i][j + 3]};
        v[1][q] = f32x4{s_b[i][j], s_b[i][j + 1], s_b[i][j + 2], s_b[i][j + 3]};
        v[2][q] = f32x4{s_r[i][j], s_r[i][j + 1], s_r[i][j + 2], s_r[i][j + 3]};
      }
      float* p = part + (size_t)blockIdx.x * h + c * 8;
      const size_t step = (size_t)nblk * h;
      if (acc) {
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
          for (int q = 0; q < 2; q++) old[a][q] = *(const f32x4*)(p + a * step + 4 * q);
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
          for (int q = 0; q < 2; q++) v[a][q] += old[a][q];
      }
#pragma unroll
      for (int a = 0; a < 3; a++)
#pragma unroll
        for (int q = 0; q < 2; q++) *(f32x4*)(p + a * step + 4 * q) = v[a][q];
    }
  }
}

// ---------------------------------------------------------------- norm backward, rows up to 1024 wide: one wave per row
// In the kernel above a 1024-wide row keeps 128 of a block's 512 threads busy, and every batch waits for a block
// reduction.  Here a wave keeps a whole row in registers (MAXI chunks of 8 values per lane) and reduces it by shuffles,
// with its next row's loads issued before the current one is reduced; its column sums stay in registers over all its
// rows, and the waves of a block add theirs up in LDS once, at the end.  4096 x 1024: 22.4 -> 10.7 us (34 MB: 6.5 us at the
// rate of a large copy), 256 x 256: 7.6 -> 4.5 us.  At 2048 columns the sums and two rows no longer fit the registers of
// two waves to a SIMD, and the kernel above is the faster one (13.6 against 14.6 us for 2048 rows).
constexpr int NWB = 8;  // waves per block
template <bool RMS, int MAXI, bool XF32, bool JOB>
__global__ __launch_bounds__(64 * NWB) void norm_bwd_wave_kernel(const bf16* __restrict__ da, const void* __restrict__ x,
                                                                const float* __restrict__ stats, const bf16* __restrict__ gamma,
                                                                const bf16* __restrict__ dres, bf16* __restrict__ dx,
                                                                float* __restrict__ part, int T, int h, int acc, bf16* __restrict__ keep, int nblk_job,
                                                                ColsumJob job) {
  const int nblk = JOB ? nblk_job : gridDim.x;
  __shared__ __attribute__((aligned(16))) float red[NWB][MAXI * 512];
  if constexpr (JOB) {
    static_assert(NWB * MAXI * 512 >= kColsumLds && NWB == 8, "room for the column sums");
    if ((int)blockIdx.x >= nblk) return colsum_tail_block(job, T, blockIdx.x - nblk, &red[0][0]);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nchunk = h >> 3;
  const float inv_h = 1.f / h;
  bf16x8 gam[MAXI];
  float sums[3][MAXI][8];
#pragma unroll
  for (int i = 0; i < MAXI; i++) {
    if (lane + 64 * i < nchunk) gam[i] = *(const bf16x8*)(gamma + (lane + 64 * i) * 8);
#pragma unroll
    for (int j = 0; j < 8; j++) { sums[0][i][j] = 0.f; sums[1][i][j] = 0.f; sums[2][i][j] = 0.f; }
  }
  // rows blockIdx + nblk * (wave + 8 k): blocks that advance together read one contiguous stretch of memory
  const int stride = nblk * NWB;
  int row = blockIdx.x + nblk * wave;
  XVec<XF32> cx[MAXI], nx[MAXI];
  bf16x8 cd[MAXI], cr[MAXI], nd[MAXI], nr[MAXI];
  float mean = 0.f, rstd = 0.f, nmean = 0.f, nrstd = 0.f;
  auto fetch = [&](int r, auto& fx, auto& fd, auto& fr, float& fm, float& fs) {
#pragma unroll
    for (int i = 0; i < MAXI; i++)
      if (lane + 64 * i < nchunk) {
        const size_t e = (size_t)r * h + (lane + 64 * i) * 8;
        fx[i].load(x, e);
        fd[i] = *(const bf16x8*)(da + e);
        fr[i] = *(const bf16x8*)(dres + e);
      }
    fm = RMS ? 0.f : stats[2 * r];
    fs = stats[2 * r + 1];
  };
  if (row < T) fetch(row, cx, cd, cr, mean, rstd);
  for (; row < T; row += stride) {
    if (row + stride < T) fetch(row + stride, nx, nd, nr, nmean, nrstd);
    const float nm = -mean * rstd;
    float sw = 0.f, swx = 0.f;
#pragma unroll
    for (int i = 0; i < MAXI; i++)
      if (lane + 64 * i < nchunk)
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const float d = bf2f(cd[i][j]);
          const float xh = __builtin_fmaf(cx[i].get(j), rstd, nm);
          const float w = d * bf2f(gam[i][j]);
          sw += w;
          swx = __builtin_fmaf(w, xh, swx);
          sums[0][i][j] = __builtin_fmaf(d, xh, sums[0][i][j]);
          sums[1][i][j] += d;
        }
    const float c1 = RMS ? 0.f : wave_sum(sw) * inv_h;
    const float c2 = wave_sum(swx) * inv_h;
#pragma unroll
    for (int i = 0; i < MAXI; i++)
      if (lane + 64 * i < nchunk) {
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 8; j++) {
          const float r = bf2f(cr[i][j]);
          const float xh = __builtin_fmaf(cx[i].get(j), rstd, nm);
          const float w = bf2f(cd[i][j]) * bf2f(gam[i][j]);
          sums[2][i][j] += r;
          o[j] = f2bf(r + rstd * (w - c1 - xh * c2));
        }
        *(bf16x8*)(dx + (size_t)row * h + (lane + 64 * i) * 8) = o;
        if (keep) *(bf16x8*)(keep + (size_t)row * h + (lane + 64 * i) * 8) = cr[i];
      }
    mean = nmean;
    rstd = nrstd;
#pragma unroll
    for (int i = 0; i < MAXI; i++) { cx[i] = nx[i]; cd[i] = nd[i]; cr[i] = nr[i]; }
  }
  const int c = threadIdx.x * 4;  // this thread's four columns of the block's sums (h <= 4 threads)
  float* p = part + (size_t)blockIdx.x * h + c;
  const size_t step = (size_t)nblk * h;
  f32x4 old[3];                   // the earlier micro-batches' sums, requested before the waves' sums meet
#pragma unroll
  for (int a = 0; a < 3; a++) old[a] = acc && c < h ? *(const f32x4*)(p + a * step) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int a = 0; a < 3; a++) {
    if (a > 0) __syncthreads();  // the previous sums have been read
#pragma unroll
    for (int i = 0; i < MAXI; i++)
      if (lane + 64 * i < nchunk) {
        float* w = &red[wave][(lane + 64 * i) * 8];
        *(f32x4*)w = f32x4{sums[a][i][0], sums[a][i][1], sums[a][i][2], sums[a][i][3]};
        *(f32x4*)(w + 4) = f32x4{sums[a][i][4], sums[a][i][5], sums[a][i][6], sums[a][i][7]};
      }
    __syncthreads();
    if (c < h) {
      f32x4 v = *(const f32x4*)&red[0][c];
#pragma unroll
      for (int w = 1; w < NWB; w++) v += *(const f32x4*)&red[w][c];
      *(f32x4*)(p + a * step) = v + old[a];
    }
  }
}

// g[c] = beta * g[c] + sum_b part[b][c] for each vector of the list.  A block takes 64 columns of one vector: 16 lanes of four columns
// side by side, 16 groups of lanes down the partial rows, whose sums meet in LDS.  Bound by latency (a few hundred KB): every
// lane has eight loads in flight, and one launch takes all the vectors that are ready.  256 partial rows of 1024 columns, three
// vectors: 11.7 us with a lane per column and two loads in flight.  Stage steps with this kernel and one launch a layer instead of
// four: 5-head stage 278.6 -> 254.7 us, the smallest 376.6 -> 352.9, BERT-Large 3792 -> 3754.
__global__ __launch_bounds__(NT) void fold_kernel(FoldList a, int beta) {
  __shared__ __attribute__((aligned(16))) float red[16][64];
  int v = 0;
  while (v + 1 < a.count && (int)blockIdx.x >= a.first[v + 1]) v++;
  const int n = a.n[v], nblk = a.nblk[v], c0 = ((int)blockIdx.x - a.first[v]) * 64;
  const int quad = threadIdx.x & 15, grp = threadIdx.x >> 4;
  const float* p = a.part[v] + c0 + 4 * quad;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  int b = grp;
  for (; b + 16 * 7 < nblk; b += 16 * 8) {
    f32x4 t[8];
#pragma unroll
    for (int k = 0; k < 8; k++) t[k] = *(const f32x4*)(p + (size_t)(b + 16 * k) * n);
#pragma unroll
    for (int k = 0; k < 8; k++) s += t[k];
  }
#pragma unroll 4
  for (; b < nblk; b += 16) s += *(const f32x4*)(p + (size_t)b * n);
  *(f32x4*)&red[grp][4 * quad] = s;
  __syncthreads();
  if (threadIdx.x < 64) {
    float sum = red[0][threadIdx.x];
#pragma unroll
    for (int k = 1; k < 16; k++) sum += red[k][threadIdx.x];
    float* g = a.g[v] + c0 + threadIdx.x;
    *g = beta ? *g + sum : sum;
  }
}

// ---------------------------------------------------------------- rotary embedding
// thread: one token, one head of Q or K, 8 pairs (i .. i+7, i + d/2 ..)
__global__ __launch_bounds__(NT) void rope_kernel(bf16* __restrict__ qkv, const float* __restrict__ cs, int T, int S, int nh,
                                                  int d, float sign) {
  const int half = d >> 1, per_head = half >> 3;
  const long idx = (long)blockIdx.x * NT + threadIdx.x;
  const long total = (long)T * 2 * nh * per_head;
  if (idx >= total) return;
  const int piece = idx % per_head;
  const int head = (idx / per_head) % (2 * nh);   // heads of Q then heads of K: contiguous in the packed row
  const int t = idx / ((long)per_head * 2 * nh);
  const int pos = t % S;
  bf16* p = qkv + (size_t)t * 3 * nh * d + (size_t)head * d + piece * 8;
  bf16x8 a = *(bf16x8*)p, b = *(bf16x8*)(p + half), oa, ob;
  const float* c = cs + ((size_t)pos * half + piece * 8) * 2;
#pragma unroll
  for (int j = 0; j < 8; j++) {
    const float co = c[2 * j], si = c[2 * j + 1] * sign;
    const float fa = bf2f(a[j]), fb = bf2f(b[j]);
    oa[j] = f2bf(fa * co - fb * si);
    ob[j] = f2bf(fb * co + fa * si);
  }
  *(bf16x8*)p = oa;
  *(bf16x8*)(p + half) = ob;
}

// ---------------------------------------------------------------- plain copy, 16 bytes per lane
__global__ __launch_bounds__(NT) void copy16_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16) {
  const size_t i = (size_t)blockIdx.x * NT + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

}  // namespace

namespace {
// one wave per row; MAXI = chunks of 8 values per lane
template <bool RMS, int MAXI>
void norm_fwd_wave_go(const void* x, bool x_f32, const void* gamma, const void* beta, void* a, float* stats, int T, int h, float eps, Keep mode, void* keep, hipStream_t s) {
  // two rows per wave where the rows suffice (the second row's loads run under the first row's arithmetic), at most 8 waves per CU
  const int waves = T >= 4096 ? 2048 : (T + 1) / 2 > 0 ? (T + 1) / 2 : 1;
  const dim3 grid((waves + NT / 64 - 1) / (NT / 64));
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(NT), 0, s, x, (const bf16*)gamma, (const bf16*)beta, (bf16*)a, stats, T, h, eps, keep); };
  if (x_f32) go(norm_fwd_wave_kernel<RMS, MAXI, true, KEEP_NONE>);
  else if (mode == KEEP_BF16) go(norm_fwd_wave_kernel<RMS, MAXI, false, KEEP_BF16>);
  else if (mode == KEEP_F32) go(norm_fwd_wave_kernel<RMS, MAXI, false, KEEP_F32>);
  else go(norm_fwd_wave_kernel<RMS, MAXI, false, KEEP_NONE>);
}

template <bool RMS, int MAXC>
void norm_fwd_go(const void* x, bool x_f32, const void* gamma, const void* beta, void* a, float* stats, int T, int h, float eps, Keep mode, void* keep, hipStream_t s) {
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(T), dim3(NT), 0, s, x, (const bf16*)gamma, (const bf16*)beta, (bf16*)a, stats, h, eps, keep); };
  if (x_f32) go(norm_fwd_kernel<RMS, MAXC, true, KEEP_NONE>);
  else if (mode == KEEP_BF16) go(norm_fwd_kernel<RMS, MAXC, false, KEEP_BF16>);
  else if (mode == KEEP_F32) go(norm_fwd_kernel<RMS, MAXC, false, KEEP_F32>);
  else go(norm_fwd_kernel<RMS, MAXC, false, KEEP_NONE>);
}
// (Instances of their own with a job: its code alone, never run, cost the block kernel 7 us at 4096 x 4096, 29.1 -> 36.4.)
template <bool RMS, int MAXC>
void norm_bwd_go(const void* da, const void* x, bool x_f32, const float* stats, const void* gamma, const void* dres, void* dx, float* part,
                 int T, int h, int acc, void* keep, const ColsumJob* job, hipStream_t s) {
  const int nblk = norm_bwd_blocks(T);
  const int rpb = (T + nblk - 1) / nblk;
  auto kernel = x_f32 ? norm_bwd_kernel<RMS, MAXC, true, false> : norm_bwd_kernel<RMS, MAXC, false, false>;
  if constexpr (!RMS)
    if (job) kernel = x_f32 ? norm_bwd_kernel<RMS, MAXC, true, true> : norm_bwd_kernel<RMS, MAXC, false, true>;
  hipLaunchKernelGGL(kernel, dim3(nblk + colsum_tail(job, T)), dim3(NTB), 0, s, (const bf16*)da, x, stats, (const bf16*)gamma, (const bf16*)dres,
                     (bf16*)dx, part, T, h, rpb, acc, (bf16*)keep, nblk, job ? *job : ColsumJob{});
}
// one wave per row, hidden <= 1024
template <bool RMS, int MAXI>
void norm_bwd_wave_go(const void* da, const void* x, bool x_f32, const float* stats, const void* gamma, const void* dres, void* dx, float* part,
                      int T, int h, int acc, void* keep, const ColsumJob* job, hipStream_t s) {
  const int nblk = norm_bwd_blocks(T);
  auto kernel = x_f32 ? norm_bwd_wave_kernel<RMS, MAXI, true, false> : norm_bwd_wave_kernel<RMS, MAXI, false, false>;
  if constexpr (!RMS)
    if (job) kernel = x_f32 ? norm_bwd_wave_kernel<RMS, MAXI, true, true> : norm_bwd_wave_kernel<RMS, MAXI, false, true>;
  hipLaunchKernelGGL(kernel, dim3(nblk + colsum_tail(job, T)), dim3(64 * NWB), 0, s, (const bf16*)da, x, stats, (const bf16*)gamma, (const bf16*)dres,
                     (bf16*)dx, part, T, h, acc, (bf16*)keep, nblk, job ? *job : ColsumJob{});
}
}  // namespace

int norm_bwd_blocks(int T) {
  static int cap = -1;
  if (cap < 0) cap = getenv("AH_NORM_NBLK") ? atoi(getenv("AH_NORM_NBLK")) : 256;  // tuning aid
  return T / 4 < cap ? (T / 4 > 0 ? T / 4 : 1) : cap;
}

#define AH_BY_CHUNKS(FN, RMS, ...)                                   \
  do {                                                               \
    const int nc = (h + 2047) / 2048;                                \
    if (nc <= 1) FN<RMS, 1>(__VA_ARGS__);                            \
    else if (nc == 2) FN<RMS, 2>(__VA_ARGS__);                       \
    else if (nc == 3) FN<RMS, 3>(__VA_ARGS__);                       \
    else if (nc == 4) FN<RMS, 4>(__VA_ARGS__);                       \
    else FN<RMS, 8>(__VA_ARGS__);                                    \
  } while (0)

hipError_t launch_norm_fwd(bool rms, const void* x, const void* gamma, const void* beta, void* a, float* stats, int T,
                           int h, float eps, hipStream_t s, bool x_f32, void* keep, bool keep_f32) {
  if (x_f32 && keep) return hipErrorInvalidValue;
  const Keep mode = !keep ? KEEP_NONE : keep_f32 ? KEEP_F32 : KEEP_BF16;
  if (h % 8 || h > 16384) return hipErrorInvalidValue;
  static int wave_rows = -1;
  if (wave_rows < 0) wave_rows = getenv("AH_NORM_FWD_BLOCK_PER_ROW") ? 0 : 1;  // tuning aid
  const int per_lane = (h / 8 + 63) / 64;   // chunks per lane with one wave per row
  if (wave_rows && per_lane <= 16) {
#define AH_WAVE_ROWS(RMS)                                                                                     \
    do {                                                                                                      \
      if (per_lane <= 2) norm_fwd_wave_go<RMS, 2>(x, x_f32, gamma, beta, a, stats, T, h, eps, mode, keep, s);             \
      else if (per_lane <= 4) norm_fwd_wave_go<RMS, 4>(x, x_f32, gamma, beta, a, stats, T, h, eps, mode, keep, s);        \
      else if (per_lane <= 8) norm_fwd_wave_go<RMS, 8>(x, x_f32, gamma, beta, a, stats, T, h, eps, mode, keep, s);        \
      else if (per_lane <= 12) norm_fwd_wave_go<RMS, 12>(x, x_f32, gamma, beta, a, stats, T, h, eps, mode, keep, s);      \
      else norm_fwd_wave_go<RMS, 16>(x, x_f32, gamma, beta, a, stats, T, h, eps, mode, keep, s);                          \
    } while (0)
    if (rms) AH_WAVE_ROWS(true);
    else AH_WAVE_ROWS(false);
#undef AH_WAVE_ROWS
    return hipGetLastError();
  }
  if (rms) AH_BY_CHUNKS(norm_fwd_go, true, x, x_f32, gamma, beta, a, stats, T, h, eps, mode, keep, s);
  else AH_BY_CHUNKS(norm_fwd_go, false, x, x_f32, gamma, beta, a, stats, T, h, eps, mode, keep, s);
  return hipGetLastError();
}

#define AH_BWD_BY_CHUNKS(RMS)                                                                        \
  do {                                                                                               \
    const int nc = (h + 4095) / 4096;                                                                \
    if (h <= 512) norm_bwd_wave_go<RMS, 1>(da, x, x_f32, stats, gamma, dres, dx, part, T, h, acc, keep, job, s);       \
    else if (h <= 1024) norm_bwd_wave_go<RMS, 2>(da, x, x_f32, stats, gamma, dres, dx, part, T, h, acc, keep, job, s); \
    else if (nc <= 1) norm_bwd_go<RMS, 1>(da, x, x_f32, stats, gamma, dres, dx, part, T, h, acc, keep, job, s);      \
    else if (nc == 2) norm_bwd_go<RMS, 2>(da, x, x_f32, stats, gamma, dres, dx, part, T, h, acc, keep, job, s); \
    else norm_bwd_go<RMS, 4>(da, x, x_f32, stats, gamma, dres, dx, part, T, h, acc, keep, job, s);              \
  } while (0)

hipError_t launch_norm_bwd(bool rms, const void* da, const void* x, const float* stats, const void* gamma, const void* dres,
                           void* dx, float* part, int T, int h, hipStream_t s, int acc, bool x_f32, void* keep, const ColsumJob* job) {
  if (job && (rms || job->n % 8)) return hipErrorInvalidValue;   // (the RMS-norm stages have no such bias)
  if (h % 8 || h > 16384) return hipErrorInvalidValue;
  if (rms) AH_BWD_BY_CHUNKS(true);
  else AH_BWD_BY_CHUNKS(false);
  return hipGetLastError();
}

hipError_t launch_fold(const FoldList& a, int beta, hipStream_t s) {
  if (a.count == 0) return hipSuccess;
  for (int v = 0; v < a.count; v++)
    if (a.n[v] % 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fold_kernel, dim3(a.first[a.count]), dim3(NT), 0, s, a, beta);
  return hipGetLastError();
}

int colsum_blocks(int T) { return (T + CS_ROWS - 1) / CS_ROWS; }

hipError_t launch_colsum_partial(const ColsumJob& c, int T, hipStream_t s) {
  if (c.n % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((c.n + 511) / 512, colsum_blocks(T)), dim3(NT), 0, s, c, T);
  return hipGetLastError();
}

hipError_t launch_rope(void* qkv, const float* cos_sin, int T, int S, int nh, int d, float sign, hipStream_t s) {
  const long total = (long)T * 2 * nh * (d / 16);
  hipLaunchKernelGGL(rope_kernel, dim3((unsigned)((total + NT - 1) / NT)), dim3(NT), 0, s, (bf16*)qkv, cos_sin, T, S, nh, d, sign);
  return hipGetLastError();
}

hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  if (bytes % 16) return hipErrorInvalidValue;
  const size_t n16 = bytes / 16;
  hipLaunchKernelGGL(copy16_kernel, dim3((unsigned)((n16 + NT - 1) / NT)), dim3(NT), 0, s, (const uint4*)src, (uint4*)dst, n16);
  return hipGetLastError();
}

}  // namespace ah
