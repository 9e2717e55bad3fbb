// Shared device helpers for the gfx950 kernels of the stage library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ah {

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

#define AH_LDS(p) ((__attribute__((address_space(3))) void*)(p))

// 16 bytes per lane, global memory straight into LDS: lane i of the wave lands at lds_base + 16*i (lds_base must be
// wave-uniform).  The source is a wave-uniform base plus a 32-bit byte offset per lane: the instruction has a form for
// just that (base in scalar registers).  The compiler only sees it if the widening of the offset stays beside the load: for a
// loop-invariant offset it hoists the widening and then spends two vector registers and a 64-bit add per load, and
// the load itself issues more slowly.  The empty statement makes the offset look rewritten each time (no instruction).
// GEMM loop, 256 x 256 tiles, against an address per lane: 4096 x 4096 x 8192 NT 198.9 -> 191.1 us, TN 203.5 -> 195.3; 4096 x 8192 x 4096 NN
// 201.3 -> 192.3 (same bits).
__device__ __forceinline__ void load16_to_lds(const void* base, uint32_t& off, void* lds_base) {
  asm("" : "+v"(off));
  __builtin_amdgcn_global_load_lds((const char*)base + off, AH_LDS(lds_base), 16, 0, 0);
}

// The same as an assembly statement: the compiler neither waits for it nor orders LDS reads after it (that is the kernel's
// business: a wait by count, and a compiler fence), and does not take it for an access that may return out of order
// with LDS reads.  M0 is set in the same statement and named as overwritten.
__device__ __forceinline__ uint32_t lds_offset(const void* p) { return (uint32_t)(uintptr_t)AH_LDS(p); }
__device__ __forceinline__ void load16_to_lds_uncounted(const void* base, uint32_t off, void* lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_offset(lds)), "v"(off), "s"(base) : "memory", "m0");
}

// Transposing LDS read: within each group of 16 lanes, lane j supplies the
// address of 4 consecutive 16-bit elements; lane i receives element (i % 4) of
// the data addressed by lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4.  With lane j
// pointing at row j/4, columns 4*(j%4).. of a row-major block, lane i ends up
// with 4 consecutive rows of column i.
__device__ __forceinline__ bf16x4 lds_read_tr4(const void* p) {
  s16x4 t = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
  return __builtin_bit_cast(bf16x4, t);
}

__device__ __forceinline__ bf16x8 cat4(bf16x4 a, bf16x4 b) {
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ float bf2f(bf16 v) { return (float)v; }
__device__ __forceinline__ bf16 f2bf(float v) { return (bf16)v; }  // round to nearest even

// tanh-form GeLU written through the logistic function: with z = kappa (u + 0.044715 u^3),
// 0.5 (1 + tanh z) = sigma(2 z), so gelu(u) = u sigma(2z) and
// gelu'(u) = sigma(2z) (1 + 2 u (1 - sigma(2z)) kappa (1 + 0.134145 u^2)).
// sigma uses the hardware exp2 and reciprocal (1 ulp each); exp2 overflow gives sigma = 0 exactly.  The constants are
// multiplied out: these run once per element in GEMM epilogues, whose length the vector instructions bound.
__device__ __forceinline__ float sigmoid2z(float u, float uu) {   // uu = u * u
  constexpr float c1 = -2.0 * 1.4426950408889634 * 0.7978845608028654, c3 = c1 * 0.044715;   // exp2(c1 u + c3 u^3) = exp(-2 z)
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u * __builtin_fmaf(c3, uu, c1)));
}
__device__ __forceinline__ float gelu_f(float u) { return u * sigmoid2z(u, u * u); }
__device__ __forceinline__ float gelu_grad_f(float u) {
  constexpr float d1 = 2.0 * 0.7978845608028654, d3 = d1 * 0.134145;
  const float uu = u * u, s = sigmoid2z(u, uu);
  return __builtin_fmaf(s * (1.0f - s) * u, __builtin_fmaf(d3, uu, d1), s);   // (u first: s (1 - s) is 0 long before u^3 overflows, from 1e13 on)
}

// silu(x) = x sigma(x) through the hardware exp2 and reciprocal
__device__ __forceinline__ float silu_f(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * x));
}

// s_waitcnt immediate (gfx9 encoding): vmcnt = n (6 bits, split), lgkmcnt = 0, expcnt untouched
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace ah
