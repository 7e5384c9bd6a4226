// Operand fragments of the token-parallel kernels and the requests that fetch them (kernels_mfma.hip, kernels_rows.hip).
#pragma once
#include "common.h"

namespace sapo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
union Frag {
  uint4 u;
  u32x4 n;
  bf16x8 v;
  f16x8 h;
};

__device__ __forceinline__ f32x16 mfma32(const Frag& a, const Frag& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h, b.h, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma16h(const Frag& a, const Frag& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, c, 0, 0, 0);
}
// x * sigmoid(x) with the hardware reciprocal (1 ulp) instead of an IEEE division: the token-parallel SwiGLU epilogue
// evaluates 64 of these per thread and tile, where the correctly rounded division alone was a dozen instructions
// each; the result is rounded to half right after.
__device__ __forceinline__ float silu_f(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

__device__ __forceinline__ unsigned lds_addr(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) void*)p;
}
// one wave-wide 1 KiB copy global -> LDS: lane l's 16 bytes (at base + off(l)) land at lds + 16 l (no immediate offset: the
// instruction would add it to the LDS address as well)
__device__ __forceinline__ void dma16(const void* base, unsigned off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory");
}
// one wave-wide 1 KiB load into registers; the value is there after a wait and a landed() that names it
template <int IMM> __device__ __forceinline__ void reg16(u32x4& d, const void* base, unsigned off) {
  asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=v"(d) : "v"(off), "s"(base), "n"(IMM) : "memory");
}
__device__ __forceinline__ void landed(u32x4& d) { asm volatile("" : "+v"(d)); }
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

}  // namespace sapo
