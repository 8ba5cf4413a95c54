// Building blocks of the kernels that keep a whole register file of sums per wave (one workgroup per compute unit):
// unrolled schedules, direct loads without address arithmetic, products that add in accumulation registers.
#pragma once
#include <utility>
#include "common.hpp"

namespace glowq {

// a pointer that is the same in every lane, moved to scalar registers
template <typename T> __device__ inline T* uniform_ptr(T* p) {
  const unsigned long long v = (unsigned long long)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (T*)(((unsigned long long)hi << 32) | lo);
}

// f(0), f(1), .. f(N - 1) with compile-time indexes (the K tile's body is past what `#pragma unroll` unrolls)
template <class F, int... I> __device__ __attribute__((always_inline)) inline void for_each_index(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __attribute__((always_inline)) inline void for_each_index(F f) {
  for_each_index(f, std::make_integer_sequence<int, N>{});
}

// Direct global -> LDS loads with a uniform base and a 32-bit byte offset per lane: no vector-ALU address arithmetic
__device__ inline void lds_dma16_off(const void* base, uint32_t off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}
__device__ inline void lds_dma16_off_coherent(const void* base, uint32_t off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 sc1" : : "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}
__device__ inline void lds_dma4_off(const void* base, uint32_t off, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" : : "v"(off), "s"(base), "s"(lds_base) : "memory", "m0");
}
// LDS reads that the compiler sees (it places their waits; the direct loads above are unknown to it)
__device__ inline u32x4_t lds16(uint32_t addr) { return *(const __attribute__((address_space(3))) u32x4_t*)addr; }
__device__ inline uint32_t lds4(uint32_t addr) { return *(const __attribute__((address_space(3))) uint32_t*)addr; }

// acc += a x b with the sum in accumulation registers, in place.  As assembly: around the builtin the register
// allocator moves the sums about (three copies per product).  It does not see the instruction's hazards either: an
// operand has to be written two instructions ahead by the vector ALU, a sum to rest before it is read (acc_settle).
// build.py reads the listing of every build for both.
template <int ACT> __device__ inline void mfma_acc(float4_t& acc, u32x4_t a, u32x4_t b) {
  if constexpr (ACT == ACT_F16) asm("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
  else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ inline void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15"); }
__device__ inline void acc_settled(float4_t& acc) { asm volatile("" : "+a"(acc)); }     // nothing that reads it moves above

}  // namespace glowq
