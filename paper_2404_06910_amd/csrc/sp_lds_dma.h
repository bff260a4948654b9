// What the two bf16 prefill kernels share: LDS-DMA, the exchange between the half-waves, a scalar load.
#pragma once

#include "sp_device.h"

namespace sp {

typedef bf16x4 __attribute__((address_space(3))) lds_bf16x4;
typedef unsigned char __attribute__((address_space(3))) lds_byte;

// max / sum partner exchange between lane L and lane L^32 (v_permlane32_swap)
__device__ __forceinline__ float xhalf_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS-DMA: every lane moves 16 bytes from its global address straight into LDS byte
// (lds_base + 16 * lane); no staging registers.  The compiler does not track these loads:
// completion is awaited with an explicit s_waitcnt vmcnt(0) before the stage barrier.
__device__ __forceinline__ void dma16(const void *gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_base), "v"(gptr) : "memory", "m0");
}

// The same with the address split into a wave-uniform base (scalar registers) and a 32-bit per-lane
// byte offset: no vector arithmetic per instruction and no 64-bit per-lane pointers to keep alive.
__device__ __forceinline__ void dma16s(const void *sbase, uint32_t voff, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(voff), "s"(sbase)
               : "memory", "m0");
}

// One dword per lane, 64 consecutive dwords in LDS: the positions of a stage's keys.
__device__ __forceinline__ void dma4(const void *gptr, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_base), "v"(gptr) : "memory", "m0");
}

// A wave-uniform float through the scalar data path (a read; its counter is not the vector one).
__device__ __forceinline__ float sload_f32(const float *p) {
  float v;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(p) : "memory");
  return v;
}

}  // namespace sp
