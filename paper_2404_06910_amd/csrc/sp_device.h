// Device-side helpers shared by the kernels: 16-byte loads, bf16 <-> fp32, wave shuffles.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kNegBig = -1.0e30f;   // finite stand-in for "no maximum yet"

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Element-type traits: a 16-byte vector holds kVec elements.
template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kVec = 4;
  __device__ static __forceinline__ void unpack(const u32x4 &r, float *f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y); f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
  __device__ static __forceinline__ float load1(const float *p) { return *p; }
  __device__ static __forceinline__ void store1(float *p, float v) { *p = v; }
};
template <> struct Elem<__bf16> {
  static constexpr int kVec = 8;
  __device__ static __forceinline__ void unpack(const u32x4 &r, float *f) {
    f[0] = bf16_lo(r.x); f[1] = bf16_hi(r.x); f[2] = bf16_lo(r.y); f[3] = bf16_hi(r.y);
    f[4] = bf16_lo(r.z); f[5] = bf16_hi(r.z); f[6] = bf16_lo(r.w); f[7] = bf16_hi(r.w);
  }
  __device__ static __forceinline__ float load1(const __bf16 *p) { return static_cast<float>(*p); }
  __device__ static __forceinline__ void store1(__bf16 *p, float v) { *p = static_cast<__bf16>(v); }
};

// A pointer whose origin the compiler cannot see (read from a table) as one into global memory: loads through it count in
// vmcnt alone, while a flat load is also waited for as an LDS access, with everything that is in flight.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(1))) T *global_ptr(const void *p) {
  return (const __attribute__((address_space(1))) T *)p;
}

__device__ __forceinline__ u32x4 ld16(const void *p) { return *reinterpret_cast<const u32x4 *>(p); }
__device__ __forceinline__ u32x4 ld16_stream(const void *p) {      // read-once data: do not keep in cache
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
}
__device__ __forceinline__ void st16(void *p, const u32x4 &v) { *reinterpret_cast<u32x4 *>(p) = v; }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

}  // namespace sp
