// Device-side helpers shared by the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace locret {

typedef uint16_t bf16_t;  // raw bf16 bits

__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round to nearest even, a NaN stays one: v_cvt_pk_bf16_f32.  (Rounding with integer instructions and a branch for NaN was half of
// the instructions of the append and of the compaction: 4096 tokens into 8 x 128-dim heads as 4-bit rows 9.0 -> 7.6 us.)
__device__ __forceinline__ bf16_t f2bf(float f) { return __builtin_bit_cast(bf16_t, (__bf16)f); }

template <typename T> struct Elem;
template <> struct Elem<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float x) { *p = x; }
};
template <> struct Elem<bf16_t> {
  static __device__ __forceinline__ float ld(const bf16_t* p) { return bf2f(*p); }
  static __device__ __forceinline__ void st(bf16_t* p, float x) { *p = f2bf(x); }
};

// 16-byte vector of storage elements: 4 floats or 8 bf16.
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  float4 raw;
  __device__ __forceinline__ float get(int i) const { return ((const float*)&raw)[i]; }
  __device__ __forceinline__ void set(int i, float x) { ((float*)&raw)[i] = x; }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  uint4 raw;
  __device__ __forceinline__ float get(int i) const { return bf2f(((const bf16_t*)&raw)[i]); }
  __device__ __forceinline__ void set(int i, float x) { ((bf16_t*)&raw)[i] = f2bf(x); }
};

}  // namespace locret
