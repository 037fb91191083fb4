// Device helpers shared by the value-synchronised solve kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace sptrsv {

template <typename T> struct Bits;
template <> struct Bits<double> {
  using U = unsigned long long;
  // exponent all ones, quiet bit (51) clear, payload nonzero: a signalling NaN
  static constexpr U kSentinel = 0x7FF4A5A5A5A5A5A5ull;
};
template <> struct Bits<float> {
  using U = unsigned int;
  static constexpr U kSentinel = 0x7FA5A5A5u;   // quiet bit (22) clear
};

template <typename T> __device__ __forceinline__ T load_agent(const T* p) {
  using U = typename Bits<T>::U;
  const U u = __hip_atomic_load(reinterpret_cast<U*>(const_cast<T*>(p)), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
  return __builtin_bit_cast(T, u);
}

template <typename T> __device__ __forceinline__ void store_agent(T* p, T v) {
  using U = typename Bits<T>::U;
  __hip_atomic_store(reinterpret_cast<U*>(p), __builtin_bit_cast(U, v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T> __device__ __forceinline__ bool is_sentinel(T v) {
  return __builtin_bit_cast(typename Bits<T>::U, v) == Bits<T>::kSentinel;
}

// fused multiply-add in the value type (FP64 or FP32: one rounding, no
// widening)
__device__ __forceinline__ double fma_t(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}
__device__ __forceinline__ float fma_t(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}

// quiets a signalling NaN, leaves every other value unchanged
__device__ __forceinline__ double canonical(double v) { return __builtin_canonicalize(v); }
__device__ __forceinline__ float canonical(float v) { return __builtin_canonicalizef(v); }

__device__ __forceinline__ int load_status(const int* s) {
  return __hip_atomic_load(const_cast<int*>(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void raise_status(int* s, int bit) {
  __hip_atomic_fetch_or(s, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

}  // namespace sptrsv
