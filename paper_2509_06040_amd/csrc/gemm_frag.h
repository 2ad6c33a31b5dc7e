// Operand fragments of the 32x32 matrix instructions: 16 bytes of k per lane.  The contraction order inside
// a pair of 16-byte chunks (lanes 0..31 hold the first, lanes 32..63 the second) is free as long as both
// operands use the same one, so fp32 takes its four elements one instruction at a time (k = e and 4 + e).
#pragma once
#include <hip/hip_runtime.h>

namespace br {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// An address that is uniform over the wave; saying so keeps it in scalar registers in every instantiation.
__device__ inline const char* scalar_ptr(const char* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return reinterpret_cast<const char*>(((unsigned long long)hi << 32) | lo);
}

template <typename T>
struct GemmFrag;
template <>
struct GemmFrag<__bf16> {
  typedef __bf16 type __attribute__((ext_vector_type(8)));
  static constexpr int STEPS = 1;  // matrix instructions per chunk pair
  static __device__ inline f32x16 mma(const type& w, const type& a, const f32x16& c, int) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, a, c, 0, 0, 0);
  }
};
template <>
struct GemmFrag<float> {
  typedef float type __attribute__((ext_vector_type(4)));
  static constexpr int STEPS = 4;
  static __device__ inline f32x16 mma(const type& w, const type& a, const f32x16& c, int e) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(w[e], a[e], c, 0, 0, 0);
  }
};

}  // namespace br
