// Operand fragments of the matrix instructions, read from a stage: 128 bytes of k of every row, 16-byte chunk c of row r
// in slot c ^ ((r >> 1) & 7) of the row.
//
// Every kernel adds the products of an output in ascending k, so a result does not depend on the kernel that a problem size
// selects: fp32 instructions are chains of fused multiply-adds over their k, lane group after lane group, and bf16
// instructions of 16 and of 32 k round alike (both checked bit for bit).
#pragma once
#include <hip/hip_runtime.h>

namespace br {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// An address that is uniform over the wave; saying so keeps it in scalar registers in every instantiation.
__device__ inline const char* scalar_ptr(const char* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return reinterpret_cast<const char*>(((unsigned long long)hi << 32) | lo);
}

// 32x32 instructions (bf16, one a chunk pair): lanes 0..31 hold the first half of an instruction's k, lanes 32..63 the second.  The fragments of chunk
// pair p (chunks 2p and 2p + 1) are at offset(row, lane / 32) ^ (p << 5).
struct GemmFrag32 {
  typedef __bf16 type __attribute__((ext_vector_type(8)));
  static __device__ inline int offset(int row, int lh) { return row * 128 + ((lh ^ ((row >> 1) & 7)) << 4); }
  static __device__ inline type load(const char* p, int off) { return *reinterpret_cast<const type*>(p + off); }
  static __device__ inline f32x16 mma(const type& w, const type& a, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, a, c, 0, 0, 0);
  }
};

// 16x16 instructions: fragment i of a stage for lane group g = lane / 16, at offset(row, g) ^ (i * FLIP), is chunk 4 i + g (bf16,
// 32 k an instruction) or word g of chunk i (fp32, 4 k).
template <typename T>
struct GemmFrag16;
template <>
struct GemmFrag16<__bf16> {
  typedef __bf16 type __attribute__((ext_vector_type(8)));
  static constexpr int COUNT = 2, FLIP = 64;  // fragments of a stage
  static __device__ inline int offset(int row, int g) { return row * 128 + ((g ^ ((row >> 1) & 7)) << 4); }
  static __device__ inline f32x4 mma(const type& w, const type& a, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a, c, 0, 0, 0);
  }
};
template <>
struct GemmFrag16<float> {
  typedef float type;
  static constexpr int COUNT = 8, FLIP = 16;
  static __device__ inline int offset(int row, int g) { return row * 128 + (((row >> 1) & 7) << 4) + g * 4; }
  static __device__ inline f32x4 mma(float w, float a, const f32x4& c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(w, a, c, 0, 0, 0); }
};

}  // namespace br
