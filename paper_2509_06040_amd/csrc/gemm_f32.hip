// fp32 GEMM: C[m, n] = sum_k A[m, k] W[n, k] with the fused epilogues, on the matrix cores
// (v_mfma_f32_32x32x2_f32 and 16x16x4, full fp32; 157 TFLOP/s nominal, twice the vector rate).  This file holds the
// choice between the ring kernel (gemm_f32_ring.hip) and the kernel for small problems (gemm_small.hip), and a vector
// kernel for operands that cannot be fetched in 16-byte pieces.
#include "common.h"
#include "dispatch.h"
#include "dit.h"
#include "prof.h"

namespace br {

// Any K, leading dimension and alignment: 64x64 tile, 16-deep, 4x4 outputs per thread, vector arithmetic.
// The matrix-core kernels fetch 16 bytes at a time and need K, lda and ldw divisible by 4 and 16-byte
// aligned operands, which every network has; single-operator calls need not.
template <int MODE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int lda, const float* __restrict__ W,
                                                       int ldw, int M, int N, int K, Epilogue<MODE, float> epi) {
  __shared__ float sA[16][64 + 4], sW[16][64 + 4];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + i * 256, row = e >> 4, kk = e & 15;
      const int gm = m0 + row, gn = n0 + row, gk = k0 + kk;
      sA[kk][row] = (gm < M && gk < K) ? A[(size_t)gm * lda + gk] : 0.f;
      sW[kk][row] = (gn < N && gk < K) ? W[(size_t)gn * ldw + gk] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = sA[kk][ty * 4 + i];
        w[i] = sW[kk][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
    }
    __syncthreads();
  }
  const int n = n0 + tx * 4;
  if (n >= N) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m < M) {
      const auto r = epi.row(m);
      epi.store(r, n, acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    }
  }
}

template <int MODE>
static br_status gemm_f32_any(const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               hipStream_t st) {
  Epilogue<MODE, float> epi{ea};
  hipLaunchKernelGGL((gemm_f32_kernel<MODE>), dim3(cdiv(N, 64), cdiv(M, 64)), dim3(256), 0, st, A, lda, W, ldw, M, N, K,
                     epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

enum { F32_TILE_32 = 0, F32_RING = 6 };  // variants

template <int MODE>
static br_status gemm_f32_mode(const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               int variant, hipStream_t st) {
  const bool chunks = K % 4 == 0 && lda % 4 == 0 && ldw % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0;
  if (!chunks) return gemm_f32_any<MODE>(A, lda, W, ldw, M, N, K, ea, st);
  // (patch embedding, condition embedding and unpatchify are a few per cent of a network: one form is enough)
  if (variant != F32_TILE_32 && gemm_f32_ring_supported(MODE, K, lda, ldw)) {
    int rb = variant < 0 ? 0 : variant >> 24 & 127, cb = variant >> 4 & 1 ? 2 : 1;
    const bool forced = variant >= 0 && (variant & 15) == F32_RING && rb >= 2 && rb <= rule::F32_RING_MAX_RB;
    const int units = device_cu_count();
    if (forced || !rule::f32_small(M, N, units)) {
      if (!forced) rule::f32_ring_tile(M, N, K, MODE == EPI_BIAS_GATE_RES ? ea.L : 0, units, &rb, &cb);
      return launch_gemm_f32_ring(MODE, A, lda, W, ldw, M, N, K, ea, rb, cb, st);
    }
  }
  return launch_gemm_small(BR_F32, MODE, A, lda, W, ldw, M, N, K, ea, st);
}

br_status launch_gemm_f32(int mode, const float* A, int lda, const float* W, int ldw, int M, int N, int K,
                          const EpiArgs& ea, int variant, hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return gemm_f32_mode<EPI_BIAS>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_BIAS_GELU: return gemm_f32_mode<EPI_BIAS_GELU>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_BIAS_GATE_RES: return gemm_f32_mode<EPI_BIAS_GATE_RES>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_PATCH_EMBED: return gemm_f32_mode<EPI_PATCH_EMBED>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_BIAS_F32: return gemm_f32_mode<EPI_BIAS_F32>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_UNPATCH: return gemm_f32_mode<EPI_UNPATCH>(A, lda, W, ldw, M, N, K, ea, variant, st);
  }
  return fail(BR_EINVAL, "gemm: unknown epilogue");
}

}  // namespace br
