// fp32 GEMM: C[m, n] = sum_k A[m, k] W[n, k] with the fused epilogues, on the matrix cores
// (v_mfma_f32_32x32x2_f32 and 16x16x4, full fp32; 157 TFLOP/s nominal, twice the vector rate).  This file holds the
// choice between the tile kernel (gemm_tile.h) and the kernel for small problems (gemm_small.hip), and a vector
// kernel for operands that cannot be fetched in 16-byte pieces.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "dit.h"
#include "gemm_tile.h"
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

template <int BM, int BN, int WGM, int WGN, int NST, int MODE>
static br_status gemm_f32_tile(const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               hipStream_t st) {
  Epilogue<MODE, float> epi{ea};
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  hipLaunchKernelGGL((gemm_tile_kernel<float, BM, BN, WGM, WGN, NST, MODE, float>), dim3(tiles_m * tiles_n), dim3(WGM * WGN * 64), 0, st,
                     A, lda, W, ldw, M, N, K, tiles_m, tiles_n, std::min(4, tiles_n), epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

enum { F32_TILE_32 = 0, F32_TILE_64 = 3, F32_TILE_128 = 5 };  // variants

// Share of the compute units' time that `tiles` equal tiles keep busy: they run in whole rounds.
static double round_fill(long long tiles) {
  const double r = (double)tiles / device_cu_count();
  return r / std::ceil(r);
}

// Measured on MI355X (gated residual, M = 1101 / 4404 / 8808 rows, N and K 1024 to 4096), all three forms
// run at a constant rate times the fill of their rounds: 133 TFLOP/s for 128x128 tiles, 132 for 64x128 and
// 102 for 32x32, each within 7 %.  The smaller tile trades rate for fill: 4404 x 1024 x 1024 takes 130 / 98 / 100 us
// (the vector kernel: 177), 4404 x 3072 x 1024 251 / 220 / 272 (401), 8808 x 4096 x 1024 558 / 570 / 728 (1011).  Far
// below one round the 32x32 form wins by its four waves per tile: 24 x 64 x 256 takes 3.7 us instead of 12.
static int f32_form(int M, int N, int K) {
  if (K % 32 != 0) return F32_TILE_32;  // the tile kernel walks K in whole stages of 32
  const double t128 = 133.0 * round_fill((long long)cdiv(M, 128) * cdiv(N, 128));
  const double t64 = 132.0 * round_fill((long long)cdiv(M, 64) * cdiv(N, 128));
  const double t32 = 102.0 * round_fill((long long)cdiv(M, 32) * cdiv(N, 32));
  // padding of ragged edges is work done for nothing
  const double used = (double)M * N;
  const double e128 = t128 * used / ((double)cdiv(M, 128) * 128 * cdiv(N, 128) * 128);
  const double e64 = t64 * used / ((double)cdiv(M, 64) * 64 * cdiv(N, 128) * 128);
  const double e32 = t32 * used / ((double)cdiv(M, 32) * 32 * cdiv(N, 32) * 32);
  if (e32 >= e64 && e32 >= e128) return F32_TILE_32;
  return e64 >= e128 ? F32_TILE_64 : F32_TILE_128;
}

template <int MODE>
static br_status gemm_f32_mode(const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               int variant, hipStream_t st) {
  const bool chunks = K % 4 == 0 && lda % 4 == 0 && ldw % 4 == 0 && (((uintptr_t)A | (uintptr_t)W) & 15) == 0;
  if (!chunks) return gemm_f32_any<MODE>(A, lda, W, ldw, M, N, K, ea, st);
  // patch embedding, condition embedding and unpatchify are a few per cent of a network: one form is enough
  constexpr bool TILED = MODE == EPI_BIAS || MODE == EPI_BIAS_GELU || MODE == EPI_BIAS_GATE_RES;
  const bool forced = variant == F32_TILE_64 || variant == F32_TILE_128 || variant == F32_TILE_32;
  const int form = forced && K % 32 == 0 ? variant : f32_form(M, N, K);
  if constexpr (TILED) {
    if (form == F32_TILE_64) return gemm_f32_tile<64, 128, 2, 2, 2, MODE>(A, lda, W, ldw, M, N, K, ea, st);
    if (form == F32_TILE_128) return gemm_f32_tile<128, 128, 2, 2, 2, MODE>(A, lda, W, ldw, M, N, K, ea, st);
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
