// bf16 GEMM on the gfx950 matrix cores: C[m, n] = sum_k A[m, k] W[n, k], fp32
// accumulate, fused epilogue.  Both operands are k-contiguous, so a lane's MFMA
// operand is one 16-byte LDS read.  The weights feed the MFMA row operand and the
// activations the column operand (v_mfma_f32_32x32x16_bf16).
//
// This file holds the dispatch and the launches of the one-tile-per-workgroup kernel (gemm_tile.h: BM x BN
// tile, WGM x WGN wavefronts); the persistent kernel for large problems is in gemm_bf16_stream.hip.
#include <cmath>

#include "common.h"
#include "dit.h"
#include "gemm_tile.h"
#include "prof.h"

namespace br {

template <int BM, int BN, int WGM, int WGN, int MODE, typename TOUT>
static br_status gemm_dma_launch(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                                 int group_n, hipStream_t st) {
  Epilogue<MODE, TOUT> epi{ea};
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  if (group_n <= 0 || group_n > tiles_n) group_n = tiles_n;
  hipLaunchKernelGGL((gemm_tile_kernel<bf16, BM, BN, WGM, WGN, MODE, TOUT>), dim3(tiles_m * tiles_n), dim3(WGM * WGN * 64),
                     0, st, A, lda, W, ldw, M, N, K, tiles_m, tiles_n, group_n, epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

// variant bits 0..3: kernel, 4 / 5 / 6 = 256x256 / 128x128 / 256x128 tiles, one tile per workgroup, LDS-direct loads
// in a four-stage ring; 7 = persistent 256x256 kernel with a continuous operand stream (gemm_bf16_stream.hip);
// bits 4..11: column-group width of the tile walk (0 = all columns).  variant < 0 = choose by problem size.
template <int MODE, typename TOUT>
static br_status gemm_variant(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                              int variant, hipStream_t st) {
  int tile, group_n = 0, row_block = 0, stagger_slack = 0, stagger_crit = 0;
  if (variant < 0) {
    // Measured on MI355X.  With r = (256x256 tiles) / (compute units):
    // up to half a round of tiles, 256x128 tiles put twice as many units to work; up to one
    // round the persistent 256x256 kernel is best; beyond that it stays best unless the last
    // round would be mostly empty (r = 1.08 costs two rounds), where 128x128 tiles win.
    const int cu = device_cu_count();
    const long long tiles_m = cdiv(M, 256), tiles_n = cdiv(N, 256);
    const long long t256 = tiles_m * tiles_n;
    const double r = (double)t256 / (double)cu;
    const bool stream_ok = gemm_stream_supported(M, N, K, (size_t)M * lda * 2, (size_t)N * ldw * 2);
    // One or two whole rounds and a last one that fills at most half the units: the rows are independent,
    // so the matrix is cut in two launches, as many rows as make whole rounds for the persistent kernel and
    // the rest -- at most half a round -- for the 256x128 tiles, which take half a tile time.  With
    // per-sample epilogue operands the cut falls between two samples.  Measured on 1101-token samples:
    // 3-16 % at 16 samples (1.1 to 4.3 rounds), 2-7 % at 24 and 32.  From three whole rounds on it does not
    // pay: the few units of a sparse last round run faster than a full round's (64 samples, N = 1024,
    // 4.3 rounds: 1-4 % slower when cut).
    if (stream_ok && r > 1.0 && r < 3.0 && (MODE == EPI_BIAS || MODE == EPI_BIAS_GELU || MODE == EPI_BIAS_GATE_RES)) {
      const long long whole = t256 / cu;
      long long head_rows = (whole * cu / tiles_n) * 256;
      const int rps = MODE == EPI_BIAS_GATE_RES ? ea.L : 256;
      head_rows = head_rows / rps * rps;
      const long long tail_rows = M - head_rows;
      if (head_rows > 0 && tail_rows > 0 && cdiv(tail_rows, 256) * tiles_n * 2 <= cu &&
          cdiv(head_rows, 256) * tiles_n <= whole * cu) {
        EpiArgs tail = ea;
        tail.out = (char*)ea.out + (size_t)head_rows * ea.ldo * sizeof(TOUT);
        if (MODE == EPI_BIAS_GATE_RES) tail.condmap = ea.condmap + head_rows / rps;
        const int head_variant = 7 | ((MODE == EPI_BIAS_GATE_RES && K <= 2048) ? (6 << 12) : 0);  // (the start stagger below)
        const br_status head = gemm_variant<MODE, TOUT>(A, lda, W, ldw, (int)head_rows, N, K, ea, head_variant, st);
        if (head != BR_OK) return head;
        return gemm_variant<MODE, TOUT>(A + (size_t)head_rows * lda, lda, W, ldw, (int)tail_rows, N, K, tail, 6, st);
      }
    }
    if (r <= 0.5)
      tile = 6;
    else if (r > 1.0 && std::ceil(r) / r > 1.4)
      tile = 5;
    else
      tile = stream_ok ? 7 : 4;
    // The fp32 gated residual reads and writes 512 KB per tile; with a short k-loop (K <= 2048) these
    // bursts of a die's 32 workgroups, all in step, are a third of the launch.  Workgroups with one tile
    // less than the longest list start up to 7 x 3 us late, in groups of four, which costs the launch
    // nothing and spreads the bursts: measured 6 % (64 samples) to 14 % (32 samples) on the image
    // network's projection GEMM (1101-token samples, N = K = 1024), nothing on deeper k-loops.
    if (MODE == EPI_BIAS_GATE_RES && K <= 2048) stagger_slack = 300;
  } else {
    tile = variant & 15;
    group_n = (variant >> 4) & 255;
    stagger_slack = ((variant >> 12) & 255) * 50;  // half microseconds -> 10 ns ticks
    stagger_crit = ((variant >> 20) & 15) * 50;
    row_block = ((variant >> 24) & 127) * 8;
  }
  ProfScope ps(st, PROF_GEMM + MODE * 8 + tile, 2.0 * M * N * K);
  switch (tile) {
    case 4: return gemm_dma_launch<256, 256, 2, 4, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 5: return gemm_dma_launch<128, 128, 2, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 6: return gemm_dma_launch<256, 128, 4, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 7: return launch_gemm_bf16_stream(MODE, A, lda, W, ldw, M, N, K, ea, group_n, row_block, stagger_slack, stagger_crit, st);
  }
  return fail(BR_EINVAL, "gemm: unknown variant");
}

br_status launch_gemm_bf16(int mode, const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K,
                           const EpiArgs& ea, int variant, hipStream_t st) {
  BR_REQUIRE(K % 64 == 0 && K >= 64, BR_ESHAPE, "bf16 gemm: K must be a positive multiple of 64");
  BR_REQUIRE(lda % 8 == 0 && ldw % 8 == 0, BR_ESHAPE, "bf16 gemm: leading dimensions must be multiples of 8");
  switch (mode) {
    case EPI_BIAS: return gemm_variant<EPI_BIAS, bf16>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_BIAS_GELU: return gemm_variant<EPI_BIAS_GELU, bf16>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_BIAS_GATE_RES: return gemm_variant<EPI_BIAS_GATE_RES, float>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_PATCH_EMBED: return gemm_variant<EPI_PATCH_EMBED, float>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_BIAS_F32: return gemm_variant<EPI_BIAS_F32, float>(A, lda, W, ldw, M, N, K, ea, variant, st);
    case EPI_UNPATCH: return gemm_variant<EPI_UNPATCH, float>(A, lda, W, ldw, M, N, K, ea, variant, st);
  }
  return fail(BR_EINVAL, "gemm: unknown epilogue");
}

}  // namespace br
