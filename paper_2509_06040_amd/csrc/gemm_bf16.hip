// bf16 GEMM on the gfx950 matrix cores: C[m, n] = sum_k A[m, k] W[n, k], fp32
// accumulate, fused epilogue.  Both operands are k-contiguous, so a lane's MFMA
// operand is one 16-byte LDS read.  The weights feed the MFMA row operand and the
// activations the column operand (v_mfma_f32_32x32x16_bf16).
//
// This file holds the choice of the kernel and the launches of the one-tile-per-workgroup kernel (gemm_tile.h);
// the persistent kernel for large problems is in gemm_bf16_stream.hip, the one for small ones in
// gemm_ksplit.hip.
#include <cmath>

#include "common.h"
#include "dit.h"
#include "gemm_tile.h"
#include "prof.h"

namespace br {

template <int BM, int BN, int WGM, int WGN, int NST, int MODE, typename TOUT>
static br_status gemm_tile_launch(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                                 int group_n, hipStream_t st) {
  Epilogue<MODE, TOUT> epi{ea};
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  // Columns in even groups of at most 8: the tiles a compute die works on at once then share both operands.
  if (group_n <= 0 || group_n > tiles_n) group_n = cdiv(tiles_n, cdiv(tiles_n, 8));
  hipLaunchKernelGGL((gemm_tile_kernel<bf16, BM, BN, WGM, WGN, NST, MODE, TOUT>), dim3(tiles_m * tiles_n), dim3(WGM * WGN * 64),
                     0, st, A, lda, W, ldw, M, N, K, tiles_m, tiles_n, group_n, epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

enum {  // bits 0..3 of a variant
  TILE_KSPLIT = 0, TILE_128_W8 = 1, TILE_64 = 2, TILE_64_128 = 3, TILE_256 = 4, TILE_128 = 5, TILE_256_128 = 6, TILE_STREAM = 7
};

// The kernel for a problem size, from 410 measured shapes (M 40 to 200 000, hidden sizes 64 to 3072 with
// their QKV, MLP and projection widths, K 64 to 12 288); it is 2 % slower on average than the best kernel
// of each shape.  r = tiles of a kind per compute unit.
static int choose_tile(int M, int N, int K, bool stream_ok) {
  const double cu = device_cu_count();
  const double r32 = (double)cdiv(M, 32) * cdiv(N, 32) / cu, r64 = (double)cdiv(M, 64) * cdiv(N, 64) / cu;
  const double r128 = (double)cdiv(M, 128) * cdiv(N, 128) / cu, r256 = (double)cdiv(M, 256) * cdiv(N, 256) / cu;
  // Up to a few 32x32 tiles a unit: the waves of a tile split K.  279 x 128 x 512 takes 3.3 us instead of
  // the 5.6 of 64x64 tiles and the 10.7 of the 256x128 tiles used before.  A long K makes the tile's operand
  // traffic (twice that of 64x64 tiles for the same outputs) the longer part sooner.
  if (r32 <= (K < 1024 ? 4.0 : 3.0)) return TILE_KSPLIT;
  // Up to one round of 64x64 tiles: two waves each, four stages of 16 KB in flight.  1101 x 1024 x 4096: 23 us
  // (34 in 128x128 tiles, 52 in 256x128).
  if (r64 <= 1.2) return TILE_64;
  // Up to one round of 128x128 tiles: half of them, so that the round is fuller (1101 x 3072 x 1024: 14.7 us,
  // 20.8 in 256x128 tiles).
  if (r128 <= 1.0) return TILE_64_128;
  // Beyond: 128x128 tiles, two workgroups a unit, or 256x256 tiles (one persistent workgroup a unit; one tile
  // per workgroup where K is not a multiple of 128), which move half the operand bytes but finish in whole rounds:
  // 13 700 x 1088 x 4352 (1.05 rounds) 135 us against 211, 39 300 x 2752 x 11 008 (6.6 rounds) 2510 against 2180.
  // A partial round costs the small tiles less than a third of one.
  const double used = (double)M * N;
  const double e256 = 1.2 * r256 / std::ceil(r256) * used / ((double)cdiv(M, 256) * 256 * cdiv(N, 256) * 256);
  const double e128 = r128 / (r128 + 0.3) * used / ((double)cdiv(M, 128) * 128 * cdiv(N, 128) * 128);
  if (e256 > e128) return stream_ok ? TILE_STREAM : TILE_256;
  return K <= 512 ? TILE_128_W8 : TILE_128;  // a short K leaves a larger share to the epilogue, where eight waves store faster (3-5 %)
}

// variant bits 0..3: kernel (see the enum); bits 4..11: column-group width of the tile walk (0 = the
// kernel's own choice); variant < 0 = choose by problem size.
template <int MODE, typename TOUT>
static br_status gemm_variant(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                              int variant, hipStream_t st) {
  int tile, group_n = 0, row_block = 0, stagger_slack = 0, stagger_crit = 0;
  if (variant < 0) {
    tile = choose_tile(M, N, K, gemm_stream_supported(M, N, K, (size_t)M * lda * 2, (size_t)N * ldw * 2));
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
    case TILE_KSPLIT: return launch_gemm_ksplit(BR_BF16, MODE, A, lda, W, ldw, M, N, K, ea, st);
    case TILE_128_W8: return gemm_tile_launch<128, 128, 4, 2, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_64: return gemm_tile_launch<64, 64, 2, 1, 4, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_64_128: return gemm_tile_launch<64, 128, 2, 2, 3, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_256: return gemm_tile_launch<256, 256, 2, 4, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_128: return gemm_tile_launch<128, 128, 2, 2, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_256_128: return gemm_tile_launch<256, 128, 4, 2, 3, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_STREAM: return launch_gemm_bf16_stream(MODE, A, lda, W, ldw, M, N, K, ea, group_n, row_block, stagger_slack, stagger_crit, st);
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
