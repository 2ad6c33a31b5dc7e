// bf16 GEMM on the gfx950 matrix cores: C[m, n] = sum_k A[m, k] W[n, k], fp32
// accumulate, fused epilogue.  Both operands are k-contiguous, so a lane's MFMA
// operand is one 16-byte LDS read.  The weights feed the MFMA row operand and the
// activations the column operand (v_mfma_f32_32x32x16_bf16).
//
// This file holds the choice of the kernel and the launches of the one-tile-per-workgroup kernel (gemm_tile.h);
// the persistent kernel for large problems is in gemm_bf16_stream.hip, the one for about one round of tiles in
// gemm_bf16_ring.hip, the one for small problems in gemm_small.hip.
#include <cmath>

#include "common.h"
#include "dispatch.h"
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
  constexpr bool LARGE = BM >= 128 && std::is_same<TOUT, bf16>::value;  // (smaller tiles are not chosen for outputs of that size)
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(tiles_m * tiles_n), dim3(WGM * WGN * 64), 0, st, A, lda, W, ldw, M, N, K, tiles_m, tiles_n, group_n, epi);
  };
  if (LARGE && rule::tile_output_streams((size_t)M * N * sizeof(TOUT))) go(gemm_tile_kernel<BM, BN, WGM, WGN, NST, MODE, TOUT, LARGE>);
  else go(gemm_tile_kernel<BM, BN, WGM, WGN, NST, MODE, TOUT, false>);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

enum {  // bits 0..3 of a variant; TILE_STREAM + 1 .. + 4: the persistent kernel with 4 .. 7 times 32 rows a tile
  TILE_32 = 0, TILE_128_W8 = 1, TILE_64 = 2, TILE_64_128 = 3, TILE_256 = 4, TILE_128 = 5, TILE_RING = 6, TILE_STREAM = 7
};

// The kernel for a problem size.  r = tiles of a kind per compute unit.  (The part for small problems is from 410
// measured shapes: M 40 to 200 000, hidden sizes 64 to 3072 with their QKV, MLP and projection widths.)
// rps: rows of a sample where the epilogue looks something up per sample, else 0.  *height: rows of a tile of the
// persistent kernel, in units of 32, or of the ring kernel, in units of 16.
static int choose_tile(int M, int N, int K, int rps, bool stream_ok, bool ring_ok, int* height) {
  const double cu = device_cu_count();
  const double r32 = (double)cdiv(M, 32) * cdiv(N, 32) / cu, r64 = (double)cdiv(M, 64) * cdiv(N, 64) / cu;
  const double r128 = (double)cdiv(M, 128) * cdiv(N, 128) / cu;
  // Up to a few 32x32 tiles a unit: four waves a tile.  279 x 128 x 512 takes 3.2 us instead of the 5.3 of 64x64
  // tiles, 300 x 1024 x 4096 10.4 instead of 23.  A long K makes the tile's operand traffic (twice that of 64x64 tiles
  // for the same outputs) the longer part sooner.
  // Beyond, the ring kernel, as long as its tiles are one round in some height: the lowest such, which spreads them over most units.
  // From two rounds on its 128 columns cost operand traffic (4404 x 3072 x 1024: 28 us in the persistent kernel, 33).  Samples
  // shorter than a wave's rows are left to the others.
  // A K below 768 hardly fills its stages and leaves its 5 us of launch, first stages and epilogue in sight, where smaller tiles come two
  // to a unit (1638 x 2048 x 256: 5.8 us in 64x128 tiles, 7.2 in 128 rows of the ring; 1400 x 2304 x 576: 9.3, 10.2).  It wins there
  // where those tiles are a little more than a round, so that some units have two and others one: 96 rows against 64x128 tiles (4404 x
  // 512 x 512: 10.1 us, 8.9 in the ring), 160 and 192 against 128x128 and the persistent kernel (2202 x 2048 x 512: 12.4,
  // 10.1; plain outputs with a K that the persistent kernel does not take stay with 128x128: 8831 x 640 x 192 9.8, 11.1).
  // 64x64 tiles stay where they make one round and the ring needs 64 rows for it, half of its last columns being empty
  // (4424 x 192 x 1536: 10.5 us, 11.1).
  // 732 shapes (M 64 to 49 000, N 64 to 6144, K 64 to 4096): 5 % faster on average than the rules below alone, 2 % slower than the best
  // kernel of each, at most 4 % slower than without the ring (1101 x 3072 x 1024: 14.6 -> 11.0 us, 1101 x 2048 x 8192: 69 -> 46).
  int ring = 0;
  for (int h = 2; ring_ok && h <= 12 && !ring; h += 2)
    if ((double)cdiv(M, 16 * h) * cdiv(N, 128) <= cu && (rps == 0 || rps >= 8 * h)) ring = h;
  if (K < 768 && !(N >= 128 && ((ring == 6 && K >= 384) || (ring >= 10 && (stream_ok || rps > 0))))) ring = 0;
  if (r32 <= (ring && K >= 768 ? (K < 1024 ? 3.0 : K == 1024 ? 2.5 : 2.0) : (K < 1024 ? 4.0 : 3.0))) return TILE_32;
  if (ring && !(ring >= 4 && r64 <= 1.0)) {
    *height = ring;
    return TILE_RING;
  }
  // What the ring kernel leaves: patch and unpatch products, gated residuals of short samples, short K.
  // Up to one round of 64x64 tiles: two waves each, four stages of 16 KB in flight.  1101 x 1024 x 4096: 23 us
  // (34 in 128x128 tiles).
  if (r64 <= 1.2) return TILE_64;
  // Up to one round of 128x128 tiles: half of them, two to a unit (1710 x 2304 x 384: 7.9 us, 9.3 and 8.2 in 128x128 tiles of four and eight waves).
  if (r128 <= 1.0) return TILE_64_128;
  // Beyond: the persistent kernel, whose tiles are 128 to 256 rows high so that the last round of tiles is full
  // (9216 x 3072 x 12 288: 545 us in 432 tiles of 256 rows, 1.7 rounds, 490 in 504 of 224; 17 616 x 1024 x 1024: 67 us
  // in 256 rows, 50 in 160), or 128x128 tiles with two workgroups a unit where those fit better.  The costs are in
  // 32 x 256 x K blocks a unit: a tile costs three quarters of a block beyond its rows (epilogue, operands of W), a
  // part of a round 0.6 of what it leaves idle (the units that work run faster at the chip's power limit); 128x128
  // tiles move twice the operand bytes.  Fitted to 124 shapes (M 500 to 100 000, N 256 to 12 288, K 256 to 12 288):
  // 0.5 % slower on average than the best kernel of each shape.
  //
  // A wave of the persistent kernel owns 16 rows per unit of height.  Where those span more than two samples, every
  // row looks its sample up by itself, with nothing fetched ahead: 4 us a block, as much as the products of K = 900
  // (59 613 rows of 93 a sample, 1536 x 1536: 324 us in 160 rows, 505 in 192; 10 960 rows of 20, 512 x 512: 24.5 us in the
  // persistent kernel, 17.1 in 128x128 tiles of eight waves, whose waves own 32 rows).  83 shapes with samples of 20 to
  // 4608 rows: 1.2 % slower on average than the best kernel of each; without this term 5.8 % on the short ones.
  double best = 1.4 * 2.0 * (r128 + 0.4);
  // eight waves store faster (3-5 %), which a short K leaves a larger share to, and own half the rows each
  int tile = K <= 512 || (rps > 0 && rps < 64) ? TILE_128_W8 : TILE_128;
  for (int h = 8; h >= 4; --h) {
    if (!stream_ok && h < 8) break;
    const double r = (double)cdiv(M, 32 * h) * cdiv(N, 256) / cu;
    const double lookups = rps > 0 && rps < 16 * h ? 900.0 / K * h : 0.0;
    const double cost = (0.4 * r + 0.6 * std::ceil(r)) * (h + 0.75 + lookups);
    if (cost < best) {
      best = cost;
      tile = stream_ok ? TILE_STREAM : TILE_256;
      *height = h;
    }
  }
  return tile;
}

// variant bits 0..3: kernel (see the enum); bits 4..11: column-group width of the tile walk (0 = the kernel's own
// choice); for the persistent kernel bits 24..30: row block of the walk in units of 8 tile rows (bits 12..23 were start
// delays of an earlier form and are ignored), for TILE_RING its tile height.  variant < 0 = choose by problem size.
template <int MODE, typename TOUT>
static br_status gemm_variant(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                              int variant, hipStream_t st) {
  int tile, group_n = 0, row_block = 0, height = 0;
  if (variant < 0) {
    tile = choose_tile(M, N, K, MODE == EPI_BIAS_GATE_RES ? ea.L : 0, gemm_stream_supported(MODE, K, (size_t)M * lda * 2, (size_t)N * ldw * 2),
                       gemm_ring_supported(MODE, 12, lda, ldw), &height);
  } else {
    tile = variant & 15;
    group_n = (variant >> 4) & 255;
    height = 8;
    if (tile == TILE_RING) {
      height = (variant >> 24) & 127;
      if (!gemm_ring_supported(MODE, height, lda, ldw)) tile = TILE_128;  // (6 alone: 256x128 tiles in earlier versions)
    }
    if (tile > TILE_STREAM && tile <= TILE_STREAM + 4) {
      height = tile - TILE_STREAM + 3;
      tile = TILE_STREAM;
    }
    row_block = ((variant >> 24) & 127) * 8;
  }
  ProfScope ps(st, PROF_GEMM + MODE * 8 + tile, 2.0 * M * N * K);
  switch (tile) {
    case TILE_32: return launch_gemm_small(BR_BF16, MODE, A, lda, W, ldw, M, N, K, ea, st);
    case TILE_128_W8: return gemm_tile_launch<128, 128, 4, 2, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_64: return gemm_tile_launch<64, 64, 2, 1, 4, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_64_128: return gemm_tile_launch<64, 128, 2, 2, 3, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_256: return gemm_tile_launch<256, 256, 2, 4, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_128: return gemm_tile_launch<128, 128, 2, 2, 2, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case TILE_RING: return launch_gemm_bf16_ring(MODE, A, lda, W, ldw, M, N, K, ea, height, group_n, st);
    case TILE_STREAM: return launch_gemm_bf16_stream(MODE, A, lda, W, ldw, M, N, K, ea, height, group_n, row_block, st);
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
