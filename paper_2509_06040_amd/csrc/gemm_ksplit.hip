// GEMM for problems that do not fill the chip with large tiles, and for fp32: C[m, n] =
// sum_k A[m, k] W[n, k] with the fused epilogues.  One workgroup per output tile; its waves split
// K between them instead of splitting the tile, so a tile of a few rows and columns still keeps four
// to eight waves busy and a long K is walked by all of them at once.
//
// A wave owns every NW-th stage of K (128 bytes of every row of the tile: 64 bf16 or 32 fp32
// values).  It fetches its own stages (global -> LDS directly) into its own slots of LDS, reads the
// operand fragments into registers, refills the slot and multiplies: the main loop has no barrier,
// and the waves run as far apart as their loads arrive.  The partial tiles are added in LDS, in a
// fixed order, and leave through the row-wise form of the epilogue.
//
// fp32 runs on the matrix cores as well (v_mfma_f32_32x32x2_f32: full fp32 products and sums at twice
// the vector rate): a lane's 16-byte chunk holds 4 consecutive k instead of 8, and the four
// instructions of a chunk pair take element e of both halves, k = e and 4 + e.
#include <type_traits>

#include "common.h"
#include "dit.h"
#include "gemm_frag.h"
#include "prof.h"

namespace br {

typedef float f32x4 __attribute__((ext_vector_type(4)));

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

template <typename T, int TM, int TN, int NW, int NST>
__shared__ __attribute__((aligned(1024))) char g_kslots[NW * NST * (TM + TN) * 32 * 128];

// Tile of 32 TM rows x 32 TN columns, NW waves, NST slots of one stage each per wave.
template <typename T, int TM, int TN, int NW, int NST, int MODE, typename TOUT>
__global__ __launch_bounds__(NW * 64) void gemm_ksplit_kernel(const T* __restrict__ A, int lda, const T* __restrict__ W,
                                                              int ldw, int M, int N, int K, int tiles_m, int tiles_n,
                                                              Epilogue<MODE, TOUT> epi) {
  constexpr int BM = TM * 32, BN = TN * 32, SLOT = (BM + BN) * 128;
  constexpr int IA = BM / 8, IW = BN / 8, LPT = IA + IW;  // loads of a stage, 8 rows of 128 bytes each
  constexpr int ES = (int)sizeof(T);
  static_assert(NST * LPT <= 48, "the wait counts below must fit the hardware counter");
  static_assert(NW * BM * BN * 4 <= NW * NST * SLOT, "the partial tiles reuse the slots");
  typedef typename GemmFrag<T>::type frag;

  // tiles of one compute die are consecutive: it shares the weight rows of a column panel
  int wg = blockIdx.x;
  {
    const int nwg = tiles_m * tiles_n, per = nwg / 8, rem = nwg % 8, x = wg % 8, i = wg / 8;
    wg = x * per + (x < rem ? x : rem) + i;
  }
  const int tile_n = wg / tiles_m, tile_m = wg - tile_n * tiles_m;
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lh = lane >> 5;

  // Chunk c (16 bytes) of row r sits in slot c ^ ((r >> 1) & 7) of its row; a load fills 8 rows
  // (lane = 8 * row + slot), so the permutation is applied to the address a lane fetches from.
  const int ld_row = lane >> 3;
  unsigned off_a[IA], off_w[IW];  // bytes from the tile's first row
  unsigned chunk_b[2];            // this lane's chunk offset in even and odd 8-row blocks
#pragma unroll
  for (int par = 0; par < 2; ++par) chunk_b[par] = ((lane & 7) ^ ((ld_row >> 1) | (4 * par))) * 16;
#pragma unroll
  for (int j = 0; j < IA; ++j) off_a[j] = (unsigned)min(j * 8 + ld_row, M - 1 - m0) * (unsigned)lda * ES + chunk_b[j & 1];
#pragma unroll
  for (int j = 0; j < IW; ++j) off_w[j] = (unsigned)min(j * 8 + ld_row, N - 1 - n0) * (unsigned)ldw * ES + chunk_b[j & 1];
  const char* a_tile = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
  const char* w_tile = reinterpret_cast<const char*>(W + (size_t)n0 * ldw);
  const int kbytes = K * ES, nst = (kbytes + 127) >> 7;  // stages of the whole K
  char* slots = g_kslots<T, TM, TN, NW, NST> + wv * (NST * SLOT);

  auto issue = [&](int st, int slot) {
    const unsigned base = (unsigned)(uintptr_t)BR_LPTR(slots) + slot * SLOT;
    const char* ap = a_tile + (size_t)st * 128;
    const char* wp = w_tile + (size_t)st * 128;
    // chunks past the end of K (last stage only) are fetched from the stage's first chunk and dropped below
    const int left = kbytes - st * 128;
    unsigned back[2];
#pragma unroll
    for (int par = 0; par < 2; ++par) back[par] = (int)chunk_b[par] < left ? 0u : chunk_b[par];
#pragma unroll
    for (int j = 0; j < IA; ++j)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base + j * 1024), "v"(off_a[j] - back[j & 1]), "s"(ap) : "memory", "m0");
#pragma unroll
    for (int j = 0; j < IW; ++j)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base + (IA + j) * 1024), "v"(off_w[j] - back[j & 1]), "s"(wp) : "memory", "m0");
  };

  f32x16 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  int fo_a[TM], fo_w[TN];  // fragment byte offsets in a slot for chunk pair 0; pair p is the same offset ^ (p << 5)
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int row = j * 32 + l32;
    fo_a[j] = row * 128 + ((lh ^ ((row >> 1) & 7)) << 4);
  }
#pragma unroll
  for (int i = 0; i < TN; ++i) {
    const int row = i * 32 + l32;
    fo_w[i] = BM * 128 + row * 128 + ((lh ^ ((row >> 1) & 7)) << 4);
  }

  // One stage: it has landed once at most `younger` stages' loads are outstanding (loads retire in
  // order); all fragments go to registers, then the slot is free again.
  auto stage = [&](int st, auto Slot, int younger) {
    constexpr int slot = decltype(Slot)::value;
    if (NST > 1 && younger > 0)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * LPT) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const char* sl = slots + slot * SLOT;
    frag fa[4][TM], fw[4][TN];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
      for (int j = 0; j < TM; ++j) fa[p][j] = *reinterpret_cast<const frag*>(sl + (fo_a[j] ^ (p << 5)));
#pragma unroll
      for (int i = 0; i < TN; ++i) fw[p][i] = *reinterpret_cast<const frag*>(sl + (fo_w[i] ^ (p << 5)));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (st + NST * NW < nst) issue(st + NST * NW, slot);
    __builtin_amdgcn_sched_barrier(0);
    if (ES == 4 && kbytes - st * 128 < 128) {  // K ends inside this stage
      const int left = kbytes - st * 128;
      const frag zero = {};
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if ((p * 2 + lh) * 16 >= left) {
#pragma unroll
          for (int j = 0; j < TM; ++j) fa[p][j] = zero;
#pragma unroll
          for (int i = 0; i < TN; ++i) fw[p][i] = zero;
        }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int e = 0; e < GemmFrag<T>::STEPS; ++e)
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j) acc[i][j] = GemmFrag<T>::mma(fw[p][i], fa[p][j], acc[i][j], e);
  };
#pragma unroll
  for (int s = 0; s < NST; ++s)
    if (wv + s * NW < nst) issue(wv + s * NW, s);
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, NST - 1>;
  for (int st = wv; st < nst; st += NST * NW) {
    stage(st, S0{}, NST > 1 && st + NW < nst);
    if (NST > 1 && st + NW < nst) stage(st + NW, S1{}, st + 2 * NW < nst);
  }
  static_assert(NST <= 2, "the loop above is written for one or two slots");

  // ---- partial tiles to LDS (rows of BN floats, 16-byte chunks permuted per row), one area per wave
  constexpr int NC = BN / 4;                       // chunks of a row
  constexpr int RMASK = NC >= 16 ? 15 : NC - 1;
  __syncthreads();                                 // every wave is done with its slots
  char* area = g_kslots<T, TM, TN, NW, NST>;
#pragma unroll
  for (int j = 0; j < TM; ++j) {
    const int row = j * 32 + l32;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int c = i * 8 + g * 2 + lh;
        const f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        *reinterpret_cast<f32x4*>(area + wv * (BM * BN * 4) + row * (BN * 4) + ((c ^ (row & RMASK)) << 4)) = v;
      }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < BM * NC; q += NW * 64) {
    const int e = q + tid;
    if (BM * NC % (NW * 64) != 0 && e >= BM * NC) break;
    const int row = e / NC, c = e % NC;
    const char* p = area + row * (BN * 4) + ((c ^ (row & RMASK)) << 4);
    f32x4 v = *reinterpret_cast<const f32x4*>(p);
#pragma unroll
    for (int w = 1; w < NW; ++w) v += *reinterpret_cast<const f32x4*>(p + w * (BM * BN * 4));
    const int m = m0 + row, n = n0 + c * 4;
    if (m < M && n < N) epi.store(epi.row(m), n, v[0], v[1], v[2], v[3]);
  }
}

template <typename T, int TM, int TN, int NW, int NST, int MODE, typename TOUT>
static br_status ksplit_launch(const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               hipStream_t st) {
  Epilogue<MODE, TOUT> epi{ea};
  const int tiles_m = cdiv(M, TM * 32), tiles_n = cdiv(N, TN * 32);
  hipLaunchKernelGGL((gemm_ksplit_kernel<T, TM, TN, NW, NST, MODE, TOUT>), dim3(tiles_m * tiles_n), dim3(NW * 64), 0, st,
                     A, lda, W, ldw, M, N, K, tiles_m, tiles_n, epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

template <typename T, int MODE, typename TOUT>
static br_status ksplit_variant(const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                                int tile, hipStream_t st) {
  if (tile == 32) return ksplit_launch<T, 1, 1, 4, 1, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, st);
  return fail(BR_EINVAL, "k-split gemm: unknown tile");
}

template <typename T, typename TACT>
static br_status ksplit_mode(int mode, const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                             int tile, hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return ksplit_variant<T, EPI_BIAS, TACT>(A, lda, W, ldw, M, N, K, ea, tile, st);
    case EPI_BIAS_GELU: return ksplit_variant<T, EPI_BIAS_GELU, TACT>(A, lda, W, ldw, M, N, K, ea, tile, st);
    case EPI_BIAS_GATE_RES: return ksplit_variant<T, EPI_BIAS_GATE_RES, float>(A, lda, W, ldw, M, N, K, ea, tile, st);
    case EPI_PATCH_EMBED: return ksplit_variant<T, EPI_PATCH_EMBED, float>(A, lda, W, ldw, M, N, K, ea, tile, st);
    case EPI_BIAS_F32: return ksplit_variant<T, EPI_BIAS_F32, float>(A, lda, W, ldw, M, N, K, ea, tile, st);
    case EPI_UNPATCH: return ksplit_variant<T, EPI_UNPATCH, float>(A, lda, W, ldw, M, N, K, ea, tile, st);
  }
  return fail(BR_EINVAL, "gemm: unknown epilogue");
}

br_status launch_gemm_ksplit(int dtype, int mode, const void* A, int lda, const void* W, int ldw, int M, int N, int K,
                             const EpiArgs& ea, int tile, hipStream_t st) {
  if (dtype == BR_BF16)
    return ksplit_mode<bf16, bf16>(mode, (const bf16*)A, lda, (const bf16*)W, ldw, M, N, K, ea, tile, st);
  return ksplit_mode<float, float>(mode, (const float*)A, lda, (const float*)W, ldw, M, N, K, ea, tile, st);
}

}  // namespace br
