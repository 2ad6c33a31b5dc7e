// GEMM for problems that do not fill the chip with large tiles, and for fp32: C[m, n] =
// sum_k A[m, k] W[n, k] with the fused epilogues.  One workgroup per output tile; its waves split
// K between them instead of splitting the tile, so a tile of 32 rows and columns still keeps four waves busy
// and a long K is walked by all of them at once.
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

namespace {
constexpr int BM = 32, BN = 32, NW = 4;           // tile, waves
constexpr int SLOT = (BM + BN) * 128;             // one stage of one wave
}  // namespace
__shared__ __attribute__((aligned(1024))) char g_kslots[NW * SLOT];

template <typename T, int MODE, typename TOUT>
__global__ __launch_bounds__(NW * 64) void gemm_ksplit_kernel(const T* __restrict__ A, int lda, const T* __restrict__ W,
                                                              int ldw, int M, int N, int K, int tiles_m, int tiles_n,
                                                              Epilogue<MODE, TOUT> epi) {
  constexpr int IA = BM / 8, IW = BN / 8;  // loads of a stage, 8 rows of 128 bytes each
  constexpr int ES = (int)sizeof(T);
  static_assert(NW * BM * BN * 4 <= NW * SLOT, "the partial tiles reuse the slots");
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
  char* slot = g_kslots + wv * SLOT;

  auto issue = [&](int st) {
    const unsigned base = (unsigned)(uintptr_t)BR_LPTR(slot);
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

  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  // fragment byte offsets in a slot for chunk pair 0; pair p is the same offset ^ (p << 5)
  const int fo_a = l32 * 128 + ((lh ^ ((l32 >> 1) & 7)) << 4), fo_w = BM * 128 + fo_a;

  if (wv < nst) issue(wv);
  for (int st = wv; st < nst; st += NW) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    frag fa[4], fw[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      fa[p] = *reinterpret_cast<const frag*>(slot + (fo_a ^ (p << 5)));
      fw[p] = *reinterpret_cast<const frag*>(slot + (fo_w ^ (p << 5)));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (st + NW < nst) issue(st + NW);  // the stage is in registers: its slot is free
    __builtin_amdgcn_sched_barrier(0);
    if (ES == 4 && kbytes - st * 128 < 128) {  // K ends inside this stage
      const int left = kbytes - st * 128;
      const frag zero = {};
#pragma unroll
      for (int p = 0; p < 4; ++p)
        if ((p * 2 + lh) * 16 >= left) {
          fa[p] = zero;
          fw[p] = zero;
        }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int e = 0; e < GemmFrag<T>::STEPS; ++e) acc = GemmFrag<T>::mma(fw[p], fa[p], acc, e);
  }

  // ---- partial tiles to LDS (rows of BN floats, 16-byte chunks permuted per row), one area per wave
  __syncthreads();  // every wave is done with its slot
  constexpr int PART = BM * BN * 4;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 v = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
    *reinterpret_cast<f32x4*>(g_kslots + wv * PART + l32 * (BN * 4) + (((2 * g + lh) ^ (l32 & 7)) << 4)) = v;
  }
  __syncthreads();
  static_assert(BM * BN / 4 == NW * 64, "one chunk of the tile per thread");
  const int row = tid / (BN / 4), c = tid % (BN / 4);
  const char* p = g_kslots + row * (BN * 4) + ((c ^ (row & 7)) << 4);
  f32x4 part[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) part[w] = *reinterpret_cast<const f32x4*>(p + w * PART);
  const f32x4 v = (part[0] + part[1]) + (part[2] + part[3]);
  const int m = m0 + row, n = n0 + c * 4;
  if (m < M && n < N) epi.store(epi.row(m), n, v[0], v[1], v[2], v[3]);
}

template <typename T, int MODE, typename TOUT>
static br_status ksplit_launch(const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               hipStream_t st) {
  Epilogue<MODE, TOUT> epi{ea};
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  hipLaunchKernelGGL((gemm_ksplit_kernel<T, MODE, TOUT>), dim3(tiles_m * tiles_n), dim3(NW * 64), 0, st, A, lda, W, ldw,
                     M, N, K, tiles_m, tiles_n, epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

template <typename T, typename TACT>
static br_status ksplit_mode(int mode, const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                             hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return ksplit_launch<T, EPI_BIAS, TACT>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_BIAS_GELU: return ksplit_launch<T, EPI_BIAS_GELU, TACT>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_BIAS_GATE_RES: return ksplit_launch<T, EPI_BIAS_GATE_RES, float>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_PATCH_EMBED: return ksplit_launch<T, EPI_PATCH_EMBED, float>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_BIAS_F32: return ksplit_launch<T, EPI_BIAS_F32, float>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_UNPATCH: return ksplit_launch<T, EPI_UNPATCH, float>(A, lda, W, ldw, M, N, K, ea, st);
  }
  return fail(BR_EINVAL, "gemm: unknown epilogue");
}

br_status launch_gemm_ksplit(int dtype, int mode, const void* A, int lda, const void* W, int ldw, int M, int N, int K,
                             const EpiArgs& ea, hipStream_t st) {
  if (dtype == BR_BF16)
    return ksplit_mode<bf16, bf16>(mode, (const bf16*)A, lda, (const bf16*)W, ldw, M, N, K, ea, st);
  return ksplit_mode<float, float>(mode, (const float*)A, lda, (const float*)W, ldw, M, N, K, ea, st);
}

}  // namespace br
