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
extern __shared__ __attribute__((aligned(1024))) char g_krows[];  // LN: the tile's rows of A, stage by stage

// LN-modulated rows of the residual stream as the A operand: eight lanes of the workgroup take a row of the tile each,
// keep it in registers (K <= 1024 / sizeof(T)) and leave it in LDS in the layout of the stages.  Every column tile does it
// again for its rows (from cache).  Sums over eight lanes cost three exchanges; a wave per row, as in ln_modulate_kernel,
// would pass eight rows through six, which takes longer than the launch that is saved.
template <typename T>
__device__ inline void ln_rows(const LnArgs& ln, int m0, int M, int K, int tid) {
  constexpr int V = 32 / (int)sizeof(T);  // float4 of a lane
  static_assert(NW * 64 == BM * 8, "eight lanes a row");
  const int row = tid >> 3, sub = tid & 7, H4 = K >> 2;
  const int m = min(m0 + row, M - 1), b = m / ln.rows_per_sample, tok = m - b * ln.rows_per_sample;
  const float4* xr = reinterpret_cast<const float4*>(ln.x + ((size_t)b * ln.L_in + tok) * K);
  const float* mrow = ln.mods + (size_t)ln.condmap[b] * ln.A;
  float4 v[V], sh[V], sc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const int c4 = sub + 8 * i;
    v[i] = sh[i] = sc[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (8 * i < H4 && c4 < H4) {
      v[i] = xr[c4];
      sh[i] = reinterpret_cast<const float4*>(mrow + ln.shift_off)[c4];
      sc[i] = reinterpret_cast<const float4*>(mrow + ln.scale_off)[c4];
    }
  }
  float s = 0.f, q = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  const float mean = s / (float)K;
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const float a = v[i].x - mean, bq = v[i].y - mean, c = v[i].z - mean, d = v[i].w - mean;
    if (sub + 8 * i < H4) q += (a * a + bq * bq) + (c * c + d * d);
  }
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
  const float rstd = 1.0f / __builtin_sqrtf(q / (float)K + 1e-6f);
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const int c4 = sub + 8 * i, byte = c4 * 4 * (int)sizeof(T);
    if (8 * i < H4 && c4 < H4)
      store4<T>(reinterpret_cast<T*>(g_krows + (byte >> 7) * (BM * 128) + row * 128 + ((((byte >> 4) & 7) ^ ((row >> 1) & 7)) << 4) + (byte & 15)),
                fmaf((v[i].x - mean) * rstd, 1.f + sc[i].x, sh[i].x), fmaf((v[i].y - mean) * rstd, 1.f + sc[i].y, sh[i].y),
                fmaf((v[i].z - mean) * rstd, 1.f + sc[i].z, sh[i].z), fmaf((v[i].w - mean) * rstd, 1.f + sc[i].w, sh[i].w));
  }
}

template <typename T, int MODE, typename TOUT, bool LN>
__global__ __launch_bounds__(NW * 64) void gemm_ksplit_kernel(const T* __restrict__ A, int lda, const T* __restrict__ W,
                                                              int ldw, int M, int N, int K, int tiles_m, int tiles_n,
                                                              Epilogue<MODE, TOUT> epi, LnArgs ln) {
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
    for (int j = 0; j < (LN ? 0 : IA); ++j)
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
  if constexpr (LN) {
    ln_rows<T>(ln, m0, M, K, tid);
    __syncthreads();
  }
  for (int st = wv; st < nst; st += NW) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    frag fa[4], fw[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      fa[p] = *reinterpret_cast<const frag*>((LN ? g_krows + st * (BM * 128) : slot) + (fo_a ^ (p << 5)));
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

template <typename T, int MODE, typename TOUT, bool LN = false>
static br_status ksplit_launch(const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               hipStream_t st, const LnArgs& ln = LnArgs{}) {
  Epilogue<MODE, TOUT> epi{ea};
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  const size_t rows = LN ? (size_t)BM * align_up((size_t)K * sizeof(T), 128) : 0;
  hipLaunchKernelGGL((gemm_ksplit_kernel<T, MODE, TOUT, LN>), dim3(tiles_m * tiles_n), dim3(NW * 64), rows, st, A, lda, W, ldw,
                     M, N, K, tiles_m, tiles_n, epi, ln);
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

// The normalised rows share the 64 KB of LDS with the slots: 32 KB of them, i.e. K <= 256 in fp32 and 512 in bf16.  Up
// to one workgroup a compute unit: beyond, what every column tile does again for itself takes longer than the launch.
bool ln_gemm_fits(int dtype, int M, int N, int K, const void* x, const void* mods, int A, int shift_off, int scale_off) {
  const size_t es = dtype == BR_BF16 ? 2 : 4;
  return (size_t)K * es <= 1024 && (K * es) % 16 == 0 && (long long)cdiv(M, BM) * cdiv(N, BN) <= device_cu_count() &&
         ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(mods)) & 15) == 0 && A % 4 == 0 && shift_off % 4 == 0 &&
         scale_off % 4 == 0;
}

template <typename T, typename TACT>
static br_status ln_mode(int mode, const LnArgs& ln, const T* W, int M, int N, int K, const EpiArgs& ea, hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return ksplit_launch<T, EPI_BIAS, TACT, true>(W, K, W, K, M, N, K, ea, st, ln);
    case EPI_BIAS_GELU: return ksplit_launch<T, EPI_BIAS_GELU, TACT, true>(W, K, W, K, M, N, K, ea, st, ln);
    case EPI_UNPATCH: return ksplit_launch<T, EPI_UNPATCH, float, true>(W, K, W, K, M, N, K, ea, st, ln);
  }
  return fail(BR_EINVAL, "layer norm gemm: unknown epilogue");
}

br_status launch_ln_gemm(int dtype, int mode, const LnArgs& ln, const void* W, int M, int N, int K, const EpiArgs& ea,
                         hipStream_t st) {
  ProfScope ps(st, PROF_GEMM + mode * 8, 2.0 * M * N * K);
  if (dtype == BR_BF16) return ln_mode<bf16, bf16>(mode, ln, (const bf16*)W, M, N, K, ea, st);
  return ln_mode<float, float>(mode, ln, (const float*)W, M, N, K, ea, st);
}

}  // namespace br
