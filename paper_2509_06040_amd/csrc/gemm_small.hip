// GEMM for problems that do not fill the chip with large tiles: C[m, n] = sum_k A[m, k] W[n, k] with the fused epilogues.
// One workgroup per 32x32 tile, a 16x16 quarter of it per wave.
//
// Every output is one chain over k, in the order of the larger kernels (gemm_frag.h): a sample's result does not depend on
// how many others share its launch.  (An earlier form let the waves split K and added four partial sums.)  The chain of
// matrix instructions takes no longer than that did: a wave has the whole of K in instructions of a quarter of the size.  What
// bounds it is the latency of the operands, so they are fetched (global -> LDS directly) in a ring of stages of
// 128 bytes of every row, all but one step in flight, one barrier a step.
//
// fp32 runs on the matrix cores as well (v_mfma_f32_16x16x4_f32: a chain of fused multiply-adds over its four k).
#include <type_traits>

#include "common.h"
#include "dit.h"
#include "gemm_frag.h"
#include "prof.h"

namespace br {

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

namespace {
constexpr int BM = 32, BN = 32, NW = 4;  // tile, waves
}  // namespace
extern __shared__ __attribute__((aligned(1024))) char g_krows[];  // LN: the tile's rows of A, stage by stage

// LN-modulated rows of the residual stream as the A operand: eight lanes of the workgroup take a row of the tile each,
// keep it in registers (K <= 1024 / sizeof(T)) and leave it in LDS in the layout of the stages.  Every column tile does it
// again for its rows (from cache).  Sums over eight lanes cost three exchanges; a wave per row, as in ln_modulate_kernel,
// would pass eight rows through six, which takes longer than the launch that is saved.  The sums are those of that
// kernel all the same: a lane holds what eight of its lanes do (sub, sub + 8, ...), and adds them up in its exchanges' order.
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
  // p[j] = sum of lane sub + 8 j there
  auto row_sum = [](const float (&p)[8]) {
    float s = ((p[0] + p[4]) + (p[2] + p[6])) + ((p[1] + p[5]) + (p[3] + p[7]));  // (distances 32, 16, 8)
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    return s;
  };
  float p[8] = {};
#pragma unroll
  for (int i = 0; i < V; ++i) p[i & 7] += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  const float mean = row_sum(p) / (float)K;
  float p2[8] = {};
#pragma unroll
  for (int i = 0; i < V; ++i)
    if (sub + 8 * i < H4) p2[i & 7] += sum_sq4(v[i], mean);
  const float q = row_sum(p2);
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

template <typename T, int MODE, typename TOUT, bool LN, int SPS, int NSLOT>
__global__ __launch_bounds__(NW * 64) void gemm_small_kernel(const T* __restrict__ A, int lda, const T* __restrict__ W,
                                                             int ldw, int M, int N, int K, int tiles_m, int tiles_n,
                                                             Epilogue<MODE, TOUT> epi, LnArgs ln) {
  constexpr int ES = (int)sizeof(T), NF = GemmFrag16<T>::COUNT;  // fragments of a stage
  constexpr int STAGE = (LN ? BN : BM + BN) * 128, OFF_W = LN ? 0 : BM * 128;  // bytes
  constexpr int LPS = SPS * (LN ? 1 : 2);                        // loads of a wave and step
  typedef typename GemmFrag16<T>::type frag;
  static_assert(BM == 8 * NW && BN == 8 * NW, "a load covers 8 rows, every wave has one of A and one of W");
  static_assert(NSLOT == 2 || NSLOT == 3, "ring depth");
  __shared__ __attribute__((aligned(1024))) char ring[NSLOT * SPS * STAGE];

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
  const int l16 = lane & 15, lq = lane >> 4;

  // Chunk c (16 bytes) of row r sits in slot c ^ ((r >> 1) & 7) of its row; a load fills 8 rows (lane = 8 * row + slot),
  // so the permutation is applied to the address a lane fetches from.
  const int ld_row = wv * 8 + (lane >> 3);
  const unsigned chunk_b = ((lane & 7) ^ ((ld_row >> 1) & 7)) * 16;
  const unsigned off_a = (unsigned)min(ld_row, M - 1 - m0) * (unsigned)lda * ES + chunk_b;  // bytes from the tile's first row
  const unsigned off_w = (unsigned)min(ld_row, N - 1 - n0) * (unsigned)ldw * ES + chunk_b;
  const char* a_tile = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
  const char* w_tile = reinterpret_cast<const char*>(W + (size_t)n0 * ldw);
  const int kbytes = K * ES, nst = (kbytes + 127) >> 7, nstep = (nst + SPS - 1) / SPS;  // stages and steps of the whole K

  auto issue = [&](int step, int slot) {
#pragma unroll
    for (int u = 0; u < SPS; ++u) {
      const int st = min(step * SPS + u, nst - 1);  // (stages past the end of K: the last once more, read by nobody)
      const unsigned base = (unsigned)(uintptr_t)BR_LPTR(ring) + (slot * SPS + u) * STAGE + wv * 1024;
      // chunks past the end of K (last stage only) are fetched from the stage's first chunk and dropped below
      const unsigned back = (int)chunk_b < kbytes - st * 128 ? 0u : chunk_b;
      if (!LN)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base), "v"(off_a - back), "s"(a_tile + (size_t)st * 128) : "memory", "m0");
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base + OFF_W), "v"(off_w - back), "s"(w_tile + (size_t)st * 128) : "memory", "m0");
    }
  };
  // At most the loads of `younger` steps are outstanding (loads retire in order), all LDS reads have arrived.  (The latter as
  // a builtin: the compiler then knows, and has no waits of its own in front of the matrix instructions.)
  auto wait = [&](int younger) {
    if (NSLOT > 2 && younger >= 1)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPS) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  };

  // byte offsets of this lane's first fragments in a stage; fragment i is at the same ^ i * FLIP
  const int fo_a = GemmFrag16<T>::offset((wv & 1) * 16 + l16, lq), fo_w = OFF_W + GemmFrag16<T>::offset((wv >> 1) * 16 + l16, lq);
  frag fa[2][SPS][NF], fw[2][SPS][NF];
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  // One step: its stages have landed for every wave and those of the step before are in registers of every wave, so that their
  // slot is refilled; the fragments of this step are read in between the matrix instructions of the step before.
  int ring_slot = 0;
  auto step = [&](auto S, auto FIRST, int t) {
    constexpr int s = decltype(S)::value;  // t % 2
    const int slot = NSLOT == 2 ? s : ring_slot;
    wait(min(NSLOT - 2, nstep - 1 - t));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (t + NSLOT - 1 < nstep) issue(t + NSLOT - 1, slot == 0 ? NSLOT - 1 : slot - 1);
#pragma unroll
    for (int u = 0; u < SPS; ++u) {
      const char* stage = ring + (slot * SPS + u) * STAGE;
      const char* rows = LN ? g_krows + min(t * SPS + u, nst - 1) * (BM * 128) : stage;
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        fa[s][u][i] = *reinterpret_cast<const frag*>(rows + (fo_a ^ (i * GemmFrag16<T>::FLIP)));
        fw[s][u][i] = *reinterpret_cast<const frag*>(stage + (fo_w ^ (i * GemmFrag16<T>::FLIP)));
        __builtin_amdgcn_sched_barrier(0);
        if (!decltype(FIRST)::value) acc = GemmFrag16<T>::mma(fw[s ^ 1][u][i], fa[s ^ 1][u][i], acc);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (NSLOT > 2) ring_slot = slot == NSLOT - 1 ? 0 : slot + 1;
  };
  auto last = [&](auto S) {
    constexpr int s = decltype(S)::value;
#pragma unroll
    for (int u = 0; u < SPS; ++u) {
      const int left = kbytes - ((nstep - 1) * SPS + u) * 128;
      if (ES == 2 ? left <= 0 : left < 128) {
        // the end of K (fp32: also inside a stage, a fragment is one chunk)
#pragma unroll
        for (int i = 0; i < NF; ++i)
          if (ES == 4 && i * 16 < left) acc = GemmFrag16<T>::mma(fw[s][u][i], fa[s][u][i], acc);
        break;
      }
#pragma unroll
      for (int i = 0; i < NF; ++i) acc = GemmFrag16<T>::mma(fw[s][u][i], fa[s][u][i], acc);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  for (int t = 0; t < NSLOT - 1 && t < nstep; ++t) issue(t, t);
  if constexpr (LN) ln_rows<T>(ln, m0, M, K, tid);  // (visible to the other waves behind the first step's barrier)
  step(I0{}, std::true_type{}, 0);
  for (int t = 1;; t += 2) {
    if (t >= nstep) {
      last(I0{});
      break;
    }
    step(I1{}, std::false_type{}, t);
    if (t + 1 >= nstep) {
      last(I1{});
      break;
    }
    step(I0{}, std::false_type{}, t + 1);
  }
  const int m = m0 + (wv & 1) * 16 + l16, n = n0 + (wv >> 1) * 16 + lq * 4;
  if (m < M && n < N) epi.store(epi.row(m), n, acc[0], acc[1], acc[2], acc[3]);
}

template <typename T, int MODE, typename TOUT, bool LN, int SPS, int NSLOT>
static br_status small_launch_n(const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                                hipStream_t st, const LnArgs& ln) {
  Epilogue<MODE, TOUT> epi{ea};
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  const size_t rows = LN ? (size_t)BM * align_up((size_t)K * sizeof(T), 128) : 0;
  hipLaunchKernelGGL((gemm_small_kernel<T, MODE, TOUT, LN, SPS, NSLOT>), dim3(tiles_m * tiles_n), dim3(NW * 64), rows, st, A, lda, W,
                     ldw, M, N, K, tiles_m, tiles_n, epi, ln);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

// Stages of a step and steps of the ring.  A barrier and the read of a step's fragments cost about 400 cycles, so a long K is
// walked in steps of four stages where two workgroups of 64 KB are all that a compute unit gets (300 x 1024 x 4096: 9.8 us,
// 12.4 in steps of two; 1024 x 64 x 1024 in fp32: 7.9 against 8.6); else two, where more workgroups share a unit
// and a short K would fetch stages for nothing (24 x 64 x 64: 2.5 us, 3.0 in steps of four).  bf16 has a third step in
// flight (1101 x 1024 x 1024: 8.6 us against 9.2), whose products are too short to hide a step's latency; fp32 does not need it.
template <typename T, int MODE, typename TOUT, bool LN = false>
static br_status small_launch(const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                              hipStream_t st, const LnArgs& ln = LnArgs{}) {
  if constexpr (!LN) {
    if ((size_t)K * sizeof(T) >= 2048 && (long long)cdiv(M, BM) * cdiv(N, BN) <= 2LL * device_cu_count())
      return small_launch_n<T, MODE, TOUT, LN, 4, 2>(A, lda, W, ldw, M, N, K, ea, st, ln);
  }
  return small_launch_n<T, MODE, TOUT, LN, 2, (sizeof(T) == 2 ? 3 : 2)>(A, lda, W, ldw, M, N, K, ea, st, ln);
}

template <typename T, typename TACT>
static br_status small_mode(int mode, const T* A, int lda, const T* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                             hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return small_launch<T, EPI_BIAS, TACT>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_BIAS_GELU: return small_launch<T, EPI_BIAS_GELU, TACT>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_BIAS_GATE_RES: return small_launch<T, EPI_BIAS_GATE_RES, float>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_PATCH_EMBED: return small_launch<T, EPI_PATCH_EMBED, float>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_BIAS_F32: return small_launch<T, EPI_BIAS_F32, float>(A, lda, W, ldw, M, N, K, ea, st);
    case EPI_UNPATCH: return small_launch<T, EPI_UNPATCH, float>(A, lda, W, ldw, M, N, K, ea, st);
  }
  return fail(BR_EINVAL, "gemm: unknown epilogue");
}

br_status launch_gemm_small(int dtype, int mode, const void* A, int lda, const void* W, int ldw, int M, int N, int K,
                             const EpiArgs& ea, hipStream_t st) {
  if (dtype == BR_BF16)
    return small_mode<bf16, bf16>(mode, (const bf16*)A, lda, (const bf16*)W, ldw, M, N, K, ea, st);
  return small_mode<float, float>(mode, (const float*)A, lda, (const float*)W, ldw, M, N, K, ea, st);
}

// The normalised rows take at most 32 KB of LDS beside 16 or 24 KB of slots, i.e. K <= 256 in fp32 and 512 in bf16: three
// workgroups fit a compute unit, and a lane holds a row's eighth in registers.  Up to one workgroup a unit: beyond, what
// every column tile does again for itself takes longer than the launch.
bool ln_gemm_fits(int dtype, int M, int N, int K, const void* x, const void* mods, int A, int shift_off, int scale_off) {
  const size_t es = dtype == BR_BF16 ? 2 : 4;
  return (size_t)K * es <= 1024 && (K * es) % 16 == 0 && (long long)cdiv(M, BM) * cdiv(N, BN) <= device_cu_count() &&
         ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(mods)) & 15) == 0 && A % 4 == 0 && shift_off % 4 == 0 &&
         scale_off % 4 == 0;
}

template <typename T, typename TACT>
static br_status ln_mode(int mode, const LnArgs& ln, const T* W, int M, int N, int K, const EpiArgs& ea, hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return small_launch<T, EPI_BIAS, TACT, true>(W, K, W, K, M, N, K, ea, st, ln);
    case EPI_BIAS_GELU: return small_launch<T, EPI_BIAS_GELU, TACT, true>(W, K, W, K, M, N, K, ea, st, ln);
    case EPI_UNPATCH: return small_launch<T, EPI_UNPATCH, float, true>(W, K, W, K, M, N, K, ea, st, ln);
  }
  return fail(BR_EINVAL, "layer norm gemm: unknown epilogue");
}

br_status launch_ln_gemm(int dtype, int mode, const LnArgs& ln, const void* W, int M, int N, int K, const EpiArgs& ea,
                         hipStream_t st) {
  if (dtype == BR_BF16) {  // (only bf16 GEMMs are instrumented)
    ProfScope ps(st, PROF_GEMM + mode * 8, 2.0 * M * N * K);
    return ln_mode<bf16, bf16>(mode, ln, (const bf16*)W, M, N, K, ea, st);
  }
  return ln_mode<float, float>(mode, ln, (const float*)W, M, N, K, ea, st);
}

}  // namespace br
