// fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32): one tile of 16 RB rows x 64 CB columns per workgroup, four waves side by side
// along the columns, stages of 32 k (128 bytes of every row) in two LDS slots.
//
// What bounds it: the matrix pipe, 32 cycles an instruction, so what a size leaves of it is decided by how evenly its tiles fill the compute
// units.  A wave owns all rows of the tile and 16 CB of its columns, which costs fragment reads (one word each, few against 32 cycles) and
// makes any height in steps of 16 rows a tile: 4404 x 1024 x 4096 takes 281 us in 144 x 128 tiles (0.97 rounds), 356 in the 32x32 tiles and
// 373 in the 64x128 ones that this kernel replaced.  Reads and loads lie one by one between the products (in bursts: 311 us there); a second
// step read ahead, with a deeper ring, gained nothing and cost workgroups a unit (96 x 64 tiles of 4404 x 1024 x 1024: 74 -> 79 us).
// 32 768 x 4096 x 4096: 149 TFLOP/s (64x128 tiles of 32x32x2 instructions 145, the vendor library 151).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "dispatch.h"
#include "dit.h"
#include "gemm_frag.h"
#include "static_for.h"

namespace br {

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

namespace {
constexpr int NW = 4, NST = 2;  // waves; stages in LDS
}

extern __shared__ __attribute__((aligned(1024))) char g_f32_ring[];

template <int RB, int CB, int MODE>
__global__ __launch_bounds__(256, 2) void gemm_f32_ring_kernel(const float* __restrict__ A, int lda, const float* __restrict__ W, int ldw,
                                                               int M, int N, int K, int tiles_m, int tiles_n, int group_n,
                                                               Epilogue<MODE, float> epi) {
  typedef GemmFrag16<float> F;
  constexpr int BM = 16 * RB, BN = 64 * CB, STAGE = (BM + BN) * 128;
  constexpr int GA = BM / 8, GT = GA + BN / 8, LPW = (GT + NW - 1) / NW;  // groups of 8 rows; loads of a wave and stage
  static_assert(NST * STAGE <= 160 * 1024 && LPW < 64, "ring");
  int wg = blockIdx.x;
  {
    const int nwg = tiles_m * tiles_n, per = nwg / 8, rem = nwg % 8, x = wg % 8, i = wg / 8;
    wg = x * per + (x < rem ? x : rem) + i;
  }
  int tile_m, tile_n;
  {
    const int gsz = tiles_m * group_n, g = wg / gsz, idx = wg - g * gsz, gn = min(group_n, tiles_n - g * group_n);
    tile_m = idx / gn;
    tile_n = g * group_n + idx - tile_m * gn;
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn0 = wv * 16 * CB;

  unsigned off[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int g = min(wv * LPW + j, GT - 1), row = (g < GA ? g : g - GA) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    off[j] = g < GA ? (unsigned)min(row, M - 1 - m0) * (unsigned)lda * 4u + c * 16 : (unsigned)min(row, N - 1 - n0) * (unsigned)ldw * 4u + c * 16;
  }
  const char* a_tile = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
  const char* w_tile = reinterpret_cast<const char*>(W + (size_t)n0 * ldw);
  const unsigned ring0 = (unsigned)(uintptr_t)BR_LPTR(g_f32_ring);
  const int nk = K / 32;
  auto load = [&](int j, int kt, int slot) __attribute__((always_inline)) {
    const int g = min(wv * LPW + j, GT - 1);
    const char* src = scalar_ptr((g < GA ? a_tile : w_tile) + (size_t)kt * 128);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(ring0 + slot * STAGE + g * 1024), "v"(off[j]), "s"(src) : "memory", "m0");
  };
  auto wait = [&](int younger) __attribute__((always_inline)) {
    if (younger >= 1)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPW) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  };

  f32x4 acc[RB][CB];
#pragma unroll
  for (int j = 0; j < RB; ++j)
#pragma unroll
    for (int i = 0; i < CB; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float fa[2][RB], fw[2][CB];
  const int fo = F::offset(l16, lq), fwo = (BM + wn0) * 128;
  auto read = [&](int slot, int s, int r, int set) __attribute__((always_inline)) {
    const char* p = g_f32_ring + slot * STAGE + (fo ^ (s * F::FLIP));
    if (r < CB) fw[set][r] = *reinterpret_cast<const float*>(p + fwo + r * 2048);
    else fa[set][r - CB] = *reinterpret_cast<const float*>(p + (r - CB) * 2048);
  };
  // One step of 4 k (number s of its stage).  Between its products, one by one: the reads of the next step's fragments (step rs of slot
  // `from`) and loads first, first + 1, ... of stage kl.
  constexpr int NM = RB * CB, NR = RB + CB, SPAN = (NM * 3 + 3) / 4;
  auto step = [&](auto Sc, int from, auto RSc, auto FIRST, auto COUNT, int kl, int to) __attribute__((always_inline)) {
    constexpr int set = decltype(Sc)::value & 1, rs = decltype(RSc)::value, first = decltype(FIRST)::value, count = decltype(COUNT)::value;
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      const int j = n / CB, i = (j & 1) ? CB - 1 - n % CB : n % CB;
      acc[j][i] = F::mma(fw[set][i], fa[set][j], acc[j][i]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = (n * NR + SPAN - 1) / SPAN; r < ((n + 1) * NR + SPAN - 1) / SPAN && r < NR; ++r) read(from, rs, r, set ^ 1);
#pragma unroll
      for (int l = n * count / NM; l < (n + 1) * count / NM; ++l) load(first + l, kl, to);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // loads of a stage go out in the first LS steps of the stage behind the one whose slot they take
  constexpr int LS = LPW > NM ? 3 : 2, LQ = (LPW + LS - 1) / LS;

  for (int s = 0; s < NST && s < nk; ++s)
#pragma unroll
    for (int j = 0; j < LPW; ++j) load(j, s, s);
  wait(min(nk, NST) - 1);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int r = 0; r < NR; ++r) read(0, 0, r, 0);
  int slot = 0;
  auto stage = [&](int kt, auto LOADS) __attribute__((always_inline)) {
    constexpr bool loads = decltype(LOADS)::value;
    const int other = slot ^ 1;
    static_for<7>([&](auto S) __attribute__((always_inline)) {
      constexpr int s = decltype(S)::value, first = std::min(s * LQ, LPW), count = loads ? std::min(LPW, (s + 1) * LQ) - first : 0;
      step(S, slot, std::integral_constant<int, s + 1>{}, std::integral_constant<int, first>{}, std::integral_constant<int, count>{}, kt - 1 + NST, other);
    });
    // Stage kt + 1 has landed and the fragments of stage kt are in registers; behind the barrier for every wave.  (Behind the last stage an
    // old one is read once more, which nobody uses.)
    wait(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    step(std::integral_constant<int, 7>{}, other, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, 0, 0);
    slot = other;
  };
  stage(0, std::false_type{});
  int kt = 1;
  for (; kt - 1 + NST < nk; ++kt) stage(kt, std::true_type{});
  for (; kt < nk; ++kt) stage(kt, std::false_type{});

  // Epilogue in the accumulator layout: block (j, i) gives lane l columns 16 i + 4 (l >> 4) .. + 3 of row 16 j + (l & 15).
  const int nb = n0 + wn0 + lq * 4, rps = epi.rows_per_sample();
  if (rps > 0 && rps < BM) {  // rows of more than two samples
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      const int m = m0 + j * 16 + l16;
#pragma unroll
      for (int i = 0; i < CB; ++i)
        if (m < M && nb + i * 16 < N) epi.store(epi.row(m), nb + i * 16, acc[j][i][0], acc[j][i][1], acc[j][i][2], acc[j][i][3]);
    }
    return;
  }
  using Epi = Epilogue<MODE, float>;
  int lo0 = 0, lo1 = 0x7fffffff;
  typename Epi::SampleC s0[CB] = {}, s1[CB] = {};
  float4 bb[CB];
  const int b0 = rps > 0 ? m0 / rps : 0;
  if (rps > 0) {
    lo0 = b0 * rps;
    lo1 = lo0 + rps;
  }
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    const int n = min(nb + i * 16, N - 4);
    bb[i] = epi.bias4(n);
    if (rps > 0) {
      s0[i] = epi.sample_consts(b0, n);
      s1[i] = epi.sample_consts(lo1 < M ? b0 + 1 : b0, n);
    }
  }
  constexpr int AHEAD = Epi::kHasAddend ? 3 : 0, NBUF = AHEAD + 1;
  float4 add[NBUF][CB];
  auto fetch = [&](int j) {
    if (!Epi::kHasAddend) return;
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const int m = min(m0 + j * 16 + l16, M - 1);
      add[j % NBUF][i] = epi.addend(m, m - (m >= lo1 ? lo1 : lo0), min(nb + i * 16, N - 4));
    }
  };
#pragma unroll
  for (int j = 0; j < AHEAD && j < RB; ++j) fetch(j);
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    if (AHEAD > 0 && j + AHEAD < RB) fetch(j + AHEAD);
    const int m = m0 + j * 16 + l16;
    const bool second = m >= lo1;
#pragma unroll
    for (int i = 0; i < CB; ++i)
      if (m < M && nb + i * 16 < N)
        epi.finish(m, m - (second ? lo1 : lo0), nb + i * 16, acc[j][i][0], acc[j][i][1], acc[j][i][2], acc[j][i][3], bb[i], second ? s1[i] : s0[i],
                   add[j % NBUF][i]);
  }
}

template <int RB, int CB, int MODE>
static br_status f32_ring_launch(const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea, hipStream_t st) {
  constexpr int BM = 16 * RB, BN = 64 * CB;
  Epilogue<MODE, float> epi{ea};
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  const int want = std::max(1, (int)std::lround(std::sqrt(tiles_m * tiles_n / 8.0 * BM / BN)));
  const int group_n = std::min(tiles_n, cdiv(tiles_n, cdiv(tiles_n, std::min(want, 8))));
  hipLaunchKernelGGL((gemm_f32_ring_kernel<RB, CB, MODE>), dim3(tiles_m * tiles_n), dim3(NW * 64), NST * (BM + BN) * 128, st, A, lda, W, ldw,
                     M, N, K, tiles_m, tiles_n, group_n, epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

template <int MODE>
static br_status f32_ring_height(const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea, int rb, int cb,
                                 hipStream_t st) {
  switch (cb == 1 ? rb : rb + 16) {
#define BR_RB(R)                                                                              \
  case R: return f32_ring_launch<R, 1, MODE>(A, lda, W, ldw, M, N, K, ea, st);                 \
  case R + 16: return f32_ring_launch<R, 2, MODE>(A, lda, W, ldw, M, N, K, ea, st);
    BR_RB(2) BR_RB(3) BR_RB(4) BR_RB(5) BR_RB(6) BR_RB(7) BR_RB(8) BR_RB(9) BR_RB(10) BR_RB(11) BR_RB(12)
#undef BR_RB
  }
  return fail(BR_EINVAL, "gemm: unknown tile height");
}

// Whole stages; a tile's rows are addressed with 32-bit byte offsets from its first one.
bool gemm_f32_ring_supported(int mode, int K, int lda, int ldw) {
  return (mode == EPI_BIAS || mode == EPI_BIAS_GELU || mode == EPI_BIAS_GATE_RES) && K % 32 == 0 &&
         16ull * rule::F32_RING_MAX_RB * lda * 4 < (1ull << 32) && 128ull * ldw * 4 < (1ull << 32);
}

br_status launch_gemm_f32_ring(int mode, const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea, int rb,
                               int cb, hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return f32_ring_height<EPI_BIAS>(A, lda, W, ldw, M, N, K, ea, rb, cb, st);
    case EPI_BIAS_GELU: return f32_ring_height<EPI_BIAS_GELU>(A, lda, W, ldw, M, N, K, ea, rb, cb, st);
    case EPI_BIAS_GATE_RES: return f32_ring_height<EPI_BIAS_GATE_RES>(A, lda, W, ldw, M, N, K, ea, rb, cb, st);
  }
  return fail(BR_EINVAL, "gemm: epilogue without a ring kernel");
}

}  // namespace br
