// bf16 GEMM for problems of up to one round of tiles: one tile of 32 to 192 rows x 128 columns per workgroup, the lowest whose number
// does not pass that of the compute units, and a ring of four to seven stages of 64 k.  Four waves, two along either side; 16x16x32
// matrix instructions, which allow heights in steps of 32.
//
// What bounds such a problem is one compute unit's share, in instruction slots: a wave's fragment reads (31 B/clk) and its part of the
// loads into LDS (64 B/clk for the unit) have to lie between the matrix instructions one by one.  1101 x 1024 x 4096 in 160 rows (56 tiles; a
// stage is 640 cycles of matrix instructions): 1100 cycles a stage with reads and loads in bursts, 900 spread out; 1860 with the
// accumulators in accumulation registers, which the compiler shuffles.  About 6 us go to launch, first stages and epilogue.  Against 64x64
// tiles (some units have two) and the persistent kernel (128 rows x 256 columns at least): 1101 x 3072 x 1024 14.6 -> 11.0 us, 1101 x 4096 x
// 1024 17.1 -> 14.3, 2202 x 1024 x 4096 36.8 -> 27.6, 4404 x 1024 x 4096 54 -> 39 (0.95 PFLOP/s).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "dit.h"
#include "gemm_epilogue.h"
#include "gemm_frag.h"

namespace br {

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

namespace {
constexpr int BN = 128, WTN = 64, CB = WTN / 16;  // columns of a tile and of a wave; its blocks of 16
constexpr int WGM = 2, NW = 4;                    // waves along the rows; in all
template <int Y, int LPW>
__device__ __forceinline__ void ring_wait(int younger) {
  if constexpr (Y == 0)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  else if (younger >= Y)
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(Y * LPW) : "memory");
  else
    ring_wait<Y - 1, LPW>(younger);
}
}  // namespace

// The ring.  (Sized at the launch: a compiler that knows how little fits a compute unit puts the accumulators into accumulation
// registers, and moves them to others and back in every step.)
extern __shared__ __attribute__((aligned(1024))) char g_ring[];

// RB: 16-row blocks of a wave; NST: stages of 64 k.
template <int RB, int NST, int MODE, typename TOUT>
__global__ __launch_bounds__(256, 2) void gemm_ring_kernel(const bf16* __restrict__ A, int lda, const bf16* __restrict__ W,
                                                              int ldw, int M, int N, int K, int tiles_m, int tiles_n,
                                                              int group_n, Epilogue<MODE, TOUT> epi) {
  typedef GemmFrag16<bf16> F;
  typedef typename F::type frag;
  constexpr int BM = 16 * RB * WGM, STAGE = (BM + BN) * 128;  // rows, bytes
  constexpr int GA = BM / 8, LPW = (GA + BN / 8) / NW;                      // 8-row groups of A; loads of a wave and stage
  static_assert((GA + BN / 8) % NW == 0 && (NST - 1) * LPW < 64 && NST * STAGE <= 160 * 1024 && NST >= 3 && NST <= 7, "ring");
  static_assert(NW * 4096 <= NST * STAGE, "epilogue staging");
  char* const ring = g_ring;

  // a compute die's tiles are consecutive, rows outermost inside a group of columns
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
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wv % WGM) * 16 * RB, wn0 = (wv / WGM) * WTN;
  const int l16 = lane & 15, lq = lane >> 4;

  // Load j of a wave fills the 8 rows of group wv * LPW + j of the stage (A's rows, then W's): lane = 8 * row + slot, and slot s of
  // row r holds chunk s ^ ((r >> 1) & 7).
  unsigned off[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int g = wv * LPW + j, row = (g < GA ? g : g - GA) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    off[j] = g < GA ? (unsigned)min(row, M - 1 - m0) * (unsigned)lda * 2u + c * 16
                    : (unsigned)min(row, N - 1 - n0) * (unsigned)ldw * 2u + c * 16;
  }
  const char* a_tile = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
  const char* w_tile = reinterpret_cast<const char*>(W + (size_t)n0 * ldw);
  const unsigned ring0 = (unsigned)(uintptr_t)BR_LPTR(ring) + wv * LPW * 1024;
  const int nk = K / 64;
  auto load = [&](int j, int kt, int slot) __attribute__((always_inline)) {
    const char* src = scalar_ptr((wv * LPW + j < GA ? a_tile : w_tile) + (size_t)kt * 128);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(ring0 + slot * STAGE + j * 1024), "v"(off[j]), "s"(src) : "memory", "m0");
  };
  // waits until at most the loads of `younger` stages are outstanding (they retire in order) and all LDS reads have arrived
  auto wait = [&](int younger) __attribute__((always_inline)) { ring_wait<NST - 1, LPW>(younger); };

  f32x4 acc[CB][RB];
#pragma unroll
  for (int i = 0; i < CB; ++i)
#pragma unroll
    for (int j = 0; j < RB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // fragments of half h (32 of the 64 k) of a stage; those of the next half are read while a half is multiplied
  frag fa[2][RB], fw[2][CB];
  const int fa0 = F::offset(wm0 + l16, lq), fw0 = BM * 128 + F::offset(wn0 + l16, lq);
  auto read = [&](int slot, int h, int r) __attribute__((always_inline)) {  // in the order of their use
    const char* p = ring + slot * STAGE;
    if (r < CB) fw[h][r] = *reinterpret_cast<const frag*>(p + (fw0 ^ (h * F::FLIP)) + r * 2048);
    else fa[h][r - CB] = *reinterpret_cast<const frag*>(p + (fa0 ^ (h * F::FLIP)) + (r - CB) * 2048);
  };

  // The first LP loads of a stage go out in the half stage in which its slot becomes free, the others in the next.
  constexpr int LP = (LPW + 1) / 2;
  for (int s = 0; s < NST - 1 && s < nk; ++s)
#pragma unroll
    for (int j = 0; j < LPW; ++j) load(j, s, s);
  if (nk >= NST) {
#pragma unroll
    for (int j = 0; j < LP; ++j) load(j, NST - 1, NST - 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * LPW + LP) : "memory");
  } else {
    wait(nk - 1);
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  // lgkmcnt(0), said to the compiler: a scalar load that it believes under way makes it wait for all LDS reads in every half stage
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int r = 0; r < CB + RB; ++r) read(0, 0, r);
  int slot = 0;
  // Half a stage's products.  Between them, one by one: the reads of the next half's fragments (half 1 - h of slot `from`), over three
  // quarters of the time so that they have arrived at its end, and `count` loads from number `first` of stage kl on.  In bursts either
  // stand in front of the wave's own matrix instructions: one wave reads 31 B/clk and the loads share 64.
  auto half = [&](auto Hc, int from, auto FIRST, auto COUNT, int kl, int to) __attribute__((always_inline)) {
    constexpr int h = decltype(Hc)::value, first = decltype(FIRST)::value, count = decltype(COUNT)::value;
    constexpr int NM = RB * CB, NR = RB + CB, SPAN = NM * 3 / 4;
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      const int j = n / CB, i = (j & 1) ? CB - 1 - n % CB : n % CB;  // (neighbours share an operand: less power)
      acc[i][j] = F::mma(fw[h][i], fa[h][j], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = (n * NR + SPAN - 1) / SPAN; r < ((n + 1) * NR + SPAN - 1) / SPAN && r < NR; ++r) read(from, 1 - h, r);
#pragma unroll
      for (int l = n * count / NM; l < (n + 1) * count / NM; ++l) load(first + l, kl, to);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // LATE: the second part of stage kt + NST - 1 is still to be fetched; EARLY: the first part of stage kt + NST
  auto step = [&](int kt, auto LATE, auto EARLY) __attribute__((always_inline)) {
    constexpr bool late = decltype(LATE)::value, early = decltype(EARLY)::value;
    const int next = slot + 1 == NST ? 0 : slot + 1, prev = slot == 0 ? NST - 1 : slot - 1;
    half(I0{}, slot, std::integral_constant<int, LP>{}, std::integral_constant<int, late ? LPW - LP : 0>{}, kt + NST - 1, prev);
    // Stage kt + 1 has landed and the fragments of stage kt are in registers; after the barrier this holds for every wave: stage
    // kt + 1 may be read and stage kt refilled.  (Behind the last stage an old one is read once more, which nobody uses.)
    wait(early ? NST - 2 : min(nk - 2 - kt, NST - 2));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    half(I1{}, next, I0{}, std::integral_constant<int, early ? LP : 0>{}, kt + NST, slot);
    slot = next;
  };
  int kt = 0;
  for (; kt + NST < nk; ++kt) step(kt, std::true_type{}, std::true_type{});
  if (kt + NST == nk) step(kt++, std::true_type{}, std::false_type{});
  for (; kt < nk; ++kt) step(kt, std::false_type{}, std::false_type{});
  __syncthreads();  // every wave is done with the ring
  wave_epilogue16<RB, MODE, TOUT>(acc, ring + wv * 4096, m0 + wm0, n0 + wn0, M, N, epi, lane);
}

template <int RB, int NST, int MODE, typename TOUT>
static br_status ring_launch(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea, int group_n,
                             hipStream_t st) {
  Epilogue<MODE, TOUT> epi{ea};
  constexpr int BM = 16 * RB * WGM;
  const int tiles_m = cdiv(M, BM), tiles_n = cdiv(N, BN);
  if (group_n <= 0) {
    // The tiles of a compute die in a nearly square patch: it fetches the fewest operand bytes into its L2.
    const int want = std::max(1, (int)std::lround(std::sqrt(tiles_m * tiles_n / 8.0 * BM / BN)));
    group_n = cdiv(tiles_n, cdiv(tiles_n, want));
  }
  if (group_n > tiles_n) group_n = tiles_n;
  hipLaunchKernelGGL((gemm_ring_kernel<RB, NST, MODE, TOUT>), dim3(tiles_m * tiles_n), dim3(NW * 64), NST * (BM + BN) * 128, st, A, lda, W, ldw, M,
                     N, K, tiles_m, tiles_n, group_n, epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

template <int MODE, typename TOUT>
static br_status ring_height(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea, int height,
                             int group_n, hipStream_t st) {
  switch (height) {
    case 2: return ring_launch<1, 7, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 4: return ring_launch<2, 6, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 6: return ring_launch<3, 5, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 8: return ring_launch<4, 5, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 10: return ring_launch<5, 4, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
    case 12: return ring_launch<6, 4, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, st);
  }
  return fail(BR_EINVAL, "gemm: unknown tile height");
}

// height: rows of a tile / 16.  A tile's rows are addressed with 32-bit byte offsets from its first one.
bool gemm_ring_supported(int mode, int height, int lda, int ldw) {
  return (mode == EPI_BIAS || mode == EPI_BIAS_GELU || mode == EPI_BIAS_F32 || mode == EPI_BIAS_GATE_RES) &&
         height >= 2 && height <= 12 && height % 2 == 0 && 16ull * height * lda * 2 < (1ull << 32) && (unsigned long long)BN * ldw * 2 < (1ull << 32);
}

br_status launch_gemm_bf16_ring(int mode, const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                                int height, int group_n, hipStream_t st) {
  switch (mode) {
    case EPI_BIAS: return ring_height<EPI_BIAS, bf16>(A, lda, W, ldw, M, N, K, ea, height, group_n, st);
    case EPI_BIAS_GELU: return ring_height<EPI_BIAS_GELU, bf16>(A, lda, W, ldw, M, N, K, ea, height, group_n, st);
    case EPI_BIAS_F32: return ring_height<EPI_BIAS_F32, float>(A, lda, W, ldw, M, N, K, ea, height, group_n, st);
    case EPI_BIAS_GATE_RES: return ring_height<EPI_BIAS_GATE_RES, float>(A, lda, W, ldw, M, N, K, ea, height, group_n, st);
  }
  return fail(BR_EINVAL, "gemm: epilogue without a ring kernel");
}

}  // namespace br
