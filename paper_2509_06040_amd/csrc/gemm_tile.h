// GEMM with one output tile per workgroup on the gfx950 matrix cores (bf16 operands):
// C[m, n] = sum_k A[m, k] W[n, k], fp32 accumulate, fused epilogue.
#pragma once
#include <type_traits>

#include "common.h"
#include "dit.h"
#include "gemm_epilogue.h"
#include "gemm_frag.h"

namespace br {

// ---------------------------------------------------------------------------
// Operand tiles go from global memory straight into LDS (global_load_lds_dwordx4, no register
// staging), 128 bytes of k of every row per stage, NST stages in a ring: one is multiplied while the others
// are in flight.  Full 128-byte lines matter: the same ring with stages of 64 bytes per row pulled a third
// less through the L2.
//
// An LDS-direct load writes 64 lanes x 16 bytes to consecutive LDS addresses, i.e. 8 tile rows of 128
// bytes; the swizzle is therefore applied on the global side: the lane that fills slot s of row r fetches
// k-chunk s ^ ((r >> 1) & 7).  Sixteen consecutive rows at one k-chunk then cover all 64 LDS banks once.
// Each stage is its own __shared__ array and the k-loop is unrolled by the number of stages, so the
// compiler can tell the buffers apart and does not serialise the LDS reads of one stage against the
// loads in flight for the others.
#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

template <int BYTES, int S>
__shared__ __attribute__((aligned(1024))) char g_stage[BYTES];

template <int BM, int BN, int WGM, int WGN, int NST, int MODE, typename TOUT, bool STREAM>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_tile_kernel(const bf16* __restrict__ A, int lda,
                                                                  const bf16* __restrict__ W, int ldw, int M, int N,
                                                                  int K, int tiles_m, int tiles_n, int group_n,
                                                                  Epilogue<MODE, TOUT> epi) {
  constexpr int KD = 64;  // k-depth of a stage
  typedef GemmFrag32::type frag;
  constexpr int NW = WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int IA = BM / 8 / NW, IW = BN / 8 / NW;  // LDS-direct loads per wave and stage
  constexpr int LPT = IA + IW;
  constexpr int SA = BM * 128, STAGE = (BM + BN) * 128;   // bytes
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "tile / wave mismatch");
  static_assert(NST >= 2 && NST <= 4 && (NST - 1) * LPT < 64, "ring depth");

  const int nwg = tiles_m * tiles_n;
  int wg = blockIdx.x;
  {
    const int per = nwg / 8, rem = nwg % 8, x = wg % 8, i = wg / 8;
    wg = x * per + (x < rem ? x : rem) + i;
  }
  int tile_m, tile_n;
  {
    const int gsz = tiles_m * group_n;
    const int g = wg / gsz, idx = wg - g * gsz;
    const int gn = min(group_n, tiles_n - g * group_n);
    tile_m = idx / gn;
    tile_n = g * group_n + idx - tile_m * gn;
  }
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wv % WGM) * WTM, wn0 = (wv / WGM) * WTN;
  const int l32 = lane & 31, lh = lane >> 5;

  // byte offset of this lane's source of each load from the tile's first row (k advances by a stage in the
  // scalar base address)
  unsigned off_a[IA], off_w[IW];
#pragma unroll
  for (int j = 0; j < IA; ++j) {
    const int row = (wv * IA + j) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    off_a[j] = (unsigned)min(row, M - 1 - m0) * (unsigned)lda * 2u + c * 16;
  }
#pragma unroll
  for (int j = 0; j < IW; ++j) {
    const int row = (wv * IW + j) * 8 + (lane >> 3), c = (lane & 7) ^ ((row >> 1) & 7);
    off_w[j] = (unsigned)min(row, N - 1 - n0) * (unsigned)ldw * 2u + c * 16;
  }
  const char* a_tile = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
  const char* w_tile = reinterpret_cast<const char*>(W + (size_t)n0 * ldw);
  // byte offsets of this lane's first operand fragments inside a stage for chunk pair 0; pair p is the same ^ (p << 5), the
  // fragments of the other 32-row blocks are 4 KB apart
  const int fa_off = GemmFrag32::offset(wm0 + l32, lh), fw_off = SA + GemmFrag32::offset(wn0 + l32, lh);

  f32x16 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = K / KD;
  // The LDS-direct loads are issued from inline assembly: the compiler then does not see LDS being written
  // and adds no waits of its own; completion is tracked here by hand.
  auto issue = [&](auto S, int kt) {
    char* stage_ptr = g_stage<STAGE, decltype(S)::value>;
    const unsigned base = (unsigned)(uintptr_t)BR_LPTR(stage_ptr);
    const char* ap = scalar_ptr(a_tile + (size_t)kt * 128);
    const char* wp = scalar_ptr(w_tile + (size_t)kt * 128);
#pragma unroll
    for (int j = 0; j < IA; ++j) {
      const unsigned src = off_a[j];
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base + (wv * IA + j) * 1024), "v"(src), "s"(ap) : "memory", "m0");
    }
#pragma unroll
    for (int j = 0; j < IW; ++j) {
      const unsigned src = off_w[j];
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(base + SA + (wv * IW + j) * 1024), "v"(src), "s"(wp) : "memory", "m0");
    }
  };
  // waits until at most the loads of `younger` stages are outstanding (loads retire in order) and all
  // LDS reads have arrived
  auto wait = [&](int younger) {
    if (NST > 3 && younger >= 3)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(3 * LPT) : "memory");
    else if (NST > 2 && younger >= 2)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * LPT) : "memory");
    else if (younger >= 1)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LPT) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  };
  // Operand fragments are read one chunk pair ahead: while the matrix instructions of pair p run, the
  // fragments of pair p + 1 are read, and behind those of the last pair the first pair of the next stage.
  // The one barrier of a stage sits in front of the last pair, where every wave has instructions in flight.
  frag fa[2][TM], fw[2][TN];
  auto read_pair = [&](const char* stage, int p, int set) {
#pragma unroll
    for (int j = 0; j < TM; ++j) fa[set][j] = GemmFrag32::load(stage + j * 4096, fa_off ^ (p << 5));
#pragma unroll
    for (int i = 0; i < TN; ++i) fw[set][i] = GemmFrag32::load(stage + i * 4096, fw_off ^ (p << 5));
  };
  auto mma_pair = [&](int set) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) acc[i][j] = GemmFrag32::mma(fw[set][i], fa[set][j], acc[i][j]);
  };
  auto step = [&](auto S, int kt) {
    constexpr int CUR = decltype(S)::value, NXT = (CUR + 1) % NST;
    const char* cur = g_stage<STAGE, CUR>;
    const char* nxt = g_stage<STAGE, NXT>;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      read_pair(cur, p + 1, (p + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);  // keep the LDS reads ahead of the MFMAs they overlap with
      mma_pair(p & 1);
      __builtin_amdgcn_sched_barrier(0);  // ... and the MFMAs ahead of the barrier
    }
    // stage kt + 1 has landed and the fragments of stage kt are in registers -> barrier -> true for every
    // wave: stage kt + 1 may be read and stage kt refilled
    wait(min(nk - 2 - kt, NST - 2));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (kt + NST < nk) issue(S, kt + NST);
    if (kt + 1 < nk) read_pair(nxt, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    mma_pair(1);
    __builtin_amdgcn_sched_barrier(0);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, (NST > 2 ? 2 : 0)>;
  using I3 = std::integral_constant<int, (NST > 3 ? 3 : 0)>;

  issue(I0{}, 0);
  if (nk > 1) issue(I1{}, 1);
  if (NST > 2 && nk > 2) issue(I2{}, 2);
  if (NST > 3 && nk > 3) issue(I3{}, 3);
  wait(min(nk, NST) - 1);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_pair(g_stage<STAGE, 0>, 0, 0);
  for (int kt = 0;; kt += NST) {
    step(I0{}, kt);
    if (kt + 1 >= nk) break;
    step(I1{}, kt + 1);
    if (kt + 2 >= nk) break;
    if constexpr (NST > 2) {
      step(I2{}, kt + 2);
      if (kt + 3 >= nk) break;
    }
    if constexpr (NST > 3) {
      step(I3{}, kt + 3);
      if (kt + 4 >= nk) break;
    }
  }
  __syncthreads();  // every wave is done with the stages
  {
    constexpr int WPS = STAGE / 4096;  // waves whose 4 KB fit in one stage
    static_assert(2 * WPS >= NW && WTN == 64, "epilogue staging needs 4 KB per wave");
    char* ebuf = (wv < WPS ? g_stage<STAGE, 0> + wv * 4096 : g_stage<STAGE, 1> + (wv - WPS) * 4096);
    wave_epilogue<TM, TN, MODE, TOUT, STREAM>(acc, ebuf, m0 + wm0, n0 + wn0, M, N, epi, lane);
  }
}

}  // namespace br
