// GEMM with one output tile per workgroup on the gfx950 matrix cores, bf16 or fp32 operands:
// C[m, n] = sum_k A[m, k] W[n, k], fp32 accumulate, fused epilogue.
#pragma once
#include <type_traits>

#include "common.h"
#include "dit.h"
#include "gemm_epilogue.h"
#include "gemm_frag.h"

namespace br {

// ---------------------------------------------------------------------------
// Operand tiles go from global memory straight into LDS
// (global_load_lds_dwordx4, no register staging), 64 bytes of k per stage, four stages,
// three of them in flight while the fourth is multiplied.  One tile's worth of
// registers is freed and, more importantly, about three times as many bytes are in
// flight per compute unit, which is what hides the L2/HBM latency.
//
// An LDS-direct load writes 64 lanes x 16 bytes to consecutive LDS addresses, i.e.
// 16 tile rows of 64 bytes; the swizzle is therefore applied on the global side:
// the lane that fills slot s of row r fetches k-chunk s ^ ((r >> 2) & 3).  Sixteen
// consecutive rows at one k-chunk then cover all 64 LDS banks exactly once.
// Each stage is its own __shared__ array and the k-loop is unrolled by the number
// of stages, so the compiler can tell the buffers apart and does not serialise the
// LDS reads of one stage against the loads in flight for the others.
#define BR_GPTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

template <int BYTES, int S>
__shared__ __attribute__((aligned(1024))) char g_stage[BYTES];

template <typename T, int BM, int BN, int WGM, int WGN, int MODE, typename TOUT>
__global__ __launch_bounds__(WGM* WGN * 64) void gemm_tile_kernel(const T* __restrict__ A, int lda,
                                                                  const T* __restrict__ W, int ldw, int M, int N,
                                                                  int K, int tiles_m, int tiles_n, int group_n,
                                                                  Epilogue<MODE, TOUT> epi) {
  constexpr int CE = 16 / (int)sizeof(T), KD = 4 * CE;  // elements of a 16-byte chunk; k-depth of a stage (64 bytes)
  typedef typename GemmFrag<T>::type frag;
  constexpr int NW = WGM * WGN;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int IA = BM / 16 / NW, IW = BN / 16 / NW;  // LDS-direct loads per wave and stage
  constexpr int LPT = IA + IW;
  constexpr int SA = BM * 64, STAGE = (BM + BN) * 64;   // bytes
  static_assert(BM % (16 * NW) == 0 && BN % (16 * NW) == 0, "tile / wave mismatch");

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

  // global source of this lane for each of its loads (k advances by KD per stage)
  const T* ga[IA];
  const T* gw[IW];
#pragma unroll
  for (int j = 0; j < IA; ++j) {
    const int row = (wv * IA + j) * 16 + (lane >> 2), c = (lane & 3) ^ ((row >> 2) & 3);
    ga[j] = A + (size_t)min(m0 + row, M - 1) * lda + c * CE;
  }
#pragma unroll
  for (int j = 0; j < IW; ++j) {
    const int row = (wv * IW + j) * 16 + (lane >> 2), c = (lane & 3) ^ ((row >> 2) & 3);
    gw[j] = W + (size_t)min(n0 + row, N - 1) * ldw + c * CE;
  }
  // byte offsets of this lane's operand fragments inside a stage, per k16 step
  int fa_off[2][TM], fw_off[2][TN];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int row = wm0 + j * 32 + l32;
      fa_off[ks][j] = row * 64 + (((ks * 2 + lh) ^ ((row >> 2) & 3)) << 4);
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int row = wn0 + i * 32 + l32;
      fw_off[ks][i] = SA + row * 64 + (((ks * 2 + lh) ^ ((row >> 2) & 3)) << 4);
    }
  }

  f32x16 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = K / KD;
  // The LDS-direct loads are issued from inline assembly: the compiler then does not
  // see LDS being written and adds no waits of its own; completion is tracked here
  // by hand.  Every step issues exactly LPT loads (past the end of K the last k-tile
  // is fetched again into a stage nobody reads), so "at most 2*LPT loads outstanding"
  // always means that the stage about to be multiplied has landed.
  auto issue = [&](auto S, int kt) {
    char* stage_ptr = g_stage<STAGE, decltype(S)::value>;
    const unsigned base = (unsigned)(uintptr_t)BR_LPTR(stage_ptr);
    const int kk = min(kt, nk - 1);
#pragma unroll
    for (int j = 0; j < IA; ++j) {
      const T* src = ga[j] + (size_t)kk * KD;
      const unsigned dst = base + (wv * IA + j) * 1024;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
    }
#pragma unroll
    for (int j = 0; j < IW; ++j) {
      const T* src = gw[j] + (size_t)kk * KD;
      const unsigned dst = base + SA + (wv * IW + j) * 1024;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
    }
  };
  // Operand fragments are prefetched one k16 half-step ahead: while the MFMAs of
  // (kt, first half) run, the fragments of (kt, second half) are read; while those
  // are multiplied, the first-half fragments of stage kt+1 are read.  The barrier
  // sits between the two halves, where every wave still has MFMAs in flight.
  frag fa0[TM], fw0[TN], fa1[TM], fw1[TN];
  auto read_half = [&](const char* stage, int ks, frag* a, frag* w) {
#pragma unroll
    for (int j = 0; j < TM; ++j) a[j] = *reinterpret_cast<const frag*>(stage + fa_off[ks][j]);
#pragma unroll
    for (int i = 0; i < TN; ++i) w[i] = *reinterpret_cast<const frag*>(stage + fw_off[ks][i]);
  };
  auto mma_half = [&](const frag* a, const frag* w) {
#pragma unroll
    for (int e = 0; e < GemmFrag<T>::STEPS; ++e)
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = GemmFrag<T>::mma(w[i], a[j], acc[i][j], e);
  };
  auto step = [&](auto S, int kt) {
    constexpr int CUR = decltype(S)::value, NXT = (CUR + 1) & 3;
    const char* cur = g_stage<STAGE, CUR>;
    const char* nxt = g_stage<STAGE, NXT>;
    read_half(cur, 1, fa1, fw1);
    __builtin_amdgcn_sched_barrier(0);  // keep the LDS reads ahead of the MFMAs they overlap with
    mma_half(fa0, fw0);
    __builtin_amdgcn_sched_barrier(0);  // ... and the MFMAs ahead of the barrier
    // own loads of stage kt+1 landed (only the two younger stages may be outstanding)
    // and both halves of stage kt are in registers -> barrier -> true for every wave:
    // stage kt+1 may be read and stage kt may be refilled
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * LPT) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(std::integral_constant<int, CUR>{}, kt + 4);
    read_half(nxt, 0, fa0, fw0);
    __builtin_amdgcn_sched_barrier(0);
    mma_half(fa1, fw1);
    __builtin_amdgcn_sched_barrier(0);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;

  issue(I0{}, 0);
  issue(I1{}, 1);
  issue(I2{}, 2);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LPT) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  issue(I3{}, 3);
  read_half(g_stage<STAGE, 0>, 0, fa0, fw0);
  for (int kt = 0;; kt += 4) {
    step(I0{}, kt);
    if (kt + 1 >= nk) break;
    step(I1{}, kt + 1);
    if (kt + 2 >= nk) break;
    step(I2{}, kt + 2);
    if (kt + 3 >= nk) break;
    step(I3{}, kt + 3);
    if (kt + 4 >= nk) break;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the refills past the end of K
  __syncthreads();                                  // every wave is done with the stages
  {
    constexpr int WPS = STAGE / 4096;  // waves whose 4 KB fit in one stage
    static_assert(2 * WPS >= NW && WTN == 64, "epilogue staging needs 4 KB per wave");
    char* ebuf = (wv < WPS ? g_stage<STAGE, 0> + wv * 4096 : g_stage<STAGE, 1> + (wv - WPS) * 4096);
    wave_epilogue<TM, TN, MODE, TOUT>(acc, ebuf, m0 + wm0, n0 + wn0, M, N, epi, lane);
  }
}

}  // namespace br
