// Persistent bf16 GEMM for gfx950: C[m, n] = sum_k A[m, k] W[n, k], fp32 accumulate, fused epilogue.  One
// workgroup per compute unit, four waves (one per SIMD, all 512 registers each), walks a list of BM x 256 output
// tiles, BM = 32 RB; a wave owns 16 RB x 128 outputs.  The operand stream (global memory -> LDS directly) never
// stops at a tile boundary: while the last k-steps of a tile are multiplied the first stages of the next tile are
// already being fetched, and they keep landing while the finished tile goes through its epilogue.
//
// What bounds it: the matrix pipe at the clock that the chip sustains on the data.  The earlier form (eight waves of
// 128 x 64, 32x32x16 instructions, a stage's refill issued in one burst) ran 147 456 x 9216 x 3072 at 1240 TFLOP/s
// with random operands and 1650 with zeros, this one at 1500 and 1990; four things make the difference:
//  - Four waves of 128 x 128 read a third less of the operands from LDS than eight of 128 x 64.
//  - Sixteen LDS-direct loads a wave and stage, spread evenly over its 128 matrix instructions.  The vector memory
//    path takes 64 bytes a clock: a burst stands in front of the wave's next matrix instructions (it is issued in
//    order), and costs a quarter of the launch.
//  - To have time for that, the two halves of a ring slot are refilled at different times.  The W fragments of a
//    stage are all read half a stage ahead, so that W's half of the slot is free early: W of stage q + 2 is fetched
//    during the first half of stage q, A of stage q + 2 during the second, and each has at least half a stage to land.
//  - 16x16x32 matrix instructions in an order in which neighbours share an operand draw less power than 32x32x16
//    ones: the clock is higher on random operands (7 to 14 % of the launch), the same on zeros.
//
// Requirements: K % 128 == 0 (every tile starts on ring slot 0), K >= 128, operands below 4 GiB.
#include <cmath>
#include <type_traits>

#include "common.h"
#include "dispatch.h"
#include "dit.h"
#include "gemm_epilogue_wide.h"
#include "gemm_frag.h"
#include "static_for.h"

namespace br {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

namespace {
constexpr int BN = 256, NW = 4;
constexpr int BK = 64;            // k-depth of a stage: 128-byte row segments (64-byte ones pull a third less through the L2)
constexpr int IW = BN / 8 / NW;   // LDS-direct loads of W per wave and stage (8 rows each)
}  // namespace

template <int BYTES, int S>
__shared__ __attribute__((aligned(1024))) char g_ring[BYTES];
__shared__ __attribute__((aligned(1024))) char g_epi[NW * WIDE_EPI_BYTES];

// Matrix instructions on accumulators that stay in the accumulation registers.  (From the builtin the compiler keeps
// some of the 64 blocks in vector registers and moves them back and forth.)  The first of a tile starts from zero.
// The compiler does not know that these are matrix instructions and adds no wait states: two between a vector instruction that
// writes an operand and the instruction, nineteen before a result is read.  The operands therefore come straight from LDS reads
// (for which it does wait) and the accumulators are touched by nothing else until the s_nop behind the loop;
// tests/test_matrix_instructions.py checks the built code for it.
__device__ __forceinline__ void mfma16(f32x4& c, const bf16x8& w, const bf16x8& a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(a));
}
__device__ __forceinline__ void mfma16_first(f32x4& c, const bf16x8& w, const bf16x8& a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(w), "v"(a));
}

// Maps the j-th tile of workgroup `wg` to (tile_m, tile_n); false when the list is exhausted.
// Consecutive workgroup ids are spread over the 8 XCDs, so XCD x = wg % 8 gets a contiguous
// range of the tile order, shared by its workgroups in round-robin.  The order: blocks of
// row_block row panels outermost, inside a block column groups of group_n, inside a group rows
// outermost.  The 32 tiles an XCD works on at once then span 8 row panels x 4 column panels (the
// squarest footprint: fewest operand panels per round), and from one round to the next the XCD
// keeps its rows of A and moves on to the next columns of W: A, the operand that does not fit
// in the Infinity Cache at the large shapes, comes from HBM once per row block, while the
// weights, which do fit, are what is fetched again.  row_block >= tiles_m gives column groups
// over all rows.
__device__ inline bool stream_tile(int wg, int nwg, int j, int tiles_m, int tiles_n, int group_n, int row_block, int* tm,
                                   int* tn) {
  const int nt = tiles_m * tiles_n;
  const int x = wg & 7, i = wg >> 3, per_x = (nwg - x + 7) >> 3;  // workgroups on this XCD
  const int per = nt / 8, rem = nt % 8;
  const int start = x * per + (x < rem ? x : rem), cnt = per + (x < rem ? 1 : 0);
  const int local = i + j * per_x;
  if (local >= cnt) return false;
  int t = start + local;
  const int bsz = row_block * tiles_n;       // tiles of a full row block
  const int rb = t / bsz;
  t -= rb * bsz;
  const int rows = min(row_block, tiles_m - rb * row_block);
  const int gsz = rows * group_n;
  const int g = t / gsz, idx = t - g * gsz;
  const int gn = min(group_n, tiles_n - g * group_n);
  *tm = rb * row_block + idx / gn;
  *tn = g * group_n + idx - (idx / gn) * gn;
  return true;
}

template <int RB, int MODE, typename TOUT, bool KEEP>
__device__ __forceinline__ void stream_tiles(const bf16* __restrict__ A, int lda, const bf16* __restrict__ W, int ldw, int M, int N, int K,
                                             int tiles_m, int tiles_n, int group_n, int row_block, const Epilogue<MODE, TOUT>& epi) {
  constexpr int BM = 32 * RB, IA = BM / 8 / NW, LPT = IA + IW;
  constexpr int SA = BM * 128, STAGE = (BM + BN) * 128;  // bytes
  constexpr int NM = 8 * RB;                             // matrix instructions of a k32-step
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wv & 1) * 16 * RB, wn0 = (wv >> 1) * 128;
  const int nst = K / BK;  // stages per tile (even)

  // A stage row is 128 bytes = eight 16-byte chunks; chunk c of row r sits in slot c ^ ((r >> 1) & 7): sixteen
  // consecutive rows at one chunk index then cover all 64 LDS banks.  An LDS-direct load fills 8 consecutive rows
  // (lane = 8 * row + slot), so the swizzle is applied to the global address that the lane fetches from.
  // Byte offset inside a stage of this lane's fragment of 16-row block 0 for k32-step 0 (row lane & 15, chunk
  // lane >> 4); block b is 2048 bytes further, step 1 is the same ^ 64.
  const int l16 = lane & 15, lq = lane >> 4;
  const int fa_off = (wm0 + l16) * 128 + ((lq ^ ((l16 >> 1) & 7)) << 4);
  const int fw_off = SA + (wn0 + l16) * 128 + ((lq ^ ((l16 >> 1) & 7)) << 4);

  // ---- load cursor: tile and stage of the operand stream that the next refill fetches; rows past the end of the
  // matrix read its last row
  int ld_j = 0, ld_q = 0;
  unsigned off_a[IA], off_w[IW];
  const char *ld_a, *ld_w;
  auto ld_tile = [&](int tm, int tn) {
    const int m0 = tm * BM, n0 = tn * BN;
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
    ld_a = reinterpret_cast<const char*>(A + (size_t)m0 * lda);
    ld_w = reinterpret_cast<const char*>(W + (size_t)n0 * ldw);
  };
  auto ld_advance = [&]() {  // to the next stage; at the end of the list the last stage stays: fetches nobody reads
    ++ld_q;
    ld_a += BK * 2;
    ld_w += BK * 2;
    if (ld_q == nst) {
      int tm, tn;
      if (stream_tile(blockIdx.x, gridDim.x, ld_j + 1, tiles_m, tiles_n, group_n, row_block, &tm, &tn)) {
        ++ld_j;
        ld_q = 0;
        ld_tile(tm, tn);
      } else {
        --ld_q;
        ld_a -= BK * 2;
        ld_w -= BK * 2;
      }
    }
  };
  auto load_a = [&](auto S, int n) {
    char* ring = g_ring<STAGE, decltype(S)::value>;
    const unsigned dst = (unsigned)(uintptr_t)BR_LPTR(ring) + (wv * IA + n) * 1024, src = off_a[n];
    const char* p = scalar_ptr(ld_a);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(src), "s"(p) : "memory", "m0");
  };
  auto load_w = [&](auto S, int n) {
    char* ring = g_ring<STAGE, decltype(S)::value>;
    const unsigned dst = (unsigned)(uintptr_t)BR_LPTR(ring) + SA + (wv * IW + n) * 1024, src = off_w[n];
    const char* p = scalar_ptr(ld_w);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(src), "s"(p) : "memory", "m0");
  };

  f32x4 acc[8][RB];           // 16x16 blocks: columns, rows
  bf16x8 fa[2][RB], fw[2][8];  // fragments of the two k32-steps of a stage
  auto read_a = [&](const char* stage, int h, int n) {
    fa[h][n] = *reinterpret_cast<const bf16x8*>(stage + (fa_off ^ (h << 6)) + n * 2048);
  };
  auto read_w = [&](const char* stage, int h, int n) {
    fw[h][n] = *reinterpret_cast<const bf16x8*>(stage + (fw_off ^ (h << 6)) + n * 2048);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // matrix instruction t of a k32-step: W block t / RB, the A blocks forwards and back
  auto mma_one = [&](auto H, auto FIRST, auto TT) {
    constexpr int h = decltype(H)::value, t = decltype(TT)::value, i = t / RB, j = (i & 1) ? RB - 1 - t % RB : t % RB;
    if constexpr (decltype(FIRST)::value && h == 0)
      mfma16_first(acc[i][j], fw[h][i], fa[h][j]);
    else
      mfma16(acc[i][j], fw[h][i], fa[h][j]);
  };
  // One stage.  It finds in registers the A and W fragments of its step 0 and all but the last W fragment of its step
  // 1, and leaves the same of the next stage.  First barrier: every wave has read its W fragments, W's half of the slot
  // is refilled behind it (stage + 2).  Second barrier: every wave has read its A fragments, and the other slot has
  // landed (only the refill of W just issued is younger); A's half is refilled behind it.
  // `stores_behind`: the wave has issued at least that many stores since the last loads of the other slot (a tile's
  // epilogue).  Memory operations retire in issue order, so their write acknowledgements need not be waited for.
  auto stage_step = [&](auto S, auto FIRST, int stores_behind) {
    constexpr int CUR = decltype(S)::value, NXT = CUR ^ 1;
    constexpr int W_STEP = (7 * RB - 2) / 8;
    using C = std::integral_constant<int, CUR>;
    const char* cur = g_ring<STAGE, CUR>;
    const char* nxt = g_ring<STAGE, NXT>;
    static_for<NM>([&](auto TT) {
      constexpr int t = decltype(TT)::value;
      if (t == 0) read_w(cur, 1, 7);
      if (t == RB) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        ld_advance();
      }
      if (t >= RB && (t - RB) % 4 == 0 && (t - RB) / 4 < RB) read_a(cur, 1, (t - RB) / 4);
      if (t >= RB + 2 && (t - RB - 2) % W_STEP == 0 && (t - RB - 2) / W_STEP < IW) load_w(C{}, (t - RB - 2) / W_STEP);
      __builtin_amdgcn_sched_barrier(0);
      mma_one(I0{}, FIRST, TT);
      __builtin_amdgcn_sched_barrier(0);
    });
    if (stores_behind >= 8 * RB)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(8 * RB + IW < 63 ? 8 * RB + IW : 63) : "memory");
    else if (stores_behind >= 4 * RB)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(4 * RB + IW) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(IW) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<NM>([&](auto TT) {
      constexpr int t = decltype(TT)::value;
      if (t % 2 == 0 && t / 2 < RB)
        read_a(nxt, 0, t / 2);
      else if (t % 2 == 0 && t / 2 < RB + 8)
        read_w(nxt, 0, t / 2 - RB);
      if (t % RB == 1 && t > RB) read_w(nxt, 1, t / RB - 1);  // (block t / RB - 1 of this step is done)
      if (t % 8 == 4) load_a(C{}, t / 8);
      __builtin_amdgcn_sched_barrier(0);
      mma_one(I1{}, FIRST, TT);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto read_first = [&]() {  // what the first stage of a tile finds in registers
#pragma unroll
    for (int n = 0; n < RB; ++n) read_a(g_ring<STAGE, 0>, 0, n);
#pragma unroll
    for (int n = 0; n < 8; ++n) read_w(g_ring<STAGE, 0>, 0, n);
#pragma unroll
    for (int n = 0; n < 7; ++n) read_w(g_ring<STAGE, 0>, 1, n);
  };

  int tm, tn;
  stream_tile(blockIdx.x, gridDim.x, 0, tiles_m, tiles_n, group_n, row_block, &tm, &tn);
  ld_tile(tm, tn);
#pragma unroll
  for (int n = 0; n < IA; ++n) load_a(I0{}, n);
#pragma unroll
  for (int n = 0; n < IW; ++n) load_w(I0{}, n);
  ld_advance();
#pragma unroll
  for (int n = 0; n < IA; ++n) load_a(I1{}, n);
#pragma unroll
  for (int n = 0; n < IW; ++n) load_w(I1{}, n);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPT) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_first();

  char* ebuf = g_epi + wv * WIDE_EPI_BYTES;
  int stores_behind = 0, tile_j = 0;
  for (;;) {
    stage_step(I0{}, std::true_type{}, stores_behind);
    stage_step(I1{}, std::false_type{}, 0);
    for (int q = 2; q < nst; q += 2) {
      stage_step(I0{}, std::false_type{}, 0);
      stage_step(I1{}, std::false_type{}, 0);
    }
    // ---- epilogue of tile (tm, tn); the next tile's first stages keep landing meanwhile.  (The compiler does not see
    // that the accumulators come from matrix instructions: the wait for the last of them is written here.)
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    stores_behind = wide_epilogue<RB, MODE, TOUT, KEEP>(acc, ebuf, tm * BM + wm0, tn * BN + wn0, M, N, epi, lane);
    ++tile_j;
    if (!stream_tile(blockIdx.x, gridDim.x, tile_j, tiles_m, tiles_n, group_n, row_block, &tm, &tn)) break;
    // read the next tile's first fragments again rather than keep them alive across the epilogue, which needs the
    // registers for the rows it fetches ahead
    read_first();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the fetches past the end of the stream
}

#define BR_STREAM_KERNEL(NAME, KEEP)                                                                                                        \
  template <int RB, int MODE, typename TOUT>                                                                                                \
  __global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(1, 1))) void NAME(                                   \
      const bf16* __restrict__ A, int lda, const bf16* __restrict__ W, int ldw, int M, int N, int K, int tiles_m, int tiles_n, int group_n, \
      int row_block, Epilogue<MODE, TOUT> epi) {                                                                                            \
    stream_tiles<RB, MODE, TOUT, KEEP>(A, lda, W, ldw, M, N, K, tiles_m, tiles_n, group_n, row_block, epi);                                 \
  }
BR_STREAM_KERNEL(gemm_bf16_stream_kernel, false)
BR_STREAM_KERNEL(gemm_bf16_stream_keep_kernel, true)
#undef BR_STREAM_KERNEL

template <int RB, int MODE, typename TOUT>
static br_status stream_launch(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               int group_n, int row_block, hipStream_t st) {
  Epilogue<MODE, TOUT> epi{ea};
  const int tiles_m = cdiv(M, 32 * RB), tiles_n = cdiv(N, BN);
  // Default walk: column groups of 4.  The 32 tiles an XCD works on at once then span 8 row
  // panels x 4 column panels, the squarest footprint, i.e. the fewest operand panels to pull
  // into its L2 per round (a third fewer fetched bytes than whole rows of 12 or 16 tiles).
  if (group_n <= 0 || group_n > tiles_n) group_n = tiles_n > 4 ? 4 : tiles_n;
  // An A operand larger than the 256 MB Infinity Cache would come from HBM once per column group
  // when the groups run over all rows (9 to 12 times for the QKV and FC1 shapes of the large
  // networks); in blocks of 8 row panels an XCD finishes all columns of its rows before it moves
  // on, and only the weights are fetched again.  Measured: 3-7 % shorter launches at those shapes,
  // no difference where A fits in the cache.
  if (row_block <= 0) row_block = ((size_t)M * K * 2 >= (256u << 20) && tiles_n > group_n) ? 8 : tiles_m;
  if (row_block > tiles_m) row_block = tiles_m;
  const int n_cu = device_cu_count();
  const int nt = tiles_m * tiles_n;
  const int grid = nt < n_cu ? nt : n_cu;
  if constexpr (std::is_same<TOUT, bf16>::value) {
    if (rule::persistent_output_stays((size_t)M * N * sizeof(TOUT), K, MODE == EPI_BIAS_GELU)) {
      hipLaunchKernelGGL((gemm_bf16_stream_keep_kernel<RB, MODE, TOUT>), dim3(grid), dim3(256), 0, st, A, lda, W, ldw, M, N, K,
                         tiles_m, tiles_n, group_n, row_block, epi);
      BR_LAUNCH_CHECK();
      return BR_OK;
    }
  }
  hipLaunchKernelGGL((gemm_bf16_stream_kernel<RB, MODE, TOUT>), dim3(grid), dim3(256), 0, st, A, lda, W, ldw, M, N, K,
                     tiles_m, tiles_n, group_n, row_block, epi);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

template <int MODE, typename TOUT>
static br_status stream_height(const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K, const EpiArgs& ea,
                               int height, int group_n, int row_block, hipStream_t st) {
  switch (height) {
    case 4: return stream_launch<4, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, row_block, st);
    case 5: return stream_launch<5, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, row_block, st);
    case 6: return stream_launch<6, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, row_block, st);
    case 7: return stream_launch<7, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, row_block, st);
  }
  return stream_launch<8, MODE, TOUT>(A, lda, W, ldw, M, N, K, ea, group_n, row_block, st);
}

bool gemm_stream_supported(int mode, int K, size_t bytes_a, size_t bytes_w) {
  return (mode == EPI_BIAS || mode == EPI_BIAS_GELU || mode == EPI_BIAS_GATE_RES || mode == EPI_BIAS_F32) && K >= 128 &&
         K % 128 == 0 && bytes_a < (1ull << 32) && bytes_w < (1ull << 32);
}

br_status launch_gemm_bf16_stream(int mode, const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K,
                                  const EpiArgs& ea, int height, int group_n, int row_block, hipStream_t st) {
  BR_REQUIRE(gemm_stream_supported(mode, K, (size_t)M * lda * 2, (size_t)N * ldw * 2), BR_ESHAPE,
             "streaming gemm: needs K % 128 == 0 and operands below 4 GiB");
  switch (mode) {
    case EPI_BIAS: return stream_height<EPI_BIAS, bf16>(A, lda, W, ldw, M, N, K, ea, height, group_n, row_block, st);
    case EPI_BIAS_GELU: return stream_height<EPI_BIAS_GELU, bf16>(A, lda, W, ldw, M, N, K, ea, height, group_n, row_block, st);
    case EPI_BIAS_GATE_RES: return stream_height<EPI_BIAS_GATE_RES, float>(A, lda, W, ldw, M, N, K, ea, height, group_n, row_block, st);
    case EPI_BIAS_F32: return stream_height<EPI_BIAS_F32, float>(A, lda, W, ldw, M, N, K, ea, height, group_n, row_block, st);
  }
  return fail(BR_EINVAL, "gemm: unknown epilogue");
}

}  // namespace br
