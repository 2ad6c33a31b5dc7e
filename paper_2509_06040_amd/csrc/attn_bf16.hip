// bf16 flash attention on the gfx950 matrix cores: softmax(Q K^T / sqrt(d)) V over
// all L tokens of a sample, one workgroup per (128 queries, head, sample), four
// wavefronts of 32 queries each, key/value tiles of 64 keys in LDS.
//
// Scores are computed transposed, S^T = K Q^T: in the 32x32 MFMA accumulator a
// lane then holds 16 keys of ONE query (the other 16 sit in lane ^ 32), so the
// reference / sum / rescale of the online softmax are per-lane scalars and the
// exponentiated tile is already laid out as the column operand of O^T = V^T P^T.
// The contraction order of that product is permuted to match the accumulator layout.
//
// Both tiles travel from global memory straight into LDS (no registers, no vector
// instructions on the way), row-major as they lie in the QKV buffer, with their 16-byte
// chunks permuted per row so that fragment reads spread over the banks.  The row operand
// of the second product needs V transposed; the LDS transpose read delivers that: in a
// group of 16 lanes, lane 4 r + q supplies the address of 8 bytes (4 values of row r) and
// lane j receives element j of rows 0..3, so each lane ends up with four consecutive keys
// of its own channel.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "dispatch.h"
#include "dit.h"
#include "prof.h"
#include "static_for.h"

namespace br {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
constexpr int KV_TILE = 64;
constexpr long long WARM_BYTES_PER_TILE = 2 << 20;  // what 256 idle compute units read while a workgroup takes a key tile

// (a uniform address; saying so keeps it in scalar registers)
static __device__ inline const char* uniform_ptr(const char* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return reinterpret_cast<const char*>(((unsigned long long)hi << 32) | lo);
}

// A buffer of `bytes` bytes from p (uniform over the wave) on.
static __device__ inline u32x4 sample_rows(const bf16* p, unsigned bytes) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  return u32x4{(unsigned)__builtin_amdgcn_readfirstlane((unsigned)v), (unsigned)__builtin_amdgcn_readfirstlane((unsigned)(v >> 32)) & 0xffffu, bytes, 0x00020000u};
}

// What the workgroups in front of a launch that leaves compute units idle do: they read the weights of the products behind the attention
// once, in whole rows, so that these find them in the memory-side cache (256 MB) instead of pulling them from HBM in columns of 128 bytes,
// 8 KB apart at K = 4096 (1101 x 1024 x 4096 with weights from HBM 25 us, from that cache 19.3).  One sample of the image network, 112 of 256
// units idle: the two gated projections of a block 37 -> 29 us, the attention itself 14.3 -> 15.3; with plain stores of the activations, which
// leave those in the caches as well, 1128 -> 1025 us a call (plain stores alone 1117, the weights alone 1117).
static __device__ inline void warm_rows(const WarmRows& w) {
  const unsigned stride = w.blocks * 256;
#pragma unroll
  for (int r = 0; r < WarmRows::RANGES; ++r) {
    const u32x4* p = reinterpret_cast<const u32x4*>(w.p[r]);
    const unsigned n = w.n16[r];
    for (unsigned i = blockIdx.x * 256 + threadIdx.x; i < n; i += 8 * stride) {
      u32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[min(i + u * stride, n - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(v[u]));  // (read for its own sake)
    }
  }
}

// Launches without such workgroups carry neither their code nor their list.  With both, head dim 128: 4 heads of 2561 tokens 58.6 -> 59.2 us, 8 of 3492
// 75.7 -> 76.5, 4 of 8 4.05 -> 4.10; 0.2 us of the host's.
struct NoWarm {};
template <bool WARM>
using Warm = std::conditional_t<WARM, WarmRows, NoWarm>;

// The (sample, head) pair and the query tile of a workgroup; false: none (a workgroup that reads weights, or one past the last pair).
// Workgroups are dispatched round-robin over the 8 XCDs.  All query tiles of one
// (sample, head) read the same keys and values, so they are given to one XCD and run
// back to back there: K/V then come out of that XCD's L2 instead of being fetched 8 times.
// (With few pairs that would leave XCDs idle: then tiles are simply dealt out in order.)
template <typename W>
static __device__ __forceinline__ bool attn_tile(const W& warm, int nq, int n_pairs, int grouped, int* pair, int* qt) {
  unsigned block = blockIdx.x;
  if constexpr (std::is_same<W, WarmRows>::value) {
    if (block < (unsigned)warm.blocks) {
      warm_rows(warm);
      return false;
    }
    block -= warm.blocks;  // (a multiple of 8)
  }
  if (grouped) {
    const int x = block & 7, slot = block >> 3;
    *pair = (slot / nq) * 8 + x;
    *qt = slot - (slot / nq) * nq;
  } else {
    *pair = block / nq;
    *qt = block - *pair * nq;
  }
  return *pair < n_pairs;
}

// Slot permutations of the K and V tiles: 16-byte chunk c of row r sits in slot c ^ swz(r).
// The LDS has 64 banks of 4 bytes; a 16-byte read is served 16 lanes at a time and an 8-byte
// read 32 lanes at a time, conflict-free when those lanes cover all 256 bytes of a bank row.
//   K (ds_read_b128, lanes 0..15 = 16 consecutive rows at one chunk index): with 256-byte rows
//   the rows must land in 16 different slots, with 128-byte rows (two per bank row) row pairs in 8.
//   V (transposing 8-byte reads, 32 lanes = 4 consecutive rows x 4 consecutive chunks): with
//   256-byte rows the four rows take the four groups of 4 slots, with 128-byte rows the rows
//   r and r + 2, which share a bank row, take different halves.
template <int DH>
__device__ inline int k_swz(int r) { return DH == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int DH>
__device__ inline int v_swz(int r) { return DH == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2); }

// With at most 256 registers a wave (two waves per SIMD) the compiler keeps the MFMA results in
// ordinary vector registers, where the softmax works on them directly (accumulation registers
// would cost a copy per element).  Head dim 64 runs three waves per SIMD (168 registers: the
// tile loop then spills nothing; a fourth wave bought no time).
// PRE: the q third of the buffer already carries the factor log2(e) / sqrt(DH), as the network's
// QKV projection writes it; otherwise the exponent is scaled here, one multiplication per score.
template <int DH, bool PRE, bool WARM>
__global__ __launch_bounds__(256, DH == 64 ? 3 : 2) void attn_bf16_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ out, int L,
                                                           int H, int NH, int n_pairs, int grouped, float scale_log2, Warm<WARM> warm) {
  constexpr int CH = DH / 8;    // 16-byte chunks per K row
  constexpr int KS = DH / 16;   // MFMA k-steps of the score product
  constexpr int DB = DH / 32;   // 32-row blocks of O^T
  constexpr int RPI = 64 / CH;              // rows covered by one 1 KB load
  constexpr int LPW = KV_TILE / RPI / 4;    // loads per wave, tile and operand
  constexpr int NPAR = RPI == 8 ? 2 : 4;    // distinct slot patterns among a wave's loads (the swizzle period is 16 rows)
  constexpr int ROW_B = CH * 16;            // bytes per row
  constexpr int TILE_B = KV_TILE * ROW_B;
  // Operand fragments are read from LDS RA matrix instructions ahead of the one that consumes them
  // (0: each read directly before its use, left to the compiler's scheduling).  With two waves a
  // SIMD the LDS latency in front of every matrix instruction is otherwise exposed: 2-4 % of the
  // launch at head dim 128, no more beyond two steps; nothing at head dim 64 with its three waves.
  constexpr int RA = DH == 64 ? 0 : 2;
  __shared__ __attribute__((aligned(1024))) char sK[2][TILE_B];
  __shared__ __attribute__((aligned(1024))) char sV[2][TILE_B];

  int pair, qt;
  if (!attn_tile(warm, (L + 127) / 128, n_pairs, grouped, &pair, &qt)) return;
  const int b = pair / NH, h = pair - b * NH;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t ld = (size_t)3 * H;
  const bf16* base = qkv + (size_t)b * L * ld + (size_t)h * DH;
  const int qi = qt * 128 + wv * 32 + l32;
  const int qc = min(qi, L - 1);
  const bool active = qt * 128 + wv * 32 < L;  // (uniform over the wave)

  bf16x8 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = *reinterpret_cast<const bf16x8*>(base + (size_t)qc * ld + ks * 16 + lh * 8);

  f32x16 o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  float m_run = 0.f, l_run = 0.f;  // reference (a bf16 value) and row sum of the probabilities taken against it
  // Row sums on the matrix pipe: v_mfma_f32_16x16x32 takes the registers of a probability step (lanes 0..15 / 16..31: keys 0..7 of
  // queries 0..15 / 16..31, lanes 32..63 their keys 8..15) as sixteen columns of four k-groups, so the even groups belong to
  // one half of the queries, the odd ones to the other; the row side is 1 where a row's result lands in that half's lanes.  Sixteen
  // cycles of the matrix pipe a step instead of four v_dot2c_f32_bf16: head dim 64 2-3 % of the launch, 128 nothing by itself.
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16)((((lane >> 4) ^ (lane >> 2)) & 1) == 0 ? 1.f : 0.f);
  asm volatile("" : "+v"(ones));
  // -m_run, sixteen times: what a score block starts from.  (One more k-step with the constant 1 on the key side needs no registers, but
  // is 2 of 34 matrix instructions of a tile at head dim 128, 2 of 18 at 64: 1-2 % of the launch.)
  f32x16 cm;
#pragma unroll
  for (int r = 0; r < 16; ++r) cm[r] = 0.f;

  // Key and value tiles go from global memory straight into LDS, 1 KB (RPI rows) per
  // instruction: lane i fills bytes 16 i .. 16 i + 15 of the instruction's span, so the chunk
  // permutation is applied on the global side.
  const unsigned ldb = (unsigned)(ld * 2);
  const int lrow = lane / CH, slot = lane % CH;
  unsigned koff[NPAR], voff[NPAR];
#pragma unroll
  for (int par = 0; par < NPAR; ++par) {
    const int r16 = ((RPI * par) & 15) + lrow;  // row of the tile, modulo the swizzle period
    koff[par] = lrow * ldb + (H + (slot ^ k_swz<DH>(r16)) * 8) * 2;
    voff[par] = lrow * ldb + (2 * H + (slot ^ v_swz<DH>(r16)) * 8) * 2;
  }
  auto issue = [&](int k0, int buf) {
    const unsigned kdst = (unsigned)(uintptr_t)BR_LPTR(sK[buf]) + wv * LPW * 1024;
    const unsigned vdst = (unsigned)(uintptr_t)BR_LPTR(sV[buf]) + wv * LPW * 1024;
    if (k0 + KV_TILE <= L) {
      const char* blk = uniform_ptr(reinterpret_cast<const char*>(base) + (size_t)(k0 + wv * LPW * RPI) * ldb);
#pragma unroll
      for (int t = 0; t < LPW; ++t) {
        const char* src = blk + (size_t)t * RPI * ldb;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(kdst + t * 1024), "v"(koff[t % NPAR]), "s"(src) : "memory", "m0");
      }
#pragma unroll
      for (int t = 0; t < LPW; ++t) {
        const char* src = blk + (size_t)t * RPI * ldb;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(vdst + t * 1024), "v"(voff[t % NPAR]), "s"(src) : "memory", "m0");
      }
    } else {  // ragged last tile: rows past the end read the last key (their scores are masked)
      const char* blk = uniform_ptr(reinterpret_cast<const char*>(base));
#pragma unroll
      for (int t = 0; t < LPW; ++t) {
        const int row = (wv * LPW + t) * RPI + lrow;
        const unsigned off = (unsigned)min(k0 + row, L - 1) * ldb + (H + (slot ^ k_swz<DH>(row)) * 8) * 2;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(kdst + t * 1024), "v"(off), "s"(blk) : "memory", "m0");
      }
#pragma unroll
      for (int t = 0; t < LPW; ++t) {
        const int row = (wv * LPW + t) * RPI + lrow;
        const unsigned off = (unsigned)min(k0 + row, L - 1) * ldb + (2 * H + (slot ^ v_swz<DH>(row)) * 8) * 2;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(vdst + t * 1024), "v"(off), "s"(blk) : "memory", "m0");
      }
    }
  };

  // transposed reads of V: in a group of 16 lanes, lane 4 r + q supplies the 8 bytes at
  // (key K0 + r, d0 + 4 q .. 4 q + 3) and lane j receives (keys K0 .. K0 + 3, d0 + j)
  const int jj = lane & 15, g1 = (lane >> 4) & 1;
  const int vrow = 4 * lh + (jj >> 2);  // row within a group of 8 keys
  unsigned vaddr[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    const int chunk = d * 4 + 2 * g1 + ((jj & 3) >> 1);
    vaddr[d] = vrow * ROW_B + (chunk ^ v_swz<DH>(vrow)) * 16 + 8 * (jj & 1);
  }

  // Two LDS buffers, one barrier per tile: the next tile is fetched while the current one is
  // multiplied.  Every iteration issues the same number of fetches (the last one fetches its
  // own tile again, into the idle buffer), so the wait below is exact.
  const int nkv = (L + KV_TILE - 1) / KV_TILE;
  issue(0, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // Pin the query fragments in registers here; left alone, the compiler sinks their loads
  // into the loop.
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));
  // One key tile.  NKB: 32-key blocks of the tile that hold any key at all (2, or 1 in a short
  // last tile); MASK: the tile runs past the end of the sequence.  Only the last tile of a
  // ragged sequence is compiled with masking, so the loop over full tiles carries none of it.
  // BUF: the LDS buffer of the tile (it & 1) as a constant, so that fragment addresses are a
  // loop-invariant per-lane register plus an immediate.
  auto tile = [&](int it, auto NKBc, auto MASKc, auto BUFc) {
    constexpr int NKB = decltype(NKBc)::value;
    constexpr bool MASK = decltype(MASKc)::value;
    constexpr int buf = decltype(BUFc)::value;
    const int k0 = it * KV_TILE;
    // the other buffer was last read one tile ago, before the previous barrier
    issue(min(it + 1, nkv - 1) * KV_TILE, buf ^ 1);

    // S^T tile minus the reference: s[kb][r] = score of key k0 + 32 kb + 8 (r/4) + 4 lh + r%4 for query
    // l32, less m_run of that query, from which the accumulators start.
    f32x16 s[2];
    auto scores = [&]() __attribute__((always_inline)) {
      if constexpr (RA == 0) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
          s[kb] = cm;
          const int row = kb * 32 + l32;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const int c = ks * 2 + lh;
            const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&sK[buf][(row * CH + (c ^ k_swz<DH>(row))) * 16]);
            s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[kb], 0, 0, 0);
          }
        }
      } else {
        constexpr int N = NKB * KS;
        auto read_k = [&](int i) __attribute__((always_inline)) {
          const int row = (i / KS) * 32 + l32, c = (i % KS) * 2 + lh;
          return *reinterpret_cast<const bf16x8*>(&sK[buf][(row * CH + (c ^ k_swz<DH>(row))) * 16]);
        };
        bf16x8 kf[RA + 1];
#pragma unroll
        for (int i = 0; i < RA && i < N; ++i) kf[i] = read_k(i);
        static_for<N>([&](auto Ic) __attribute__((always_inline)) {
          constexpr int i = decltype(Ic)::value;
          if (i + RA < N) kf[(i + RA) % (RA + 1)] = read_k(i + RA);
          __builtin_amdgcn_sched_barrier(0);
          s[i / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i % (RA + 1)], qf[i % KS], i % KS == 0 ? cm : s[i / KS], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        });
      }
      if (MASK) {  // keys past the end
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = k0 + kb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
            if (key >= L) s[kb][r] = -INFINITY;
          }
      }
    };
    // p = 2^(s) (scores already in units of log2 e / sqrt(d)) or 2^(s scale): rounded to bf16 as the
    // column operand of the second product, step 2 kb + j; l_tile = the query's sum of the rounded values
    // (what that product sums), in both of its lanes.
    bf16x8 pf[2 * NKB];
    float l_tile;
    auto probabilities = [&]() __attribute__((always_inline)) {
      f32x4 lt = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < 2 * NKB; ++st) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = s[st >> 1][8 * (st & 1) + e];
          pf[st][e] = (bf16)__builtin_amdgcn_exp2f(PRE ? x : x * scale_log2);
        }
        lt = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[st], lt, 0, 0, 0);
      }
      l_tile = lt[0];
    };
    // Softmax does not care which reference m is subtracted as long as numerator and denominator use
    // the same one; here it is whatever the query's running maximum was when it last had to move.
    // It has to move only when a probability would leave the comfortable range, and since
    // probabilities are positive that shows in the row sum the kernel forms anyway: no maximum is
    // taken on the way.  When some query's sum of 64 probabilities passes 2^11 (or is not a number:
    // overflow), the scores are formed once more, the reference follows the maximum (rounded to bf16;
    // the accumulators are rescaled, 1 + DH/2 multiplications per lane) and the probabilities are taken
    // again.  With an exact running maximum nearly every tile of a sequence rescales, and maximum,
    // scale-and-subtract and rescale were half of the kernel's vector instructions -- which on this chip
    // are not hidden behind the matrix instructions.  A wave's first tile has no reference yet and goes
    // there at once (512 workgroups of 93 tokens 8.5 -> 7.9 us, a lone one of 64 tokens 4.45 -> 4.2).
    if (it != 0) {
      scores();
      probabilities();
    }
    if (it == 0 || __builtin_amdgcn_ballot_w64(!(l_tile <= 2048.f)) != 0) {
      scores();
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = __builtin_elementwise_maximum(mx, s[kb][r]);
      mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32, 64));
      float m_new = (float)(bf16)(m_run + (it == 0 ? mx : fmaxf(mx, 0.f)));
      float delta = m_new - m_run;
      // A query with a probability that is not finite (itself or a key it meets is not, or no key of a first tile scores above -inf) has
      // no result.  Zero times that is not zero, so its probabilities stay out of the sums it shares an instruction for.
      const bool lost = !((PRE ? mx - delta : (mx - delta) * scale_log2) <= 127.f);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(lost) != 0, 0)) {
        m_new = lost ? m_run : m_new;
        delta = lost ? 0.f : delta;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) s[kb][r] = lost ? -INFINITY : s[kb][r];
      }
      if (it != 0) {
        const float alpha = __builtin_amdgcn_exp2f(PRE ? -delta : -delta * scale_log2);
        l_run *= alpha;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
      }
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[kb][r] -= delta;
      m_run = m_new;
#pragma unroll
      for (int r = 0; r < 16; ++r) cm[r] = -m_new;
      asm volatile("" : "+v"(cm));
      probabilities();
      l_tile = lost ? __builtin_nanf("") : l_tile;
    }
    l_run += l_tile;

    // O^T += V^T P^T; k-slot (lh, e) of step (kb, j) is key 32 kb + 16 j + 8 (e/4) + 4 lh + e%4
    const char __attribute__((address_space(3)))* vt = (const char __attribute__((address_space(3)))*)BR_LPTR(sV[buf]);
    if constexpr (RA == 0) {
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
          for (int d = 0; d < DB; ++d) {
            const auto* p0 = vt + vaddr[d] + (kb * 32 + j * 16) * ROW_B;
            const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p0);
            const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * ROW_B));
            union { s16x4 s[2]; bf16x8 v; } u;
            u.s[0] = v0;
            u.s[1] = v1;
            o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u.v, pf[2 * kb + j], o[d], 0, 0, 0);
          }
        }
    } else {
      constexpr int N = 2 * NKB * DB;
      auto read_v = [&](int i) __attribute__((always_inline)) {
        const int st = i / DB, d = i % DB;  // step st = 2 kb + j covers keys 16 st .. 16 st + 15
        const auto* p0 = vt + vaddr[d] + st * 16 * ROW_B;
        union { s16x4 s[2]; bf16x8 v; } u;
        u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p0);
        u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * ROW_B));
        return u.v;
      };
      bf16x8 vf[RA + 1];
#pragma unroll
      for (int i = 0; i < RA && i < N; ++i) vf[i] = read_v(i);
      static_for<N>([&](auto Ic) __attribute__((always_inline)) {
        constexpr int i = decltype(Ic)::value;
        if (i + RA < N) vf[(i + RA) % (RA + 1)] = read_v(i + RA);
        __builtin_amdgcn_sched_barrier(0);
        o[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[i % (RA + 1)], pf[i / DB], o[i % DB], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    // the next tile has landed in this wave's share of the other buffer; after the barrier, in all of it
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  using K1 = std::integral_constant<int, 1>;
  using K2 = std::integral_constant<int, 2>;
  const int nfull = L / KV_TILE;
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  if (active) {
    int it = 0;
    for (; it + 2 <= nfull; it += 2) {
      tile(it, K2{}, std::false_type{}, B0{});
      tile(it + 1, K2{}, std::false_type{}, B1{});
    }
    if (it < nfull) tile(it, K2{}, std::false_type{}, B0{});
    if (nfull < nkv) {
      const bool one = L - nfull * KV_TILE <= 32;
      if (nfull & 1) {
        if (one) tile(nfull, K1{}, std::true_type{}, B1{});
        else tile(nfull, K2{}, std::true_type{}, B1{});
      } else {
        if (one) tile(nfull, K1{}, std::true_type{}, B0{});
        else tile(nfull, K2{}, std::true_type{}, B0{});
      }
    }
  } else {
    // a wave whose 32 queries all lie past the end only keeps up its share of the tile traffic
    for (int it = 0; it < nkv; ++it) {
      issue(min(it + 1, nkv - 1) * KV_TILE, (it & 1) ^ 1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
  }
  const float inv = 1.f / l_run;
  if (qi < L) {
    bf16* orow = out + ((size_t)b * L + qi) * H + (size_t)h * DH;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 v = {(bf16)(o[d][4 * g] * inv), (bf16)(o[d][4 * g + 1] * inv), (bf16)(o[d][4 * g + 2] * inv),
                    (bf16)(o[d][4 * g + 3] * inv)};
        *reinterpret_cast<bf16x4*>(orow + d * 32 + g * 8 + lh * 4) = v;
      }
  }
}

// Head dim 64, pipelined by one key tile: the probabilities of a tile are taken between the matrix instructions of the next tile's scores.
// What bounds it, in cycles of a wave and tile (64 keys, 32 queries): 576 of matrix instructions, as many of the vector ALU (32 v_exp_f32 of
// 16 cycles each, 16 conversions), 700 and more of LDS reads shared by four waves.  A wave alone on its SIMD takes 560 for the first half of
// an iteration and 430 for the second; in the order of the kernel above, with tile loads that branch for the ragged tile, 1800.  At full
// load it is the power limit that binds, and the second score tile leaves room for two waves per SIMD only.  Head dim 64, above ->
// here: 144 workgroups of 1101 tokens 15.7 -> 13.1 us, 288 21.3 -> 19.3, 272 of 2100 34.7 -> 32.2, 376 of 6000 91.7 -> 85.0; where the
// first is the faster one: attention_pipelined.  Inside a network, where the rows come from the product before, the 144 take 18.3 -> 14 us, 17 with two buffers
// of LDS instead of four.  (At head dim 128 it does not fit 256 registers: 1068 TFLOP/s at 4608 tokens, 1168 above.)
template <int DH, bool PRE, bool WARM>
__global__ __launch_bounds__(256, 2) void attn_bf16_pipe_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ out, int L,
                                                           int H, int NH, int n_pairs, int grouped, float scale_log2, Warm<WARM> warm) {
  constexpr int CH = DH / 8;    // 16-byte chunks per K row
  constexpr int KS = DH / 16;   // MFMA k-steps of the score product
  constexpr int DB = DH / 32;   // 32-row blocks of O^T
  constexpr int RPI = 64 / CH;              // rows covered by one 1 KB load
  constexpr int LPW = KV_TILE / RPI / 4;    // loads per wave, tile and operand
  constexpr int ROW_B = CH * 16;            // bytes per row
  constexpr int TILE_B = KV_TILE * ROW_B;
  // Operand fragments, keys and values in turn, pass through a ring of FR and are read from LDS RA matrix instructions ahead.
  constexpr int FR = 8, RA = 4;
  constexpr int NB = 4;  // LDS buffers of the keys and of the values
  __shared__ __attribute__((aligned(1024))) char sK[NB][TILE_B];
  __shared__ __attribute__((aligned(1024))) char sV[NB][TILE_B];

  int pair, qt;
  if (!attn_tile(warm, (L + 127) / 128, n_pairs, grouped, &pair, &qt)) return;
  const int b = pair / NH, h = pair - b * NH;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t ld = (size_t)3 * H;
  const bf16* base = qkv + (size_t)b * L * ld + (size_t)h * DH;
  const int qi = qt * 128 + wv * 32 + l32;
  const int qc = min(qi, L - 1);
  const bool active = qt * 128 + wv * 32 < L;  // (uniform over the wave)

  bf16x8 qf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    qf[ks] = *reinterpret_cast<const bf16x8*>(base + (size_t)qc * ld + ks * 16 + lh * 8);

  f32x16 o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  float m_run = 0.f, l_run = 0.f;  // reference (a bf16 value) and row sum of the probabilities taken against it
  // Row sums on the matrix pipe: v_mfma_f32_16x16x32 takes the registers of a probability step (lanes 0..15 / 16..31: keys 0..7 of
  // queries 0..15 / 16..31, lanes 32..63 their keys 8..15) as sixteen columns of four k-groups, so the even groups belong to
  // one half of the queries, the odd ones to the other; the row side is 1 where a row's result lands in that half's lanes.  Sixteen
  // cycles of the matrix pipe a step instead of four v_dot2c_f32_bf16: head dim 64 2-3 % of the launch, 128 nothing by itself.
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16)((((lane >> 4) ^ (lane >> 2)) & 1) == 0 ? 1.f : 0.f);
  asm volatile("" : "+v"(ones));
  // -m_run, sixteen times: what a score block starts from.  (One more k-step with the constant 1 on the key side needs no registers, but
  // is 2 of 34 matrix instructions of a tile at head dim 128, 2 of 18 at 64: 1-2 % of the launch.)
  f32x16 cm;
#pragma unroll
  for (int r = 0; r < 16; ++r) cm[r] = 0.f;

  // Key and value tiles go from global memory straight into LDS, 1 KB (RPI rows) per instruction: lane i fills bytes 16 i .. 16 i + 15 of
  // the instruction's span, so the chunk permutation is applied on the global side.  Buffer loads whose bound is the end of the sample:
  // rows past it arrive as zeros (their scores are masked), so a load is an instruction and an addition, without branches or scalar address
  // arithmetic, which cost a wave 150 cycles a load.
  const unsigned ldb = (unsigned)(ld * 2);
  const int lrow = lane / CH, slot = lane % CH;
  unsigned koff[LPW], voff[LPW];  // byte offset of the next tile's rows
#pragma unroll
  for (int t = 0; t < LPW; ++t) {
    const int row = (wv * LPW + t) * RPI + lrow;
    koff[t] = row * ldb + (H + (slot ^ k_swz<DH>(row)) * 8) * 2;
    voff[t] = row * ldb + (2 * H + (slot ^ v_swz<DH>(row)) * 8) * 2;
  }
  const u32x4 rows = sample_rows(base, (unsigned)(L - 1) * ldb + (2 * H + DH) * 2);
  const unsigned lds_k = (unsigned)(uintptr_t)BR_LPTR(sK[0]) + wv * LPW * 1024, lds_v = (unsigned)(uintptr_t)BR_LPTR(sV[0]) + wv * LPW * 1024;
  auto load_k = [&](int t, int buf) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_k + buf * TILE_B + t * 1024), "v"(koff[t]), "s"(rows) : "memory", "m0");
    koff[t] = __builtin_elementwise_add_sat(koff[t], KV_TILE * ldb);
  };
  auto load_v = [&](int t, int buf) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_v + buf * TILE_B + t * 1024), "v"(voff[t]), "s"(rows) : "memory", "m0");
    voff[t] = __builtin_elementwise_add_sat(voff[t], KV_TILE * ldb);
  };
  const int nkv = (L + KV_TILE - 1) / KV_TILE;
  auto load_keys = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < LPW; ++t) load_k(t, buf);
  };
  auto load_values = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < LPW; ++t) load_v(t, buf);
  };

  // transposed reads of V: in a group of 16 lanes, lane 4 r + q supplies the 8 bytes at
  // (key K0 + r, d0 + 4 q .. 4 q + 3) and lane j receives (keys K0 .. K0 + 3, d0 + j)
  const int jj = lane & 15, g1 = (lane >> 4) & 1;
  const int vrow = 4 * lh + (jj >> 2);  // row within a group of 8 keys
  unsigned vaddr[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    const int chunk = d * 4 + 2 * g1 + ((jj & 3) >> 1);
    vaddr[d] = vrow * ROW_B + (chunk ^ v_swz<DH>(vrow)) * 16 + 8 * (jj & 1);
  }

  // The loop is pipelined by one tile.  Iteration `it` finds the scores of its tile in registers and has two halves: the score product of
  // tile it + 1, with the probabilities of tile it between its matrix instructions, and the product of those with the values of tile it.
  // Between the halves lies the one barrier: the keys of tile it + 2 and the values of tile it + 1 have landed and every wave is done with
  // the keys of it + 1 and the values of it - 1, whose buffers take those of it + 5 and it + 3 during the second half.  (Rows that the
  // product before has just written take 2000 cycles and more to arrive.)  Every wave issues the same loads in the same order, so the
  // keys of it + 3 and it + 4 and the values of it + 2 may be under way at the barrier.
  load_keys(0);
  load_keys(1);
  load_values(0);
  load_keys(2);
  load_values(1);
  load_keys(3);
  load_values(2);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(5 * LPW) : "memory");
  __syncthreads();
  if (!active) {  // a wave whose 32 queries all lie past the end only keeps up its share of the tile traffic
    __syncthreads();
    load_keys(0);
    for (int it = 0; it < nkv; ++it) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * LPW) : "memory");
      __syncthreads();
      load_values((it + 3) & (NB - 1));
      load_keys((it + 5) & (NB - 1));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return;
  }
  // Pin the query fragments in registers here; left alone, the compiler sinks their loads
  // into the loop.
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));

  constexpr int NQK = 2 * KS;  // matrix instructions of a score tile
  f32x16 s[2][2];              // [tile parity][32-key block]
  bf16x8 fr[FR], pf[4];
  // Score tile minus the reference: s[.][kb][r] = score of key 32 kb + 8 (r/4) + 4 lh + r%4 for query l32, less m_run of that query, from
  // which the accumulators start.
  auto read_k = [&](int buf, int i) __attribute__((always_inline)) {
    const int row = (i / KS) * 32 + l32, c = (i % KS) * 2 + lh;
    return *reinterpret_cast<const bf16x8*>(&sK[0][0] + buf * TILE_B + (row * CH + (c ^ k_swz<DH>(row))) * 16);
  };
  auto score_step = [&](auto Ic, auto Sc, int buf) __attribute__((always_inline)) {
    constexpr int i = decltype(Ic)::value, S = decltype(Sc)::value;
    if constexpr (i + RA < NQK) fr[(i + RA) % FR] = read_k(buf, i + RA);
    s[S][i / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % FR], qf[i % KS], i % KS == 0 ? cm : s[S][i / KS], 0, 0, 0);
  };
  auto scores = [&](auto Sc, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < RA; ++i) fr[i] = read_k(buf, i);
    static_for<NQK>([&](auto Ic) __attribute__((always_inline)) {
      score_step(Ic, Sc, buf);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // p = 2^(s) (scores already in units of log2 e / sqrt(d)) or 2^(s scale): rounded to bf16 as the column operand of the second product,
  // step 2 kb + j; l_tile = the query's sum of the rounded values (what that product sums), in both of its lanes.
  f32x4 lt;
  auto prob = [&](auto Sc, int at, int n) __attribute__((always_inline)) {  // elements at .. at + n - 1 of the tile's 32
#pragma unroll
    for (int e = at; e < at + n; ++e) {
      const float x = s[decltype(Sc)::value][e >> 4][e & 15];
      pf[e >> 3][e & 7] = (bf16)__builtin_amdgcn_exp2f(PRE ? x : x * scale_log2);
    }
  };
  auto row_sum = [&](int st) __attribute__((always_inline)) { lt = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[st], lt, 0, 0, 0); };
  // Moves the reference to the running maximum of the tile in s[S] and takes the tile's scores down to it.
  auto settle = [&](auto Sc, auto NKBc, auto FIRSTc) __attribute__((always_inline)) {
    constexpr int S = decltype(Sc)::value, NKB = decltype(NKBc)::value;
    constexpr bool first = decltype(FIRSTc)::value;
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = __builtin_elementwise_maximum(mx, s[S][kb][r]);
    mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32, 64));
    float m_new = (float)(bf16)(m_run + (first ? mx : fmaxf(mx, 0.f)));
    float delta = m_new - m_run;
    // A query with a probability that is not finite (itself or a key it meets is not, or no key of a first tile scores above -inf) has
    // no result.  Zero times that is not zero, so its probabilities stay out of the sums it shares an instruction for.
    const bool lost = !((PRE ? mx - delta : (mx - delta) * scale_log2) <= 127.f);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(lost) != 0, 0)) {
      m_new = lost ? m_run : m_new;
      delta = lost ? 0.f : delta;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[S][kb][r] = lost ? -INFINITY : s[S][kb][r];
    }
    if (!first) {
      const float alpha = __builtin_amdgcn_exp2f(PRE ? -delta : -delta * scale_log2);
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
    }
    l_run = lost ? __builtin_nanf("") : l_run;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[S][kb][r] -= delta;
    m_run = m_new;
#pragma unroll
    for (int r = 0; r < 16; ++r) cm[r] = -m_new;
    asm volatile("" : "+v"(cm));
  };
  auto mask = [&](int it, auto Sc, auto NKBc) __attribute__((always_inline)) {  // keys past the end
#pragma unroll
    for (int kb = 0; kb < decltype(NKBc)::value; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (it * KV_TILE + kb * 32 + 8 * (r >> 2) + 4 * lh + (r & 3) >= L) s[decltype(Sc)::value][kb][r] = -INFINITY;
  };
  // One iteration.  P: parity of `it`, as a constant for the registers of the scores; NKB: 32-key blocks of the tile that hold any key at all (2,
  // or 1 in a short last tile); MASK: the tile runs past the end of the sequence; NEXT: there is a tile it + 1.
  auto tile = [&](int it, auto Pc, auto NKBc, auto MASKc, auto NEXTc) __attribute__((always_inline)) {
    constexpr int P = decltype(Pc)::value, NKB = decltype(NKBc)::value;
    constexpr bool NEXT = decltype(NEXTc)::value, MASK = decltype(MASKc)::value;
    using S0 = std::integral_constant<int, P>;      // score registers of tile it
    using S1 = std::integral_constant<int, P ^ 1>;  // and of tile it + 1
    const int b0 = it & (NB - 1), b1 = (it + 1) & (NB - 1), b2 = (it + 2) & (NB - 1), b3 = (it + 3) & (NB - 1);
    if constexpr (MASK) {
      if (it != 0) mask(it, S0{}, NKBc);  // (the first tile is, before its maximum is taken)
    }
    lt = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (NEXT) {
      constexpr int PER = 32 / NQK;  // probabilities behind a matrix instruction
      static_for<NQK>([&](auto Ic) __attribute__((always_inline)) {
        constexpr int i = decltype(Ic)::value;
        score_step(Ic, S1{}, b1);
        if constexpr (i * PER % 8 == 0 && i > 0) row_sum(i * PER / 8 - 1);
        prob(S0{}, i * PER, PER);
        __builtin_amdgcn_sched_barrier(0);
      });
      row_sum(3);
    } else {
#pragma unroll
      for (int st = 0; st < 2 * NKB; ++st) {
        prob(S0{}, 8 * st, 8);
        row_sum(st);
      }
    }
    // Softmax does not care which reference m is subtracted as long as numerator and denominator use
    // the same one; here it is whatever the query's running maximum was when it last had to move.
    // It has to move only when a probability would leave the comfortable range, and since
    // probabilities are positive that shows in the row sum the kernel forms anyway: no maximum is
    // taken on the way.  When some query's sum of 64 probabilities passes 2^11 (or is not a number:
    // overflow), the reference follows the maximum (rounded to bf16; the accumulators are rescaled,
    // 1 + DH/2 multiplications per lane), the probabilities are taken again and the next tile's scores, which started from the old
    // reference, are formed once more.  With an exact running maximum nearly every tile of a sequence rescales, and maximum,
    // scale-and-subtract and rescale were half of the kernel's vector instructions.
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(lt[0] <= 2048.f)) != 0, 0)) {
      settle(S0{}, NKBc, std::false_type{});
      lt = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = 0; st < 2 * NKB; ++st) {
        prob(S0{}, 8 * st, 8);
        row_sum(st);
      }
      if constexpr (NEXT) scores(S1{}, b1);
    }
    l_run += lt[0];
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * LPW) : "memory");
    __syncthreads();

    // O^T += V^T P^T; k-slot (lh, e) of step (kb, j) is key 32 kb + 16 j + 8 (e/4) + 4 lh + e%4
    const char __attribute__((address_space(3)))* vt = (const char __attribute__((address_space(3)))*)BR_LPTR(sV[0]) + b0 * TILE_B;
    constexpr int N = 2 * NKB * DB;
    auto read_v = [&](int i) __attribute__((always_inline)) {
      const int st = i / DB, d = i % DB;  // step st = 2 kb + j covers keys 16 st .. 16 st + 15
      const auto* p0 = vt + vaddr[d] + st * 16 * ROW_B;
      union { s16x4 s[2]; bf16x8 v; } u;
      u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p0);
      u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p0 + 8 * ROW_B));
      return u.v;
    };
#pragma unroll
    for (int i = 0; i < RA && i < N; ++i) fr[i] = read_v(i);
    static_for<N>([&](auto Ic) __attribute__((always_inline)) {
      constexpr int i = decltype(Ic)::value;
      if constexpr (i + RA < N) fr[(i + RA) % FR] = read_v(i + RA);
      else if constexpr (NEXT) fr[i + RA - N] = read_k(b2, i + RA - N);  // (of tile it + 2; where there is none, nobody uses it)
      __builtin_amdgcn_sched_barrier(0);
      o[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[i % FR], pf[i / DB], o[i % DB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (NEXT && i < 2 * LPW) {
        if constexpr (i < LPW) load_v(i, b3);
        else load_k(i - LPW, b1);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
  };
  using K1 = std::integral_constant<int, 1>;
  using K2 = std::integral_constant<int, 2>;
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using YES = std::true_type;
  using NO = std::false_type;
  const int left = L - (nkv - 1) * KV_TILE;  // keys of the last tile
  scores(P0{}, 0);
  __syncthreads();  // every wave is done with the first keys
  load_keys(0);
  if (nkv == 1) {
    if (left <= 32) {
      mask(0, P0{}, K1{});
      settle(P0{}, K1{}, YES{});
    } else {
      if (left < KV_TILE) mask(0, P0{}, K2{});
      settle(P0{}, K2{}, YES{});
    }
  } else {
    settle(P0{}, K2{}, YES{});
#pragma unroll
    for (int i = 0; i < RA; ++i) fr[i] = read_k(1, i);
  }
  int it = 0;
  for (; it + 2 < nkv; it += 2) {
    tile(it, P0{}, K2{}, NO{}, YES{});
    tile(it + 1, P1{}, K2{}, NO{}, YES{});
  }
  auto last = [&](auto Pc) __attribute__((always_inline)) {
    if (left == KV_TILE) tile(nkv - 1, Pc, K2{}, NO{}, NO{});
    else if (left > 32) tile(nkv - 1, Pc, K2{}, YES{}, NO{});
    else tile(nkv - 1, Pc, K1{}, YES{}, NO{});
  };
  if (it + 2 == nkv) {
    tile(it, P0{}, K2{}, NO{}, YES{});
    last(P1{});
  } else {
    last(P0{});
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the end
  const float inv = 1.f / l_run;
  if (qi < L) {
    bf16* orow = out + ((size_t)b * L + qi) * H + (size_t)h * DH;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 v = {(bf16)(o[d][4 * g] * inv), (bf16)(o[d][4 * g + 1] * inv), (bf16)(o[d][4 * g + 2] * inv),
                    (bf16)(o[d][4 * g + 3] * inv)};
        *reinterpret_cast<bf16x4*>(orow + d * 32 + g * 8 + lh * 4) = v;
      }
  }
}


br_status launch_attention_bf16(const bf16* qkv, bf16* out, int B, int L, int NH, int DH, int q_prescaled, const WarmRows& next, hipStream_t st) {
  BR_REQUIRE(L >= 1, BR_EINVAL, "attention: empty sequence");
  // the ragged last tile addresses its rows with 32-bit byte offsets from the sample's first row
  BR_REQUIRE((unsigned long long)L * 3ull * NH * DH * 2ull < (1ull << 32), BR_ESHAPE,
             "attention: one sample's QKV rows exceed 4 GiB");
  const long long n_pairs = (long long)B * NH;
  const int grouped = n_pairs >= 32 ? 1 : 0;
  const long long n_blocks = (grouped ? (n_pairs + 7) / 8 * 8 : n_pairs) * cdiv(L, 128);
  BR_REQUIRE(n_blocks <= 0x7FFFFFFFLL, BR_ESHAPE, "attention: too many workgroups for one launch");
  // Where the launch leaves compute units idle: as much of the list as they read meanwhile (see warm_rows).
  const int n_cu = device_cu_count();
  WarmRows warm = next;
  warm.blocks = next.n16[0] > 0 && q_prescaled ? (n_cu - (int)std::min<long long>(n_blocks, n_cu)) / 8 * 8 : 0;
  unsigned budget = (unsigned)(WARM_BYTES_PER_TILE / 16 * (cdiv(L, KV_TILE) + 4) / 256 * warm.blocks);
  size_t bytes = 0;
  for (const unsigned n : next.n16) bytes += (size_t)n * 16;
  if (warm.blocks < 32 || !rule::read_ahead((size_t)budget * 16, bytes)) warm.blocks = 0;  // (at head dim 64 fewer workgroups than units: the pipelined loop)
  for (unsigned& n : warm.n16) {
    n = std::min(n, budget);
    budget -= n;
  }
  dim3 g((unsigned)n_blocks + warm.blocks), blk(256);
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)DH));
  const int H = NH * DH;
  ProfScope ps(st, PROF_ATTN + DH, 4.0 * B * (double)L * L * H);
  auto go = [&](auto kernel, const auto& w) { hipLaunchKernelGGL(kernel, g, blk, 0, st, qkv, out, L, H, NH, (int)n_pairs, grouped, scale_log2, w); };
  const bool pipe = rule::attention_pipelined(DH, L, n_blocks, n_cu);  // bit for bit the same either way
  if (warm.blocks > 0 && pipe) go(attn_bf16_pipe_kernel<64, true, true>, warm);
  else if (warm.blocks > 0 && DH == 128) go(attn_bf16_kernel<128, true, true>, warm);
  else if (pipe && q_prescaled) go(attn_bf16_pipe_kernel<64, true, false>, NoWarm{});
  else if (pipe) go(attn_bf16_pipe_kernel<64, false, false>, NoWarm{});
  else if (DH == 64 && q_prescaled) go(attn_bf16_kernel<64, true, false>, NoWarm{});
  else if (DH == 64) go(attn_bf16_kernel<64, false, false>, NoWarm{});
  else if (DH == 128 && q_prescaled) go(attn_bf16_kernel<128, true, false>, NoWarm{});
  else if (DH == 128) go(attn_bf16_kernel<128, false, false>, NoWarm{});
  else return fail(BR_ESHAPE, "bf16 attention: head dim must be 64 or 128");
  BR_LAUNCH_CHECK();
  return BR_OK;
}

}  // namespace br
