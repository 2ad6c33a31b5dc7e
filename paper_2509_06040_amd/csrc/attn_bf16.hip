// bf16 flash attention on the gfx950 matrix cores: softmax(Q K^T / sqrt(d)) V over all L tokens of a sample.  A workgroup takes 128 or (head dim 128) 256
// queries of a (sample, head) pair, 32 a wave, over key/value tiles of 64 keys in LDS.
//
// Scores are computed transposed, S^T = K Q^T, in 16x16x32 matrix instructions: a lane then holds four keys of ONE query per block
// of 16 keys (the others sit in the lanes 16, 32 and 48 further), so the reference / sum / rescale of the online softmax are per-lane
// scalars, and the exponentiated blocks of 32 keys are, register for register, the column operand of O^T = V^T P^T, whose contraction order
// is permuted to match: k-slot (quarter g of the lanes, e) is key 16 (e / 4) + 4 g + e % 4.  The row sums are a matrix instruction with
// a row side of ones on the same registers.
//
// The loop is woven from three half tiles of 32 keys: between one another stand the matrix instructions of the scores of half j + 1 and of
// the product of half j - 1 with its values, and the exponentials of half j, which depend on neither.  What bounds it: the matrix pipe
// (544 cycles a wave and half tile at head dim 128) and, at head dim 64, the vector ALU as well (256 of exponentials and 32 of
// conversions beside 288).  One after the other, and in 32x32x16 instructions, which touch twice the accumulators for a product and draw more power, the two
// pipes took turns: 24 heads of 128, 4608 tokens, 8 samples 1780 us (1.16 PFLOP/s) -> 1585 (1.30); 12 heads of 32 768 tokens 5370 -> 4560
// (1.45); 16 heads of 64, 1101 tokens, 64 samples 368 -> 347 (0.92), 12 heads of 64, 4608 tokens, 8 samples 488 -> 445 (1.17).
//
// Both tiles travel from global memory straight into LDS (no registers, no vector instructions on the way), row-major as they lie in the QKV
// buffer, with their 16-byte chunks permuted per row so that fragment reads spread over the banks.  The row operand of the second product
// needs V transposed; the LDS transpose read delivers that: in a group of 16 lanes, lane 4 r + q supplies the address of 8 bytes (4 values
// of row r) and lane j receives element j of rows 0..3, so each lane ends up with four consecutive keys of its own channel.
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
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

constexpr int KV_TILE = 64;
constexpr float REF_LIMIT = 2048.f;  // a query's reference moves when its probabilities of a half tile add up to more
constexpr long long WARM_BYTES_PER_TILE = 2 << 20;  // what 256 idle compute units read while a workgroup takes a key tile

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
template <int NT>
static __device__ inline void warm_rows(const WarmRows& w) {
  const unsigned stride = w.blocks * NT;
#pragma unroll
  for (int r = 0; r < WarmRows::RANGES; ++r) {
    const u32x4* p = reinterpret_cast<const u32x4*>(w.p[r]);
    const unsigned n = w.n16[r];
    for (unsigned i = blockIdx.x * NT + threadIdx.x; i < n; i += 8 * stride) {
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

// The (sample, head) pair and the first query of a workgroup; false: none.
// Workgroups are dispatched round-robin over the 8 XCDs.  All query tiles of one
// (sample, head) read the same keys and values, so they are given to one XCD and run
// back to back there: K/V then come out of that XCD's L2 instead of being fetched 8 times.
// (With few pairs that would leave XCDs idle: then tiles are simply dealt out in order.)
//
// plan: bit 0: grouped so; bits 1..3: parts that a tile is cut into from tile bits 4.. on (of a die, if grouped), each with 16 queries a
// wave: the last round of tiles spreads over units that would be idle.  (12 heads of 33 272 tokens are 6.09 rounds of 256 queries on 256
// units: 5520 us, with the last 24 tiles in four parts 5010; 8 heads of 1101 tokens, 40 tiles, 28.6 -> 15.0.)
static __device__ __forceinline__ bool attn_tile(unsigned block, int nq, int n_pairs, int plan, int tile_rows, int* pair, int* q_first, int* parts) {
  const bool grouped = plan & 1;
  const int split = (plan >> 1) & 7, whole = plan >> 4;
  int t = grouped ? block >> 3 : block, sub = 0;
  *parts = 1;
  if (split > 1 && t >= whole) {
    sub = (t - whole) % split;
    t = whole + (t - whole) / split;
    *parts = split;
  }
  *pair = t / nq;
  *q_first = (t - *pair * nq) * tile_rows + sub * (tile_rows / *parts);
  if (grouped) *pair = *pair * 8 + (block & 7);
  return *pair < n_pairs;
}

// Slot permutations of the K and V tiles: 16-byte chunk c of row r sits in slot c ^ swz(r).
// The LDS has 64 banks of 4 bytes; a 16-byte read is served 16 lanes at a time and an 8-byte
// read 32 lanes at a time, conflict-free when those lanes cover all 256 bytes of a bank row.
//   K (ds_read_b128, lanes 0..15 = 16 consecutive rows at one chunk index): with 256-byte rows
//   the rows must land in 16 different slots, with 128-byte rows (two per bank row) row pairs in 8.
//   V (transposing 8-byte reads, 32 lanes = 8 consecutive rows x 2 consecutive chunks): with 256-byte rows
//   the eight rows take the eight pairs of slots, with 128-byte rows the four row pairs the four.
template <int DH>
__device__ inline int k_swz(int r) { return DH == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int DH>
__device__ inline int v_swz(int r) { return DH == 128 ? ((r & 7) << 1) : (((r >> 1) & 3) << 1); }

// 16 QB queries a wave (waves from `waves` on only help with the loads), from q_first on, of (sample, head) pair `pair`.
// NW waves, NB buffers of keys and of values.  SHORT: fewer key tiles than NB, all fetched at the start; else at least NB.
// PRE: the q third of the buffer already carries the factor log2(e) / sqrt(DH), as the network's QKV projection writes it; otherwise
// the exponent is scaled here, one multiplication per score.
template <int DH, int NW, int NB, int QB, bool SHORT, bool PRE>
static __device__ __forceinline__ void attn_queries(char* lds, const bf16* __restrict__ qkv, bf16* __restrict__ out, int L, int H, int NH, int pair,
                                                    int q_first, int waves, float scale_log2) {
  constexpr int CH = DH / 8;                // 16-byte chunks per K row
  constexpr int KS = DH / 32;               // k-steps of the score product
  constexpr int DB = DH / 16;               // 16-row blocks of O^T
  constexpr int RPI = 64 / CH;              // rows covered by one 1 KB load
  constexpr int LPW = KV_TILE / RPI / NW;   // loads per wave, tile and operand
  constexpr int ROW_B = CH * 16;            // bytes per row
  constexpr int TILE_B = KV_TILE * ROW_B;
  constexpr int FR = QB == 1 ? 8 : 4, RA = FR - 1;  // ring of operand fragments; read ahead
  constexpr int NS = 2 * DB;                // slots of a step (2 KS score blocks, DB value blocks)
  static_assert(2 * KS == DB && NS % FR == 0 && LPW >= 1 && 2 * LPW <= NS && NB >= 2, "");

  const int b = pair / NH, h = pair - b * NH;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t ld = (size_t)3 * H;
  const bf16* base = qkv + (size_t)b * L * ld + (size_t)h * DH;
  const int q0 = q_first + wv * (16 * QB);
  const bool active = wv < waves && q0 < L;  // (uniform over the wave)

  bf16x8 qf[QB][KS];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[qb][ks] = *reinterpret_cast<const bf16x8*>(base + (size_t)min(q0 + qb * 16 + l16, L - 1) * ld + ks * 32 + lq * 8);

  f32x4 o[DB][QB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) o[d][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[QB] = {}, l_run[QB] = {};  // reference (a bf16 value) and row sum of the probabilities taken against it
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.f;
  asm volatile("" : "+v"(ones));
  f32x4 cm[QB];  // -m_run, four times: what a score block starts from
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) cm[qb] = f32x4{0.f, 0.f, 0.f, 0.f};

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
    // (a row that does not exist: its product need not fit 32 bits)
    koff[t] = row < L ? row * ldb + (H + (slot ^ k_swz<DH>(row)) * 8) * 2 : 0xFFFFFFFFu;
    voff[t] = row < L ? row * ldb + (2 * H + (slot ^ v_swz<DH>(row)) * 8) * 2 : 0xFFFFFFFFu;
  }
  const u32x4 rows = sample_rows(base, (unsigned)(L - 1) * ldb + (2 * H + DH) * 2);
  const int nkv = (L + KV_TILE - 1) / KV_TILE;
  const int v_base = (SHORT ? nkv : NB) * TILE_B;
  const unsigned lds_k = (unsigned)(uintptr_t)BR_LPTR(lds) + wv * LPW * 1024, lds_v = lds_k + v_base;
  // buf: bytes of the buffer
  auto load_k = [&](int t, int buf) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_k + buf + t * 1024), "v"(koff[t]), "s"(rows) : "memory", "m0");
    koff[t] = __builtin_elementwise_add_sat(koff[t], KV_TILE * ldb);
  };
  auto load_v = [&](int t, int buf) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_v + buf + t * 1024), "v"(voff[t]), "s"(rows) : "memory", "m0");
    voff[t] = __builtin_elementwise_add_sat(voff[t], KV_TILE * ldb);
  };
  // addresses of this lane's fragments in buffer 0, first half
  unsigned kaddr[KS], vaddr[DB];
  static_for<KS>([&](auto Kc) __attribute__((always_inline)) {
    constexpr int ks = decltype(Kc)::value;
    kaddr[ks] = l16 * ROW_B + (((ks * 4 + lq) ^ k_swz<DH>(l16)) << 4);
  });
  const int vrow = 4 * lq + (l16 >> 2);
  static_for<DB>([&](auto Dc) __attribute__((always_inline)) {
    constexpr int d = decltype(Dc)::value;
    vaddr[d] = v_base + vrow * ROW_B + (((2 * d + ((l16 & 3) >> 1)) ^ v_swz<DH>(vrow)) << 4) + 8 * (l16 & 1);
  });

  auto fetch_k = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < LPW; ++t) load_k(t, buf);
  };
  auto fetch_v = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < LPW; ++t) load_v(t, buf);
  };
  if constexpr (!SHORT) {  // K 0, V 0, K 1, V 1, ... K NB - 1; the first two and V 0 now
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      fetch_k(i * TILE_B);
      if (i + 1 < NB) fetch_v(i * TILE_B);
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((2 * NB - 4) * LPW) : "memory");
  } else {
    for (int i = 0; i < nkv; ++i) {
      fetch_k(i * TILE_B);
      fetch_v(i * TILE_B);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();
  // The one barrier of a tile, in the middle of tile t: the keys of t + 2 and the values of t + 1 have landed, every wave is done with the keys of t
  // and the values of t - 1, whose buffers take those of t + NB and t + NB - 1 behind it.  What the first slots of the next step read
  // was there one barrier earlier, so that those reads need not wait for this one.  (Two buffers: the keys of t + 1 and the values of t have landed, and those
  // reads come behind it; one more barrier in front of the last tile, for its values.)
  auto turn = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NB == 2 ? 0 : 2 * (NB - 3) * LPW) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  if (!active) {  // a wave without queries only keeps up its share of the tile traffic
    if constexpr (!SHORT) {
      int b0 = 0;
      for (int t = 0; t + 1 < nkv; ++t) {
        turn();
        fetch_v((b0 == 0 ? NB * TILE_B : b0) - TILE_B);
        fetch_k(b0);
        b0 = b0 == (NB - 1) * TILE_B ? 0 : b0 + TILE_B;
      }
      if constexpr (NB == 2) turn();
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    return;
  }
  // Pin the query fragments in registers here; left alone, the compiler sinks their loads into the loop.
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[qb][ks]));

  typedef const char __attribute__((address_space(3)))* lptr;
  const lptr l0 = (lptr)BR_LPTR(lds);
  auto read_k = [&](int ks, int kb, int off) __attribute__((always_inline)) {  // off: bytes of buffer and half
    return *(const bf16x8 __attribute__((address_space(3)))*)(l0 + kaddr[ks] + (off + kb * 16 * ROW_B));
  };
  auto read_v = [&](int d, int off) __attribute__((always_inline)) {
    const lptr p = l0 + vaddr[d] + off;
    union { s16x4 s[2]; bf16x8 v; } u;
    u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p);
    u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 16 * ROW_B));
    return u.v;
  };
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  using YES = std::true_type;
  using NO = std::false_type;
  f32x4 s[2][2][QB];     // [parity of the half tile][block of 16 keys][block of 16 queries]
  bf16x8 pf[2][QB];      // [parity][block of queries]
  bf16x8 fr[FR];
  f32x4 lt[QB];
  auto mma = [](bf16x8 a, bf16x8 bb, f32x4 c) __attribute__((always_inline)) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bb, c, 0, 0, 0); };
  auto prob = [&](auto Pc, int e) __attribute__((always_inline)) {
    constexpr int P = decltype(Pc)::value;  // element e: block of keys, block of queries, key
    const int kb = e / (4 * QB), qb = (e >> 2) % QB, r = e & 3;
    const float x = s[P][kb][qb][r];
    pf[P][qb][kb * 4 + r] = (bf16)__builtin_amdgcn_exp2f(PRE ? x : x * scale_log2);
  };
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  auto row_sum = [&](auto Pc, int qb) __attribute__((always_inline)) { lt[qb] = mma(ones, pf[decltype(Pc)::value][qb], zero); };
  // Softmax does not care which reference m is subtracted as long as numerator and denominator use
  // the same one; here it is whatever the query's running maximum was when it last had to move.
  // It has to move only when a probability would leave the comfortable range, and since
  // probabilities are positive that shows in the row sum the kernel forms anyway: no maximum is
  // taken on the way.  When a query's sum of 32 probabilities passes the limit (or is not a number:
  // overflow), its reference follows the maximum (rounded to bf16; the accumulators are rescaled), the probabilities are
  // taken again and the next half's scores, which started from the old reference, are taken down to the new one.  With an exact running
  // maximum nearly every tile of a sequence rescales, and maximum, scale-and-subtract and rescale were half of the kernel's vector
  // instructions.  Each query moves for itself: its result does not depend on which queries share its wave.  (A query that is not
  // finite, or that some key scores +inf, has a NaN among its own sums and no other query's.)
  // A query's first reference (m_first) is its maximum over the first half tile with a key that scores above -inf.  Where that is not the very first one, for
  // some query of the wave, the halves behind are looked through once, with keys straight from memory, before the loop (which then meets
  // nothing but zeros until that half).  Without any such key there is no result: zero by zero.
  auto top = [&](auto Pc, int qb) __attribute__((always_inline)) {
    constexpr int P = decltype(Pc)::value;
    const f32x4 v = __builtin_elementwise_maximum(s[P][0][qb], s[P][1][qb]);
    float mx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(v[0], v[1]), __builtin_elementwise_maximum(v[2], v[3]));
    mx = __builtin_elementwise_maximum(mx, __shfl_xor(mx, 16, 64));
    return __builtin_elementwise_maximum(mx, __shfl_xor(mx, 32, 64));
  };
  float m_first[QB];
  auto settle = [&](auto Pc, bool first, bool next) __attribute__((always_inline)) {
    constexpr int P = decltype(Pc)::value;
    static_for<QB>([&](auto Qc) __attribute__((always_inline)) {
      constexpr int qb = decltype(Qc)::value;
      const float mx = first ? m_first[qb] : top(Pc, qb);
      const float m_new = first || !(lt[qb][0] <= REF_LIMIT) ? (float)(bf16)(m_run[qb] + (first ? mx : fmaxf(mx, 0.f))) : m_run[qb];
      const float delta = m_new - m_run[qb];
      if (!first) {
        const float alpha = __builtin_amdgcn_exp2f(PRE ? -delta : -delta * scale_log2);
        l_run[qb] *= alpha;
        static_for<DB>([&](auto Dc) __attribute__((always_inline)) { o[decltype(Dc)::value][qb] *= alpha; });
      }
      s[P][0][qb] -= delta;
      s[P][1][qb] -= delta;
      if (next) {
        s[P ^ 1][0][qb] -= delta;
        s[P ^ 1][1][qb] -= delta;
      }
      m_run[qb] = m_new;
      cm[qb] = f32x4{-m_new, -m_new, -m_new, -m_new};
      asm volatile("" : "+v"(cm[qb]));
    });
  };
  auto probs = [&](auto Pc) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8 * QB; ++e) prob(Pc, e);
    static_for<QB>([&](auto Qc) __attribute__((always_inline)) { row_sum(Pc, decltype(Qc)::value); });
  };
  auto check = [&](auto Pc, bool next) __attribute__((always_inline)) {
    bool fits = lt[0][0] <= REF_LIMIT;
    if constexpr (QB == 2) fits = fits && lt[1][0] <= REF_LIMIT;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!fits) != 0, 0)) {
      settle(Pc, false, next);
      probs(Pc);
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) l_run[qb] += lt[qb][0];
  };
  auto mask = [&](int j, auto Pc) __attribute__((always_inline)) {  // keys past the end
    constexpr int P = decltype(Pc)::value;
    static_for<2 * QB>([&](auto Ic) __attribute__((always_inline)) {
      constexpr int kb = decltype(Ic)::value / QB, qb = decltype(Ic)::value % QB;
      const int at = L - (j * 32 + kb * 16 + 4 * lq);  // keys of this lane's four that exist
      const f32x4 v = s[P][kb][qb];
      s[P][kb][qb] = f32x4{at > 0 ? v[0] : -INFINITY, at > 1 ? v[1] : -INFINITY, at > 2 ? v[2] : -INFINITY, at > 3 ? v[3] : -INFINITY};
    });
  };
  // the parts of a step one after the other (first and last tile)
  auto scores = [&](auto Pc, int off) __attribute__((always_inline)) {
    constexpr int P = decltype(Pc)::value;
    static_for<DB>([&](auto Ic) __attribute__((always_inline)) {
      constexpr int ks = decltype(Ic)::value >> 1, kb = decltype(Ic)::value & 1;
      const bf16x8 kf = read_k(ks, kb, off);
      static_for<QB>([&](auto Qc) __attribute__((always_inline)) {
        constexpr int qb = decltype(Qc)::value;
        s[P][kb][qb] = mma(kf, qf[qb][ks], ks == 0 ? cm[qb] : s[P][kb][qb]);
      });
    });
  };
  auto values = [&](auto Pc, int off) __attribute__((always_inline)) {
    constexpr int P = decltype(Pc)::value;
    static_for<DB>([&](auto Dc) __attribute__((always_inline)) {
      constexpr int d = decltype(Dc)::value;
      const bf16x8 vf = read_v(d, off);
      static_for<QB>([&](auto Qc) __attribute__((always_inline)) { o[d][decltype(Qc)::value] = mma(vf, pf[P][decltype(Qc)::value], o[d][decltype(Qc)::value]); });
    });
  };
  constexpr int HALF = 32 * ROW_B;
  // One step, half tile j = 2 t + P: scores of j + 1 (even slots), product of j - 1 with its values (odd ones) and probabilities of j in between.
  // Fragments are read RA slots ahead, across the ends of the steps (kn, vn: where the next step's lie).
  auto frag_of = [&](auto Nc, int koffs, int voffs) __attribute__((always_inline)) {
    constexpr int n = decltype(Nc)::value, i = n / 2;
    if constexpr (n % 2 == 0) return read_k(i >> 1, i & 1, koffs);
    else return read_v(i, voffs);
  };
  auto step = [&](auto Pc, int koffs, int voffs, int kn, int vn, auto LOADc, int lk, int lv) __attribute__((always_inline)) {
    constexpr int P = decltype(Pc)::value;
    constexpr bool LOAD = decltype(LOADc)::value, AHEAD = SHORT || NB > 2 || P == 1;
    constexpr int EN = DH == 128 && QB == 2 ? NS - 4 : NS - 2;  // the probabilities are taken in the first EN slots
    static_for<NS>([&](auto Nc) __attribute__((always_inline)) {
      constexpr int n = decltype(Nc)::value, i = n / 2, NE = 8 * QB;
      if constexpr (n + RA < NS) fr[(n + RA) % FR] = frag_of(std::integral_constant<int, n + RA>{}, koffs, voffs);
      else if constexpr (AHEAD) fr[(n + RA) % FR] = frag_of(std::integral_constant<int, n + RA - NS>{}, kn, vn);
      __builtin_amdgcn_sched_barrier(0);
      static_for<QB>([&](auto Qc) __attribute__((always_inline)) {
        constexpr int qb = decltype(Qc)::value;
        if constexpr (n % 2 == 0) s[P ^ 1][i & 1][qb] = mma(fr[n % FR], qf[qb][i >> 1], (i >> 1) == 0 ? cm[qb] : s[P ^ 1][i & 1][qb]);
        else o[i][qb] = mma(fr[n % FR], pf[P ^ 1][qb], o[i][qb]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (qb == 0 && n < EN) {
#pragma unroll
          for (int e = NE * n / EN; e < NE * (n + 1) / EN; ++e) prob(Pc, e);
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (n == EN) {
          row_sum(Pc, qb);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
      if constexpr (LOAD && n < 2 * LPW) {
        if constexpr (n < LPW) load_v(n, lv);
        else load_k(n - LPW, lk);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    check(Pc, true);
  };

  scores(P0{}, 0);
  if (L < 32) mask(0, P0{});
  auto unset = [&]() __attribute__((always_inline)) {
    bool none = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) none = none || m_first[qb] == -INFINITY;
    return __builtin_amdgcn_ballot_w64(none) != 0;
  };
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) m_first[qb] = top(P0{}, qb);
  if (__builtin_expect(unset(), 0)) {
#pragma unroll 1
    for (int j = 1; j * 32 < L; ++j) {
      static_for<DB>([&](auto Ic) __attribute__((always_inline)) {
        constexpr int ks = decltype(Ic)::value >> 1, kb = decltype(Ic)::value & 1;
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(base + (size_t)min(j * 32 + kb * 16 + l16, L - 1) * ld + H + ks * 32 + lq * 8);
        static_for<QB>([&](auto Qc) __attribute__((always_inline)) {
          constexpr int qb = decltype(Qc)::value;
          s[1][kb][qb] = mma(kf, qf[qb][ks], ks == 0 ? zero : s[1][kb][qb]);
        });
      });
      mask(j, P1{});
#pragma unroll
      for (int qb = 0; qb < QB; ++qb) {
        const float mx = top(P1{}, qb);
        m_first[qb] = m_first[qb] == -INFINITY ? mx : m_first[qb];
      }
      if (!unset()) break;
    }
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) m_first[qb] = m_first[qb] == -INFINITY ? 0.f : m_first[qb];
  }
  settle(P0{}, true, false);
  int bl = 0;  // buffer of the last tile
  if (nkv > 1) {
    // first tile
    scores(P1{}, HALF);
    probs(P0{});
    check(P0{}, true);
    // tile t in buffer B: half 2t (keys: second half of t; values: second half of t - 1), half 2t + 1 (keys: first of t + 1, values: first of t)
    auto tile = [&](auto Bc) __attribute__((always_inline)) {
      constexpr int B = decltype(Bc)::value, BP = (B + NB - 1) % NB, BN = (B + 1) % NB;
      step(P0{}, B * TILE_B + HALF, BP * TILE_B + HALF, BN * TILE_B, B * TILE_B, NO{}, 0, 0);
      turn();
      if constexpr (NB == 2) static_for<RA>([&](auto Nc) __attribute__((always_inline)) { fr[decltype(Nc)::value] = frag_of(Nc, BN * TILE_B, B * TILE_B); });
      step(P1{}, BN * TILE_B, B * TILE_B, BN * TILE_B + HALF, B * TILE_B + HALF, YES{}, B * TILE_B, BP * TILE_B);
    };
    if constexpr (!SHORT) {
      turn();
      static_for<RA>([&](auto Nc) __attribute__((always_inline)) { fr[decltype(Nc)::value] = frag_of(Nc, TILE_B, 0); });
      step(P1{}, TILE_B, 0, TILE_B + HALF, HALF, YES{}, 0, (NB - 1) * TILE_B);
      // (In one copy of a tile, with the offsets added to every address, a lone wave's instructions cost more than the code's first run: cut tiles of 16
      // heads of 64, 1101 tokens, 12.9 -> 13.5 us, 8 heads of 128 15.0 -> 16.7.)
      int left = nkv - 2;
      while (left > 0) {
        bool done = false;
        static_for<NB>([&](auto Ic) __attribute__((always_inline)) {
          if (done) return;
          constexpr int B = (decltype(Ic)::value + 1) % NB;
          tile(std::integral_constant<int, B>{});
          done = --left == 0;
        });
      }
      bl = (nkv - 1) % NB;
      if constexpr (NB == 2) turn();
    } else {  // (fewer tiles than buffers: tile t in buffer t, nothing to wait for)
      static_for<RA>([&](auto Nc) __attribute__((always_inline)) { fr[decltype(Nc)::value] = frag_of(Nc, TILE_B, 0); });
      step(P1{}, TILE_B, 0, TILE_B + HALF, HALF, NO{}, 0, 0);
      for (int at = TILE_B; at < (nkv - 1) * TILE_B; at += TILE_B) {
        step(P0{}, at + HALF, at - HALF, at + TILE_B, at, NO{}, 0, 0);
        step(P1{}, at + TILE_B, at, at + TILE_B + HALF, at + HALF, NO{}, 0, 0);
      }
      bl = nkv - 1;
    }
  }
  // last tile
  const int j = 2 * (nkv - 1), bo = bl * TILE_B, po = (bl == 0 ? NB - 1 : bl - 1) * TILE_B;
  const bool two = L - j * 32 > 32;
  if (two) scores(P1{}, bo + HALF);
  if (!two && j > 0 && L < j * 32 + 32) mask(j, P0{});
  probs(P0{});
  if (j > 0) values(P1{}, po + HALF);
  check(P0{}, two);
  if (two) {
    if (L < j * 32 + 64) mask(j + 1, P1{});
    probs(P1{});
    values(P0{}, bo);
    check(P1{}, false);
    values(P1{}, bo + HALF);
  } else {
    values(P0{}, bo);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the end
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const float inv = 1.f / l_run[qb];
    const int qi = q0 + qb * 16 + l16;
    if (qi < L) {
      bf16* orow = out + ((size_t)b * L + qi) * H + (size_t)h * DH + lq * 4;
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        bf16x4 v = {(bf16)(o[d][qb][0] * inv), (bf16)(o[d][qb][1] * inv), (bf16)(o[d][qb][2] * inv), (bf16)(o[d][qb][3] * inv)};
        *reinterpret_cast<bf16x4*>(orow + d * 16) = v;
      }
    }
  }
}

// Forms of the loop.  WIDE: head dim 128, eight waves, two a SIMD (228 registers), four buffers of 32 KB, one workgroup a compute unit; head dim 64, four
// waves, three workgroups a unit (168 registers, 48 KB; two with four or eight buffers: 5 to 40 % slower from three workgroups a unit on, no faster below).
// PAIR: head dim 128, four waves and two buffers, two workgroups a unit: one's first fetch, last tile and stores run beside the other's loop, and tiles are
// finer (rule::attention_pair; 64 samples of 24 heads, 192 tokens 109 -> 74 us, 257 172 -> 118, 1024 859 -> 770).  AHEAD: beside workgroups that read weights.
constexpr int ATTN_WIDE = 0, ATTN_PAIR = 1, ATTN_AHEAD = 2;  // (an unnamed enumeration in a kernel's type has another name on the host than on the device)
template <int DH, int KIND>
struct AttnForm {
  static constexpr int NW = KIND == ATTN_AHEAD || (KIND == ATTN_WIDE && DH == 128) ? 8 : 4, NB = KIND == ATTN_PAIR ? 2 : KIND == ATTN_AHEAD || DH == 128 ? 4 : 3;
  static constexpr int WPE = KIND == ATTN_AHEAD || DH == 128 ? 2 : 3, QB = KIND == ATTN_AHEAD ? 1 : 2, BM = 16 * QB * NW;
};
constexpr int SHORT_NW = 4, SHORT_BM = 32 * SHORT_NW;
template <int DH>
constexpr int SHORT_TILES = DH == 128 ? 3 : 2;  // key tiles that the kernel of short sequences takes
template <int DH>
constexpr int TILES_B = 2 * KV_TILE * DH * 2;   // bytes of a buffer of keys and one of values

extern __shared__ __attribute__((aligned(1024))) char g_tiles[];

// At least NB key tiles; AHEAD: any number, tiles of 128 queries by eight waves of 16, as two waves a SIMD issue what one alone takes twice as long for: one image
// sample (144 tiles of 16 heads of 64) 1044 us a call with
// four waves of 32, 1038 with twice the workgroups of four waves of 16, 1026 so.
template <int DH, bool PRE, int KIND>
__global__ __launch_bounds__((AttnForm<DH, KIND>::NW) * 64, (AttnForm<DH, KIND>::WPE)) void attn_bf16_kernel(
    const bf16* __restrict__ qkv, bf16* __restrict__ out, int L, int H, int NH, int n_pairs, int plan, float scale_log2, Warm<KIND == ATTN_AHEAD> warm) {
  using F = AttnForm<DH, KIND>;
  constexpr int NW = F::NW, NB = F::NB, BM = F::BM;
  unsigned block = blockIdx.x;
  if constexpr (KIND == ATTN_AHEAD) {
    if (block < (unsigned)warm.blocks) {
      warm_rows<NW * 64>(warm);
      return;
    }
    block -= warm.blocks;  // (a multiple of 8)
  }
  int pair, q_first, parts;
  if (!attn_tile(block, (L + BM - 1) / BM, n_pairs, plan, BM, &pair, &q_first, &parts) || q_first >= L) return;
  auto run = [&](auto QBc, auto SHORTc, int waves) __attribute__((always_inline)) {
    attn_queries<DH, NW, NB, decltype(QBc)::value, decltype(SHORTc)::value, PRE>(g_tiles, qkv, out, L, H, NH, pair, q_first, waves, scale_log2);
  };
  using Q1 = std::integral_constant<int, 1>;
  using Q2 = std::integral_constant<int, 2>;
  if constexpr (KIND == ATTN_AHEAD) {
    if (L <= (NB - 1) * KV_TILE) run(Q1{}, std::true_type{}, NW);
    else run(Q1{}, std::false_type{}, NW);
  } else {
    if (KIND == ATTN_PAIR || parts == 1) run(Q2{}, std::false_type{}, NW);
    else run(Q1{}, std::false_type{}, 2 * NW / parts);
  }
}

// Fewer key tiles than NB: without the loop's code and with LDS for these tiles alone, so that more workgroups share a unit.  (Queries scaled ahead:
// scale_log2 = 1.)
template <int DH>
__global__ __launch_bounds__(SHORT_NW * 64, DH == 128 ? 2 : 3) void attn_bf16_short_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ out, int L, int H,
                                                                                             int NH, int n_pairs, int plan, float scale_log2) {
  constexpr int NB = SHORT_TILES<DH> + 1;
  int pair, q_first, parts;
  if (!attn_tile(blockIdx.x, (L + SHORT_BM - 1) / SHORT_BM, n_pairs, plan, SHORT_BM, &pair, &q_first, &parts) || q_first >= L) return;
  if (parts == 1) attn_queries<DH, SHORT_NW, NB, 2, true, false>(g_tiles, qkv, out, L, H, NH, pair, q_first, SHORT_NW, scale_log2);
  else attn_queries<DH, SHORT_NW, NB, 1, true, false>(g_tiles, qkv, out, L, H, NH, pair, q_first, SHORT_NW, scale_log2);
}

template <int DH>
static br_status attn_launch(const bf16* qkv, bf16* out, int B, int L, int NH, bool prescaled, const WarmRows& next, hipStream_t st) {
  const long long n_pairs = (long long)B * NH;
  const int grouped = n_pairs >= 32 ? 1 : 0, n_cu = device_cu_count(), H = NH * DH, nkv = cdiv(L, KV_TILE);
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)DH));
  // tiles of BM queries: of a die if grouped, else of all
  auto tiles = [&](int rows) { return (grouped ? (n_pairs + 7) / 8 : n_pairs) * cdiv(L, rows); };
  const int dies = grouped ? 8 : 1;
  BR_REQUIRE(tiles(128) * dies <= 0x7FFFFFFFLL, BR_ESHAPE, "attention: too many workgroups for one launch");
  // Where the launch leaves compute units idle: as much of the list as they read meanwhile (see warm_rows).
  WarmRows warm = next;
  const long long n_blocks = tiles(128) * dies;
  warm.blocks = next.n16[0] > 0 && prescaled ? (n_cu - (int)std::min<long long>(n_blocks, n_cu)) / 8 * 8 : 0;
  unsigned budget = (unsigned)(WARM_BYTES_PER_TILE / 16 * (nkv + 4) / 256 * warm.blocks);
  size_t bytes = 0;
  for (const unsigned n : next.n16) bytes += (size_t)n * 16;
  if (warm.blocks >= 32 && rule::read_ahead((size_t)budget * 16, bytes)) {
    using F = AttnForm<DH, ATTN_AHEAD>;
    for (unsigned& n : warm.n16) {
      n = std::min(n, budget);
      budget -= n;
    }
    hipLaunchKernelGGL((attn_bf16_kernel<DH, true, ATTN_AHEAD>), dim3((unsigned)(n_blocks + warm.blocks)), dim3(F::NW * 64), std::min(nkv, F::NB) * TILES_B<DH>, st,
                       qkv, out, L, H, NH, (int)n_pairs, grouped | 1 << 1, scale_log2, warm);
    BR_LAUNCH_CHECK();
    return BR_OK;
  }
  const bool pair = DH == 128 && rule::attention_pair(L, tiles(128), tiles(256), n_cu / dies), brief = !pair && nkv <= SHORT_TILES<DH>;
  const long long n = tiles(pair || brief ? 128 : AttnForm<DH, ATTN_WIDE>::BM), slots = (long long)n_cu / dies * (DH == 64 ? 3 : 1);
  const long long whole = brief ? 0 : n / slots * slots;
  const int split = !pair && n < (1 << 26) ? rule::attention_parts(DH, brief, n - whole, whole, n_cu / dies) : 1;
  const int plan = grouped | split << 1 | (split > 1 ? (int)whole << 4 : 0);
  const dim3 g((unsigned)((split > 1 ? whole + (n - whole) * split : n) * dies));
  auto loop = [&](auto KINDc) {
    constexpr int KIND = decltype(KINDc)::value;
    using F = AttnForm<DH, KIND>;
    const dim3 b(F::NW * 64);
    if (prescaled)
      hipLaunchKernelGGL((attn_bf16_kernel<DH, true, KIND>), g, b, F::NB * TILES_B<DH>, st, qkv, out, L, H, NH, (int)n_pairs, plan, scale_log2, NoWarm{});
    else hipLaunchKernelGGL((attn_bf16_kernel<DH, false, KIND>), g, b, F::NB * TILES_B<DH>, st, qkv, out, L, H, NH, (int)n_pairs, plan, scale_log2, NoWarm{});
  };
  if (pair) {
    if constexpr (DH == 128) loop(std::integral_constant<int, ATTN_PAIR>{});
  } else if (brief) {
    hipLaunchKernelGGL((attn_bf16_short_kernel<DH>), g, dim3(SHORT_NW * 64), nkv * TILES_B<DH>, st, qkv, out, L, H, NH, (int)n_pairs, plan,
                       prescaled ? 1.f : scale_log2);
  } else {
    loop(std::integral_constant<int, ATTN_WIDE>{});
  }
  BR_LAUNCH_CHECK();
  return BR_OK;
}

br_status launch_attention_bf16(const bf16* qkv, bf16* out, int B, int L, int NH, int DH, int q_prescaled, const WarmRows& next, hipStream_t st) {
  BR_REQUIRE(L >= 1, BR_EINVAL, "attention: empty sequence");
  // the rows of a sample are addressed with 32-bit byte offsets from its first one
  BR_REQUIRE((unsigned long long)L * 3ull * NH * DH * 2ull < (1ull << 32), BR_ESHAPE,
             "attention: one sample's QKV rows exceed 4 GiB");
  ProfScope ps(st, PROF_ATTN + DH, 4.0 * B * (double)L * L * NH * DH);
  if (DH == 64) return attn_launch<64>(qkv, out, B, L, NH, q_prescaled, next, st);
  if (DH == 128) return attn_launch<128>(qkv, out, B, L, NH, q_prescaled, next, st);
  return fail(BR_ESHAPE, "bf16 attention: head dim must be 64 or 128");
}

}  // namespace br
