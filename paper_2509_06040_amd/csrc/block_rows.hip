// The row-local part of a network block in one launch, for narrow networks: everything between two attentions works on
// each row by itself, so a workgroup takes 16 RT rows of the residual stream through
//   output projection -> gated residual -> LayerNorm-modulate -> MLP (GELU) -> gated residual -> LayerNorm-modulate
//   -> QKV projection of the next block, or final linear and unpatchify behind the last one,
// and, as the head of the network, through patch gathering -> patch embedding -> LayerNorm-modulate -> QKV projection of
// the first block.  A block is then two launches (attention, this) instead of five to seven, and nothing but the residual
// rows and the QKV rows passes through memory.
//
// What bounds it: a chain of instructions and waits with few rows, then the weights, 12 H^2 of them, that every workgroup streams through its
// compute unit.  The activations stay in LDS.  Every wave fetches the weights of its own columns, 16 rows of 128 or 256 bytes a step, in whole
// lines into a ring of its own (global -> LDS directly), 8 to 16 KB ahead and across the ends of the phases: the next phase's
// weights are under way while a phase's last products, its barrier and the LayerNorm run, and no barrier waits for weights.
// (Fetched straight into registers, in the layout of the matrix instruction, four lanes of a load touch four lines: 14
// bytes a clock of a compute unit, a quarter of this.)  The hidden sizes that networks have (MLP ratio 4) get a form laid out at compile time; one loop
// serves all phases of any other: whole velocity calls of bf16 hidden 64, 90 rows 121 -> 93 us, 31 590 rows 593 -> 473; 128, 90 rows 369 -> 281,
// 24 732 rows 894 -> 694; 256, 1778 rows 198 -> 162; fp32 64, 200 rows 103 -> 92; 96, 122 rows 272 -> 234; 128, 762 rows 335 -> 285.
//
// Every output is one chain over k in ascending order (gemm_frag.h), every rounding and every LayerNorm sum is where
// the separate kernels have it: the results are theirs bit for bit, whatever the number of rows selects.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "common.h"
#include "dit.h"
#include "gemm_frag.h"
#include "prof.h"
#include "static_for.h"

namespace br {

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

namespace {
constexpr int NW = 8, NT = NW * 64;  // waves, threads
constexpr int RING_B = 8192;         // LDS of a wave's weights in flight
constexpr int LDS_LIMIT = 160 * 1024;

}  // namespace

// n / d for n d < 2^32 by a multiplication (a division is 35 instructions, one after the other)
struct FastDiv {
  unsigned m;
  FastDiv() = default;
  explicit FastDiv(int d) : m(d > 1 ? (unsigned)(((1ull << 32) + d - 1) / d) : 0u) {}
  __device__ __forceinline__ int div(int n) const { return m ? (int)__umulhi((unsigned)n, m) : n; }
};

// p[i] of a uniform index i of an array that no kernel under way writes, through the scalar cache
__device__ __forceinline__ int scalar_load(const int* p, int i) {
  typedef const int __attribute__((address_space(4)))* cptr;
  return ((cptr)p)[__builtin_amdgcn_readfirstlane(i)];
}

struct RowsArgs {
  FastDiv by_L, by_H4, by_mq, by_pd, by_pw, by_ph, by_pt, by_gw, by_gh;
  int M, L, n_img;                  // rows; rows and image rows of a sample
  int H, RH, NTAIL;                 // hidden size, MLP width, columns of the tail (3 H or the patch vector)
  float* x;                         // [M, H] residual stream
  const float* mods;                // modulation vectors: per group, consecutive from mods_off (see the kernel)
  int A, mods_off;                  // row length; offset of the floats taken
  const int* modmap;                // [samples] group (body)
  const void* attn;                 // [M, H] (body)
  const void *w0, *fc1_w, *fc2_w, *tail_w;  // w0: output projection, or patch embedding (head)
  const float *b0, *fc1_b, *fc2_b, *tail_b;
  void* qkv;                        // [M, 3 H]
  int qcols;
  float qscale;
  Epilogue<EPI_UNPATCH, float> fin;
  // head
  SampleMap sm;
  int s0, B, v_rows_mode;
  int *modmap_out, *vrows;
  const float *z, *pos, *cond_emb;
  long long D;
  int pd, lt, lh, lw, pt, ph, pw, gh, gw, Nc;
  // LDS: byte offsets of the regions behind the residual rows
  int o_act, o_hid, o_mods, o_bias, o_vrow, o_ring;
};

enum { ROWS_HEAD = 0, ROWS_BODY = 1, ROWS_LAST = 2 };

// Weights that a wave of the form for hidden size `h` has in flight: 16, 12 or 8 KB, whatever fits beside rows of (at most) two samples.
constexpr int rows_ring(int es, int h, int rt) {
  const int rest = 16 * rt * (h * 4 + h * es + 4 * h * es) + 2 * 6 * h * 4 + 9 * h * 4 + 4096;
  return rest + NW * 16384 <= LDS_LIMIT ? 16384 : rest + NW * 12288 <= LDS_LIMIT ? 12288 : 8192;
}

// HC: hidden size, MLP ratio 4, patch vectors of at most 256 bytes and 128 elements, with everything about the phases known to the compiler;
// 0: any sizes.
template <typename T, int RT, int SPS, int KIND, int HC>
__global__ __launch_bounds__(NT) void block_rows_kernel(RowsArgs a) {
  constexpr int ES = (int)sizeof(T), BMR = 16 * RT, LPR = NT / BMR, V = 64 / LPR;
  extern __shared__ __attribute__((aligned(1024))) char lds[];
  char* const xs = lds;                 // residual rows, 16-byte chunk c of row r in slot c ^ (r & xm)
  char* const act = lds + a.o_act;      // operand rows in stages of 128 bytes a row (gemm_frag.h)
  char* const hid = lds + a.o_hid;      // MLP rows (head: patch rows), likewise
  float* const smods = reinterpret_cast<float*>(lds + a.o_mods);
  float* const sbias = reinterpret_cast<float*>(lds + a.o_bias);
  int* const svrow = reinterpret_cast<int*>(lds + a.o_vrow);

  const int H = HC ? HC : a.H, RH = HC ? 4 * HC : a.RH, NTAIL = HC && KIND != ROWS_LAST ? 3 * HC : a.NTAIL, H4 = H >> 2, M = a.M, L = a.L;
  const int m0 = blockIdx.x * BMR;
  const int mods_n = KIND == ROWS_HEAD ? 2 * H : 6 * H;  // floats of a sample's vectors
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xm = (H & 63) == 0 ? 15 : (H & 31) == 0 ? 7 : 3;
  const int b_first = a.by_L.div(m0);

  if (KIND == ROWS_HEAD && blockIdx.x == 0) {  // per-sample maps of the batch
    for (int i = tid; i < a.B; i += NT) {
      const int b = a.s0 + i;
      a.modmap_out[i] = a.sm.group ? a.sm.group[b] : a.sm.group0 + sample_cond(a.sm, b);
      a.vrows[i] = a.v_rows_mode == 1 ? sample_row(a.sm, b) : (a.v_rows_mode == 2 ? i : b);
    }
  }
  // behind the last block only image rows have an output
  if (KIND == ROWS_LAST && m0 - b_first * L >= a.n_img && a.by_L.div(min(m0 + BMR, M) - 1) == b_first) return;

  // modulation group of a sample (forms for a hidden size; a uniform index: scalar loads, which wait for none of the others)
  auto group_of = [&](int b) __attribute__((always_inline)) {
    return KIND != ROWS_HEAD ? scalar_load(a.modmap, b)
           : a.sm.group      ? scalar_load(a.sm.group, a.s0 + b)
                             : a.sm.group0 + (a.sm.cond ? scalar_load(a.sm.cond, a.s0 + b) : sample_cond(a.sm, a.s0 + b));
  };
  const int g_first = HC ? group_of(b_first) : 0;
  // ---- rows, modulation vectors and biases to LDS (global -> LDS directly, 1 KB per wave and instruction)
  auto fill = [&](char* dst, const void* src) __attribute__((always_inline)) {
    const unsigned d = (unsigned)(uintptr_t)BR_LPTR(dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(d), "v"(src) : "memory", "m0");
  };
  if (KIND != ROWS_HEAD) {
    const int n_act = BMR * (((H * ES + 127) >> 7) * 8), kc = H * ES / 16;
    for (int p = wv; p * 64 < n_act; p += NW) {
      const int i = p * 64 + lane, row = (i >> 3) & (BMR - 1), c = (i / (8 * BMR)) * 8 + ((i & 7) ^ ((row >> 1) & 7));
      fill(act + p * 1024, reinterpret_cast<const char*>(a.attn) + (size_t)min(m0 + row, M - 1) * H * ES + min(c, kc - 1) * 16);
    }
  }
  for (int p = wv; p * 64 < BMR * H4; p += NW) {
    const int i = p * 64 + lane, row = HC ? i / (HC / 4 + !HC) : a.by_H4.div(i), c = (i - row * H4) ^ (row & xm), m = min(m0 + row, M - 1);
    const float* src = a.x + (size_t)m * H;
    if (KIND == ROWS_HEAD) {  // what the patch embedding is added to, or the embedded condition token
      const int b = a.by_L.div(m), tok = m - b * L;
      src = tok < a.n_img ? a.pos + (size_t)tok * H : a.cond_emb + ((size_t)sample_cond(a.sm, a.s0 + b) * a.Nc + (tok - a.n_img)) * H;
    }
    fill(xs + p * 1024, src + c * 4);
  }
  const int b_last = a.by_L.div(min(m0 + BMR, M) - 1), mq = mods_n >> 2;
  if constexpr (HC == 0) {  // (a lane looks up its own sample's: one wait for all, in front of what waits for nothing)
    const int n_mods = (b_last - b_first + 1) * mq;
    for (int p = wv; p * 64 < n_mods; p += NW) {
      const int i = min(p * 64 + lane, n_mods - 1), s = a.by_mq.div(i), b = b_first + s;
      const int g = KIND != ROWS_HEAD ? a.modmap[b] : a.sm.group ? a.sm.group[a.s0 + b] : a.sm.group0 + sample_cond(a.sm, a.s0 + b);
      fill(reinterpret_cast<char*>(smods) + p * 1024, a.mods + (size_t)g * a.A + a.mods_off + (i - s * mq) * 4);
    }
  }
  // biases: first product | FC1 | FC2 | tail
  const float *const b_0 = a.b0, *const b_1 = a.fc1_b, *const b_2 = a.fc2_b, *const b_3 = a.tail_b;
  const int nb1 = H4, nb2 = KIND == ROWS_HEAD ? nb1 : nb1 + (RH >> 2), nb3 = KIND == ROWS_HEAD ? nb2 : nb2 + H4,
            nb4 = nb3 + (NTAIL >> 2);
  for (int p = wv; p * 64 < nb4; p += NW) {
    const int i = min(p * 64 + lane, nb4 - 1);
    const float* src = i < nb1 ? b_0 + i * 4 : i < nb2 ? b_1 + (i - nb1) * 4 : i < nb3 ? b_2 + (i - nb2) * 4 : b_3 + (i - nb3) * 4;
    fill(reinterpret_cast<char*>(sbias) + p * 1024, src);
  }
  if constexpr (HC != 0) {
    for (int b = b_first; b <= b_last; ++b) {
      const int g = b == b_first ? g_first : group_of(b);
      const float* src = a.mods + (size_t)g * a.A + a.mods_off;
      char* const dst = reinterpret_cast<char*>(smods) + (b - b_first) * mods_n * 4;
      for (int p = wv; p * 64 < mq; p += NW)
        if (p * 64 + lane < mq) fill(dst + p * 1024, src + (p * 64 + lane) * 4);
    }
  }
  if (HC && KIND == ROWS_LAST && wv == 0) {  // where the samples of these rows go
    const unsigned d = (unsigned)(uintptr_t)BR_LPTR(svrow);
    const int* const src = a.fin.a.vrows + min(b_first + lane, b_last);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(d), "v"(src) : "memory", "m0");
  }
  auto gather = [&]() __attribute__((always_inline)) {
  if (KIND == ROWS_HEAD) {  // patch vectors (c, dt, dh, dw) of the image rows
#pragma unroll 2
    for (int e = tid; e < BMR * a.pd; e += NT) {
      const int row = a.by_pd.div(e), el = e - row * a.pd, m = min(m0 + row, M - 1), b = a.by_L.div(m), tok = min(m - b * L, a.n_img - 1);
      const int t1 = a.by_gw.div(tok), tt = a.by_gh.div(t1), tw = tok - t1 * a.gw, th = t1 - tt * a.gh;
      const int e1 = a.by_pw.div(el), e2 = a.by_ph.div(e1), c = a.by_pt.div(e2);
      const int dw = el - e1 * a.pw, dh = e1 - e2 * a.ph, dt = e2 - c * a.pt;
      const long long idx = (((long long)c * a.lt + tt * a.pt + dt) * a.lh + th * a.ph + dh) * a.lw + tw * a.pw + dw;
      const int byte = el * ES;
      *reinterpret_cast<T*>(hid + (byte >> 7) * (BMR * 128) + row * 128 + ((((byte >> 4) & 7) ^ ((row >> 1) & 7)) << 4) + (byte & 15)) =
          (T)a.z[(size_t)sample_row(a.sm, a.s0 + b) * a.D + idx];
    }
    // zeros to the end of the last step, whose weights are the row's first ones once more.  (An infinite one among them makes a NaN where
    // the product alone is infinite; the LayerNorm of the row makes that of either.)
    const int end = HC ? 16 : (a.pd * ES + SPS * 128 - 1) / (SPS * 128) * (SPS * 8);
    for (int row = tid; row < BMR; row += NT)
      for (int c = a.pd * ES / 16; c < end; ++c)
        *reinterpret_cast<float4*>(hid + (c >> 3) * (BMR * 128) + row * 128 + (((c & 7) ^ ((row >> 1) & 7)) << 4)) = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  };
  // this lane's fragments of a step (of its row of the weights, and of its operand row of row tile 0): GemmFrag16
  typedef typename GemmFrag16<T>::type frag;
  constexpr int NF = GemmFrag16<T>::COUNT, FLIP = GemmFrag16<T>::FLIP;
  const int fo = GemmFrag16<T>::offset(l16, lq);
  // four columns of operand row `row` as T
  auto put = [&](char* op, int row, int n, float v0, float v1, float v2, float v3) __attribute__((always_inline)) {
    const int byte = n * ES;
    store4<T>(reinterpret_cast<T*>(op + (byte >> 7) * (BMR * 128) + row * 128 + ((((byte >> 4) & 7) ^ ((row >> 1) & 7)) << 4) + (byte & 15)), v0, v1, v2, v3);
  };
  auto x_at = [&](int row, int c4) __attribute__((always_inline)) { return reinterpret_cast<float4*>(xs + row * H * 4 + ((c4 ^ (row & xm)) << 4)); };
  int srow[RT];  // modulation vectors of this lane's row of each row tile (floats)
#pragma unroll
  for (int r = 0; r < RT; ++r) srow[r] = (a.by_L.div(min(m0 + r * 16 + l16, M - 1)) - b_first) * mods_n;

  // LayerNorm of the rows in xs, modulated with the vectors at `shift` and `shift` + H, to `act`; LPR lanes a row, whose sums are
  // those of ln_modulate_kernel's 64 (this lane holds what its lanes sub, sub + LPR, ... do).  The rows go to memory as well.
  auto layer_norm = [&](int shift, bool store) __attribute__((always_inline)) {
    const int row = tid / LPR, sub = tid % LPR, m = m0 + row;
    const float* mr = smods + (a.by_L.div(min(m, M - 1)) - b_first) * mods_n + shift;
    float4 v[V];
    float p[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int c4 = sub + LPR * i;
      v[i] = c4 < H4 ? *x_at(row, c4) : make_float4(0.f, 0.f, 0.f, 0.f);
      p[i] = (v[i].x + v[i].y) + (v[i].z + v[i].w);
      if (store && c4 < H4 && m < M) *reinterpret_cast<float4*>(a.x + (size_t)m * H + c4 * 4) = v[i];
    }
    auto row_sum = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int d = V / 2; d > 0; d >>= 1)
#pragma unroll
        for (int j = 0; j < d; ++j) p[j] += p[j + d];
      return lanes_sum<LPR>(p[0]);
    };
    const float mean = row_sum() / (float)H;
#pragma unroll
    for (int i = 0; i < V; ++i) p[i] = sub + LPR * i < H4 ? sum_sq4(v[i], mean) : 0.f;
    const float rstd = 1.0f / __builtin_sqrtf(row_sum() / (float)H + 1e-6f);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int c4 = sub + LPR * i;
      if (c4 < H4) {
        const float4 sh = reinterpret_cast<const float4*>(mr)[c4], sc = reinterpret_cast<const float4*>(mr + H)[c4];
        put(act, row, c4 * 4, fmaf((v[i].x - mean) * rstd, 1.f + sc.x, sh.x), fmaf((v[i].y - mean) * rstd, 1.f + sc.y, sh.y),
            fmaf((v[i].z - mean) * rstd, 1.f + sc.z, sh.z), fmaf((v[i].w - mean) * rstd, 1.f + sc.w, sh.w));
      }
    }
  };
  auto bias4 = [&](int at) __attribute__((always_inline)) { return *reinterpret_cast<const float4*>(sbias + at); };

  if constexpr (HC != 0) {
    // ---- The phases (0 the first product, 1 FC1, 2 FC2, 3 the tail; head: 0 and 3) laid out at compile time: a wave's column blocks wv, wv + NW,
    // ... of each, KS steps a block, are one list of steps, and everything a step needs is an immediate.  What bounded the form for any sizes was the
    // issue of instructions: a wave takes one about every six cycles, and the products were a tenth of them beside the cursor, loops
    // and branches.  Cycles of a workgroup, any sizes -> this: bf16 hidden 64 20 800 -> 9800, 128 24 600 -> 15 100, 256 54 400 -> 45 200; fp32 64 27 800 ->
    // 18 600 (before its reads moved between the products).  (In the form for any sizes neither more weights in flight nor fragments read a step ahead gained anything.)
    // Left at 64 in bf16: 3600 until rows and modulation vectors are there, 950 a LayerNorm, 100 to 450 a barrier, 700 to 1000 a phase.
    // A wave without a column block in a round fetches the last one all the same: what it waits for is a number of loads.
    constexpr int STEP_B = SPS * 2048, RING = rows_ring(ES, HC, RT), PD = RING / STEP_B, LPS = 2 * SPS;  // LPS: loads of a step
    constexpr bool HEAD = KIND == ROWS_HEAD, LAST = KIND == ROWS_LAST;
    constexpr int KB = HC * ES, KS = KB / (SPS * 128);
    static_assert(KB % (SPS * 128) == 0 && PD >= 2, "");
    constexpr int NB0 = (HC + 127) / 128, KS0 = HEAD ? 2 / SPS : KS;
    constexpr int NB1 = HEAD ? 0 : (4 * HC + 127) / 128, NB2 = HEAD ? 0 : (HC + 127) / 128, KS2 = 4 * KS;
    constexpr int NB3 = LAST ? 1 : (3 * HC + 127) / 128;
    constexpr int S1 = NB0 * KS0, S2 = S1 + NB1 * KS, S3 = S2 + NB2 * KS2, S = S3 + NB3 * KS;  // first step of a phase
    char* const my_ring = lds + a.o_ring + wv * RING;
    const unsigned ring = (unsigned)(uintptr_t)BR_LPTR(my_ring);
    const int lrow = lane >> 3, ch[2] = {((lane & 7) ^ ((lrow >> 1) & 7)) * 16, (((lane & 7) ^ ((lrow >> 1) & 7)) * 16) ^ 64};
    const int kb0 = HEAD ? a.pd * ES : KB;
    const int ntail = LAST ? NTAIL : 3 * HC;
    // A load fills eight rows (lane = 8 row + slot), slot s of row r from chunk s ^ ((r >> 1) & 7): a scalar address and these offsets
    unsigned off_h[2], off_r[2], off_0[2], off_t[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      off_h[i] = (lrow + 8 * i) * KB + ch[i];
      off_r[i] = (lrow + 8 * i) * (4 * KB) + ch[i];
      off_0[i] = (lrow + 8 * i) * kb0;
      off_t[i] = min(lrow + 8 * i, ntail - 1 - max(min(wv, (ntail + 15) / 16 - 1), 0) * 16) * KB + ch[i];
    }
    auto fetch = [&](auto Sc) __attribute__((always_inline)) {
      constexpr int at = decltype(Sc)::value;
      const unsigned ring_at = ring;
      if constexpr (at < S) {
        constexpr int ph = at < S1 ? 0 : at < S2 ? 1 : at < S3 ? 2 : 3;
        constexpr int first = ph == 0 ? 0 : ph == 1 ? S1 : ph == 2 ? S2 : S3, ks = ph == 0 ? KS0 : ph == 2 ? KS2 : KS;
        constexpr int i = (at - first) / ks, k = (at - first) % ks;
        const int blocks = ph == 1 ? HC / 4 : ph == 3 ? (ntail + 15) / 16 : HC / 16;
        const int kb = ph == 0 ? kb0 : ph == 2 ? 4 * KB : KB;
        const int cb = min(wv + NW * i, blocks - 1);
        const char* base = reinterpret_cast<const char*>(ph == 0 ? a.w0 : ph == 1 ? a.fc1_w : ph == 2 ? a.fc2_w : a.tail_w) + (size_t)(cb * 16) * kb;
        constexpr unsigned slot = at % PD * STEP_B;
#pragma unroll
        for (int l = 0; l < LPS; ++l) {
          unsigned o = ph == 0 && HEAD ? off_0[l & 1] : ph == 2 ? off_r[l & 1] : ph == 3 && LAST ? off_t[l & 1] : off_h[l & 1];
          int c = k * (SPS * 128) + (l >> 1) * 128;
          if constexpr (ph == 0 && HEAD) {  // (what lies past the end of a patch vector is fetched from the start of its row)
            const int at_k = c + ch[l & 1];
            o += at_k < kb0 ? at_k : 0;
            c = 0;
          }
          const char* src = scalar_ptr(base + c);
          asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(ring_at), "v"(o), "s"(src), "n"(slot + l * 1024) : "memory", "m0", "scc");
        }
      }
    };
    static_for<PD>([&](auto Sc) __attribute__((always_inline)) { fetch(Sc); });
    gather();
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LPS * (PD < S ? PD : S)) : "memory");  // all but the weights
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    frag w[2][SPS][NF], o[2][SPS][RT][NF];
    f32x4 acc[RT];
    auto landed = [&](auto Sc) __attribute__((always_inline)) {  // waits for a step
      constexpr int at = decltype(Sc)::value, young = at + PD - 1 < S - 1 ? PD - 1 : S - 1 - at;
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPS * young) : "memory");
    };
    const int n0 = wv * 16 + lq * 4;  // this lane's columns of the wave's first block
    // A phase: NBp blocks of KSp steps from step FIRST on, operand rows at `op`, N columns; epi(i) takes the sums of block i.  A step's slot is refilled
    // as soon as its fragments are in registers; the next step's are read behind its products, in fp32 between them (BETWEEN): those are sixteen that
    // wait for one another (hidden 128, 762 rows: 300 -> 285 us a call; bf16, with four: 281 -> 286).
    auto run = [&](auto FIRSTc, auto NBc, auto KSc, const char* op, int n_cols, auto&& epi) __attribute__((always_inline)) {
      constexpr int FIRST = decltype(FIRSTc)::value, NBp = decltype(NBc)::value, KSp = decltype(KSc)::value, NMMA = SPS * NF;
      constexpr bool BETWEEN = ES == 4;
      // fragment f of step j of the phase (rows of one step are read once, to set 0)
      auto read_w = [&](auto Jc, int u, int i) __attribute__((always_inline)) {
        constexpr int j = decltype(Jc)::value, slot = (FIRST + j) % PD * STEP_B;
        w[j & 1][u][i] = *reinterpret_cast<const frag*>(my_ring + (fo ^ (i * FLIP)) + (slot + u * 2048));
      };
      auto read_o = [&](auto Jc, int u, int i) __attribute__((always_inline)) {
        constexpr int j = decltype(Jc)::value, k = j % KSp;
#pragma unroll
        for (int r = 0; r < RT; ++r)
          o[KSp == 1 ? 0 : j & 1][u][r][i] = *reinterpret_cast<const frag*>(op + (fo ^ (i * FLIP)) + (k * SPS * BMR * 128 + (u * RT + r) * 2048));
      };
      if (wv * 16 < n_cols) {
        landed(FIRSTc);
        static_for<NMMA>([&](auto Fc) __attribute__((always_inline)) {
          constexpr int f = decltype(Fc)::value;
          read_w(std::integral_constant<int, 0>{}, f / NF, f % NF);
          read_o(std::integral_constant<int, 0>{}, f / NF, f % NF);
        });
      }
      static_for<NBp * KSp>([&](auto Jc) __attribute__((always_inline)) {
        constexpr int j = decltype(Jc)::value, i = j / KSp, k = j % KSp, at = FIRST + j;
        constexpr bool more = j + 1 < NBp * KSp;
        const bool here = (wv + NW * i) * 16 < n_cols;  // (uniform; false in the last round alone)
        if (here) {
          if constexpr (k == 0) {
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
          __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
          asm volatile("" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        fetch(std::integral_constant<int, at + PD>{});
        if (here) {
          if constexpr (more && BETWEEN) landed(std::integral_constant<int, at + 1>{});
          static_for<NMMA>([&](auto Fc) __attribute__((always_inline)) {
            constexpr int f = decltype(Fc)::value, u = f / NF, n = f % NF;
            static_for<RT>([&](auto Rc) __attribute__((always_inline)) {
              constexpr int r = decltype(Rc)::value;
              acc[r] = GemmFrag16<T>::mma(w[j & 1][u][n], o[KSp == 1 ? 0 : j & 1][u][r][n], acc[r]);
            });
            if constexpr (more && BETWEEN) {  // (of a block that the wave does not have: something from the ring, for nobody)
              read_w(std::integral_constant<int, j + 1>{}, u, n);
              if constexpr (KSp > 1) read_o(std::integral_constant<int, j + 1>{}, u, n);
            }
            if constexpr (BETWEEN) __builtin_amdgcn_sched_barrier(0);
          });
          if constexpr (more && !BETWEEN) {
            if ((wv + NW * ((j + 1) / KSp)) * 16 < n_cols) {
              landed(std::integral_constant<int, at + 1>{});
              static_for<NMMA>([&](auto Fc) __attribute__((always_inline)) {
                constexpr int f = decltype(Fc)::value;
                read_w(std::integral_constant<int, j + 1>{}, f / NF, f % NF);
                if constexpr (KSp > 1) read_o(std::integral_constant<int, j + 1>{}, f / NF, f % NF);
              });
            }
          }
        }
        if constexpr (k == KSp - 1) {
          if (here) epi(std::integral_constant<int, i>{});
        }
      });
    };
    // where this lane's four columns of block 0 lie: MLP rows, residual rows, biases, gate; block i is a constant further
    auto put_at = [&](int row) __attribute__((always_inline)) {
      const int byte = n0 * ES;
      return hid + (byte >> 7) * (BMR * 128) + row * 128 + ((((byte >> 4) & 7) ^ ((row >> 1) & 7)) << 4) + (byte & 15);
    };
    const float* const bias_l = sbias + n0;
    auto bias_of = [&](int at) __attribute__((always_inline)) { return *reinterpret_cast<const float4*>(bias_l + at); };
    auto residual = [&](auto Ic, int bias_off, int gate_off) __attribute__((always_inline)) {
      constexpr int n = decltype(Ic)::value * 128;
      const float4 bb = bias_of(bias_off + n);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        float4* x = reinterpret_cast<float4*>(reinterpret_cast<char*>(x_at(r * 16 + l16, n0 >> 2)) + n * 4);
        float4 v = *x;
        if constexpr (HEAD) {  // image rows: position + (product + bias)
          const int m = min(m0 + r * 16 + l16, M - 1);
          if (m - a.by_L.div(m) * L < a.n_img) {
            v.x = (acc[r][0] + bb.x) + v.x;
            v.y = (acc[r][1] + bb.y) + v.y;
            v.z = (acc[r][2] + bb.z) + v.z;
            v.w = (acc[r][3] + bb.w) + v.w;
            *x = v;
          }
        } else {  // rows += gate * (product + bias)
          const float4 g = *reinterpret_cast<const float4*>(smods + srow[r] + n0 + (gate_off + n));
          v.x = fmaf(g.x, acc[r][0] + bb.x, v.x);
          v.y = fmaf(g.y, acc[r][1] + bb.y, v.y);
          v.z = fmaf(g.z, acc[r][2] + bb.z, v.z);
          v.w = fmaf(g.w, acc[r][3] + bb.w, v.w);
          *x = v;
        }
      }
    };
    run(std::integral_constant<int, 0>{}, std::integral_constant<int, NB0>{}, std::integral_constant<int, KS0>{}, HEAD ? hid : act, HC,
        [&](auto Ic) __attribute__((always_inline)) { residual(Ic, 0, 0); });
    __syncthreads();
    layer_norm(HEAD ? 0 : HC, HEAD);
    __syncthreads();
    if constexpr (!HEAD) {
      run(std::integral_constant<int, S1>{}, std::integral_constant<int, NB1>{}, std::integral_constant<int, KS>{}, act, 4 * HC,
          [&](auto Ic) __attribute__((always_inline)) {
            constexpr int i = decltype(Ic)::value;
            const float4 bb = bias_of(HC + i * 128);
#pragma unroll
            for (int r = 0; r < RT; ++r)
              store4<T>(reinterpret_cast<T*>(put_at(r * 16 + l16) + i * (ES * BMR * 128)), gelu_tanh_f(acc[r][0] + bb.x), gelu_tanh_f(acc[r][1] + bb.y),
                        gelu_tanh_f(acc[r][2] + bb.z), gelu_tanh_f(acc[r][3] + bb.w));
          });
      __syncthreads();
      run(std::integral_constant<int, S2>{}, std::integral_constant<int, NB2>{}, std::integral_constant<int, KS2>{}, hid, HC,
          [&](auto Ic) __attribute__((always_inline)) { residual(Ic, 5 * HC, 3 * HC); });
      __syncthreads();
      layer_norm(4 * HC, !LAST);
      __syncthreads();
    }
    run(std::integral_constant<int, S3>{}, std::integral_constant<int, NB3>{}, std::integral_constant<int, KS>{}, act, ntail,
        [&](auto Ic) __attribute__((always_inline)) {
          constexpr int n = decltype(Ic)::value * 128;
          const float4 bb = bias_of((HEAD ? HC : 6 * HC) + n);
          const float cs = n0 + n < a.qcols ? a.qscale : 1.f;
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const int m = m0 + r * 16 + l16;
            const float v0 = acc[r][0] + bb.x, v1 = acc[r][1] + bb.y, v2 = acc[r][2] + bb.z, v3 = acc[r][3] + bb.w;
            if constexpr (LAST) {
              const int b = a.by_L.div(min(m, M - 1)), tok = m < M ? m - b * L : a.n_img;
              if (tok < a.n_img && n0 < ntail) a.fin.scatter_unpatch({(long long)svrow[b - b_first] * a.D, nullptr, tok}, n0, v0, v1, v2, v3);
            } else {
              if (m < M) store4<T>(reinterpret_cast<T*>(a.qkv) + (size_t)m * (3 * HC) + n0 + n, v0 * cs, v1 * cs, v2 * cs, v3 * cs);
            }
          }
        });
    return;
  } else {
  gather();
  // ---- phases: 0 the first product, 1 FC1, 2 FC2, 3 the tail (head: 0 and 3).  One has N columns, 16 a block, dealt out to the
  // waves; a row of its weights is kb bytes, in steps of SPS times 128.
  constexpr int STEP_B = SPS * 2048, PD = RING_B / STEP_B;
  int slot = 0;
  struct Phase {
    const char* w;
    int N, kb, steps;
  };
  auto phase = [&](int ph) {  // (from the kernel's arguments: copies in scalar registers cost 11 to 36 spilled ones, bf16 hidden 64, 28 200 rows 280 -> 296 us)
    Phase p;
    p.w = reinterpret_cast<const char*>(ph == 0 ? a.w0 : ph == 1 ? a.fc1_w : ph == 2 ? a.fc2_w : a.tail_w);
    p.N = ph == 1 ? a.RH : ph == 3 ? a.NTAIL : H;
    p.kb = (ph == 2 ? a.RH : KIND == ROWS_HEAD && ph == 0 ? a.pd : H) * ES;
    p.steps = (p.kb + SPS * 128 - 1) / (SPS * 128);
    return p;
  };
  // The fetch cursor: place in the wave's list of column blocks of all phases.  A load fills eight rows (lane = 8 row + slot), slot
  // s of row r from chunk s ^ ((r >> 1) & 7).  Only a patch vector may end inside a step: what lies past its end is fetched from
  // the start of the row.
  char* const my_ring = lds + a.o_ring + wv * RING_B;
  const unsigned ring = (unsigned)(uintptr_t)BR_LPTR(my_ring);
  const int lrow = lane >> 3, chunk0 = ((lane & 7) ^ ((lrow >> 1) & 7)) * 16, chunk1 = chunk0 ^ 64;
  int f_ph = 0, f_cb = wv, f_left, f_off, f_slot = 0;
  unsigned f_row0, f_row1;
  Phase fp = phase(0);
  auto f_block = [&]() __attribute__((always_inline)) {  // to a block that exists; at the end of the list a last one stays
    while (f_cb * 16 >= fp.N && f_ph < 3) {
      f_ph = KIND == ROWS_HEAD ? 3 : f_ph + 1;
      fp = phase(f_ph);
      f_cb = wv;
    }
    f_row0 = (unsigned)min(f_cb * 16 + lrow, fp.N - 1) * (unsigned)fp.kb;
    f_row1 = (unsigned)min(f_cb * 16 + 8 + lrow, fp.N - 1) * (unsigned)fp.kb;
    f_off = 0;
    f_left = fp.steps;
  };
  auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < SPS; ++u) {
      const unsigned dst = ring + f_slot + u * 2048;
      const int at0 = f_off + u * 128 + chunk0, at1 = f_off + u * 128 + chunk1;
      const unsigned o0 = f_row0 + (KIND != ROWS_HEAD || at0 < fp.kb ? at0 : 0), o1 = f_row1 + (KIND != ROWS_HEAD || at1 < fp.kb ? at1 : 0);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(o0), "s"(fp.w) : "memory", "m0");
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst + 1024), "v"(o1), "s"(fp.w) : "memory", "m0");
    }
    f_slot = (f_slot + STEP_B) & (RING_B - 1);
    f_off += SPS * 128;
    if (--f_left == 0) {
      f_cb += NW;
      f_block();
    }
  };
  long long vo[RT];  // last: where the sample of this lane's rows starts in v
  int vtok[RT];
  if constexpr (KIND == ROWS_LAST) {
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int m = m0 + r * 16 + l16, b = a.by_L.div(min(m, M - 1));
      vtok[r] = m < M ? m - b * L : a.n_img;
      vo[r] = (long long)a.fin.a.vrows[b] * a.D;
    }
  }
  f_block();
#pragma unroll 1
  for (int i = 0; i < PD; ++i) fetch();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

#pragma unroll 1
  for (int ph = 0; ph < 4; ph = KIND == ROWS_HEAD ? ph + 3 : ph + 1) {
    const Phase p = phase(ph);
    const char* const op = ph == 2 || (KIND == ROWS_HEAD && ph == 0) ? hid : act;
    frag o[SPS][RT][NF];
    const int bias_at = ph == 0 ? 0 : KIND == ROWS_HEAD || ph == 1 ? H : ph == 2 ? H + RH : 2 * H + RH;
#pragma unroll 1
    for (int cb = wv; cb * 16 < p.N; cb += NW) {
      f32x4 acc[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
      const char* os = op;
#pragma unroll 1
      for (int k = 0; k < p.steps; ++k) {
        // the step has landed (PD - 1 younger ones may be under way), its fragments are read, its slot is refilled
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * SPS * (PD - 1)) : "memory");
        frag w[SPS][NF];
#pragma unroll
        for (int u = 0; u < SPS; ++u)
#pragma unroll
          for (int i = 0; i < NF; ++i) w[u][i] = *reinterpret_cast<const frag*>(my_ring + slot + u * 2048 + (fo ^ (i * FLIP)));
        if (p.steps > 1 || cb == wv) {  // (rows of one step stay in registers)
#pragma unroll
          for (int u = 0; u < SPS; ++u)
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
              for (int i = 0; i < NF; ++i) o[u][r][i] = *reinterpret_cast<const frag*>(os + (u * RT + r) * 2048 + (fo ^ (i * FLIP)));
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < SPS; ++u)
#pragma unroll
          for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r] = GemmFrag16<T>::mma(w[u][i], o[u][r][i], acc[r]);
        fetch();
        slot = (slot + STEP_B) & (RING_B - 1);
        os += SPS * BMR * 128;
      }
      const int n = cb * 16 + lq * 4;
      if (n < p.N) {
        const float4 bb = bias4(bias_at + n);
        if (ph == 1) {  // hidden row = GELU(product + bias)
#pragma unroll
          for (int r = 0; r < RT; ++r)
            put(hid, r * 16 + l16, n, gelu_tanh_f(acc[r][0] + bb.x), gelu_tanh_f(acc[r][1] + bb.y), gelu_tanh_f(acc[r][2] + bb.z),
                gelu_tanh_f(acc[r][3] + bb.w));
        } else if (ph == 3) {
          const float cs = n < a.qcols ? a.qscale : 1.f;
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const int m = m0 + r * 16 + l16;
            const float v0 = acc[r][0] + bb.x, v1 = acc[r][1] + bb.y, v2 = acc[r][2] + bb.z, v3 = acc[r][3] + bb.w;
            if constexpr (KIND == ROWS_LAST) {
              if (vtok[r] < a.n_img) a.fin.scatter_unpatch({vo[r], nullptr, vtok[r]}, n, v0, v1, v2, v3);
            } else {
              if (m < M) store4<T>(reinterpret_cast<T*>(a.qkv) + (size_t)m * NTAIL + n, v0 * cs, v1 * cs, v2 * cs, v3 * cs);
            }
          }
        } else if (KIND == ROWS_HEAD) {  // image rows: position + (product + bias)
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const int m = min(m0 + r * 16 + l16, M - 1);
            if (m - a.by_L.div(m) * L < a.n_img) {
              float4* x = x_at(r * 16 + l16, n >> 2);
              float4 v = *x;
              v.x = (acc[r][0] + bb.x) + v.x;
              v.y = (acc[r][1] + bb.y) + v.y;
              v.z = (acc[r][2] + bb.z) + v.z;
              v.w = (acc[r][3] + bb.w) + v.w;
              *x = v;
            }
          }
        } else {  // rows += gate * (product + bias); a sample's vectors: gate, shift, scale, gate of the MLP, shift, scale of the tail
          const int gate = ph == 0 ? 0 : 3 * H;
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            const float4 g = *reinterpret_cast<const float4*>(smods + srow[r] + gate + n);
            float4* x = x_at(r * 16 + l16, n >> 2);
            float4 v = *x;
            v.x = fmaf(g.x, acc[r][0] + bb.x, v.x);
            v.y = fmaf(g.y, acc[r][1] + bb.y, v.y);
            v.z = fmaf(g.z, acc[r][2] + bb.z, v.z);
            v.w = fmaf(g.w, acc[r][3] + bb.w, v.w);
            *x = v;
          }
        }
      }
    }
    if (ph == 3) break;
    __syncthreads();
    if (ph == 1) continue;
    layer_norm(KIND == ROWS_HEAD ? 0 : ph == 0 ? H : 4 * H, KIND == ROWS_HEAD || (KIND == ROWS_BODY && ph == 2));
    __syncthreads();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the fetches past the end of the list
  }
}

namespace {
struct RowsLds {
  int act, hid, mods, bias, vrow, ring, total;
};
// KIND's vectors of a sample: 2 H floats (head) or 6 H; samples that 16 rt rows can touch: at most (16 rt - 2) / L + 2.  ring: bytes of a wave's
// weights in flight in a form for a hidden size, which also keeps the samples' places in v; 0: the form for any sizes
RowsLds rows_lds(const br_model* m, int rt, bool head, int ntail, int ring) {
  const int es = m->cfg.dtype == BR_BF16 ? 2 : 4, rows = 16 * rt, samples = std::min(rows, (rows - 2) / m->L + 2);
  const size_t op = (size_t)rows * align_up((size_t)m->H * es, 128);
  const size_t hid = (size_t)rows * align_up((size_t)(head ? m->pd : m->R * m->H) * es, 256);
  const size_t mods = align_up((size_t)samples * (head ? 2 : 6) * m->H * 4, 1024);
  const size_t bias = align_up((size_t)(head ? m->H + ntail : 2 * m->H + m->R * m->H + ntail) * 4, 1024);
  RowsLds l;
  size_t o = (size_t)rows * m->H * 4;
  l.act = (int)o;
  l.hid = (int)(o += op);
  l.mods = (int)(o += hid);
  l.bias = (int)(o += mods);
  l.vrow = (int)(o += bias);
  l.ring = (int)(o += ring ? 256 : 0);
  l.total = (int)std::min<size_t>(o + (size_t)NW * (ring ? ring : RING_B), 1 << 30);
  return l;
}
}  // namespace

// Row tiles of 16 per workgroup for M rows, 0: the separate kernels.  One tile while that gives every compute unit at most one
// workgroup, two beyond (the weights are then streamed half as often), as far as the rows fit the LDS.  Whole velocity calls in us,
// separate kernels -> fused:  bf16 hidden 64: 55 rows 105 -> 73, 2940 190 -> 117, 49 000 531 -> 400;  128: 279 rows 91 -> 68,
// 13 500 300 -> 190, 55 700 550 -> 442;  192: 55 rows 122 -> 101;  256 (one tile only): 248 rows 169 -> 158, 3968 237 -> 172.
// fp32 64: 24 rows 81 -> 64, 26 400 410 -> 358;  128 (one tile only): 762 rows 670 -> 655, 1905 177 -> 161.  Wider rows stream
// more weights than the launches cost.  fp32 96 in two tiles keeps the separate kernels where the last round of workgroups is less than a
// quarter full (three blocks, velocity time fused / separate: 8280 rows 1.04, 9984 1.03, 24 984 1.01, 49 992 1.03; 12 000 0.86, 64 992
// 0.98); narrower rows win there too (8280 rows: bf16 64 0.71, 128 0.77, fp32 32 0.78, 64 0.87).
int rows_fused_tiles(const br_model* m, const FwdBuffers& fb, int M) {
  const bool bf = m->cfg.dtype == BR_BF16;
  const uintptr_t p = (uintptr_t)fb.x | (uintptr_t)fb.mods | (uintptr_t)fb.xn | (uintptr_t)fb.qkv | (uintptr_t)fb.cond_emb;
  if ((p & 15) != 0 || m->H * (bf ? 2 : 4) % 128 != 0 || m->H > (bf ? 256 : 128) || M > 65535) return 0;  // (FastDiv: M L < 2^32)
  const int cu = device_cu_count(), rt = cdiv(M, 16) <= cu ? 1 : 2;
  if (rt == 2 && m->H * (bf ? 2 : 4) > 256 && (cdiv(M, 32) - 1) % cu + 1 < cu / 4) return 0;
  for (int head = 0; head < 2; ++head)
    if (rows_lds(m, rt, head, std::max(3 * m->H, m->pd), 0).total > LDS_LIMIT) return 0;
  return rt;
}

// block < 0: the head of the network; else the rows of block `block` and the tail behind it.
br_status launch_block_rows(const br_model* m, const FwdBuffers& fb, const SampleMap& sm, int b0, int B, int v_rows_mode,
                            const float* z, float* v_out, int block, int rt, hipStream_t st) {
  const br_model_cfg& c = m->cfg;
  const size_t es = c.dtype == BR_BF16 ? 2 : 4;
  const int H = m->H, RH = m->R * H, k = std::max(block, 0);
  const bool head = block < 0, last = block == m->NB - 1;
  auto w = [&](int id, size_t per_block, int i) { return (const char*)m->w[id] + (size_t)i * per_block * es; };
  auto bias = [&](int id, size_t per_block, int i) { return (const float*)m->w[id] + (size_t)i * per_block; };
  RowsArgs a{};
  a.M = B * m->L; a.L = m->L; a.n_img = m->n_img;
  a.H = H; a.RH = RH;
  a.by_L = FastDiv(m->L); a.by_H4 = FastDiv(H / 4);
  a.x = fb.x;
  a.mods = fb.mods; a.A = m->A;
  a.mods_off = head ? 0 : k * 6 * H + 2 * H;
  a.by_mq = FastDiv((head ? 2 * H : 6 * H) / 4);
  a.modmap = fb.modmap;
  a.attn = fb.xn;
  a.D = m->D;
  if (head) {
    a.w0 = m->w[BR_W_PATCH_W]; a.b0 = (const float*)m->w[BR_W_PATCH_B];
    a.sm = sm; a.s0 = b0; a.B = B; a.v_rows_mode = v_rows_mode;
    a.modmap_out = fb.modmap; a.vrows = fb.vrows;
    a.z = z; a.pos = (const float*)m->w[BR_W_POS]; a.cond_emb = fb.cond_emb;
    a.pd = m->pd; a.lt = c.latent_t; a.lh = c.latent_h; a.lw = c.latent_w;
    a.pt = c.patch_t; a.ph = c.patch_h; a.pw = c.patch_w; a.gh = m->gh; a.gw = m->gw; a.Nc = m->Nc;
    a.by_pd = FastDiv(m->pd); a.by_pw = FastDiv(c.patch_w); a.by_ph = FastDiv(c.patch_h); a.by_pt = FastDiv(c.patch_t);
    a.by_gw = FastDiv(m->gw); a.by_gh = FastDiv(m->gh);
  } else {
    a.w0 = w(BR_W_PROJ_W, (size_t)H * H, k); a.b0 = bias(BR_W_PROJ_B, H, k);
    a.fc1_w = w(BR_W_FC1_W, (size_t)RH * H, k); a.fc1_b = bias(BR_W_FC1_B, RH, k);
    a.fc2_w = w(BR_W_FC2_W, (size_t)RH * H, k); a.fc2_b = bias(BR_W_FC2_B, H, k);
  }
  if (last) {
    a.NTAIL = m->pd;
    a.tail_w = m->w[BR_W_FINAL_W]; a.tail_b = (const float*)m->w[BR_W_FINAL_B];
    EpiArgs& e = a.fin.a;
    e.out = v_out; e.vrows = fb.vrows;
    e.lt = c.latent_t; e.lh = c.latent_h; e.lw = c.latent_w;
    e.pt = c.patch_t; e.ph = c.patch_h; e.pw = c.patch_w; e.gh = m->gh; e.gw = m->gw;
  } else {
    a.NTAIL = 3 * H;
    a.tail_w = w(BR_W_QKV_W, (size_t)3 * H * H, block + 1); a.tail_b = bias(BR_W_QKV_B, (size_t)3 * H, block + 1);
    a.qkv = fb.qkv;
    if (c.dtype == BR_BF16) {  // (as in forward())
      a.qcols = H;
      a.qscale = (float)(1.4426950408889634 / sqrt((double)m->DH));
    }
  }
  const double flops = 2.0 * a.M * H * ((head ? m->pd : H + 2.0 * RH) + a.NTAIL);
  ProfScope ps(st, PROF_BLOCK_ROWS + (head ? 0 : last ? 2 : 1), flops, c.dtype == BR_BF16);  // (only bf16 networks are instrumented)
  auto go = [&](auto Tc, auto RTc, auto SPSc, auto HCc) {
    constexpr int R_ = decltype(RTc)::value, S_ = decltype(SPSc)::value, H_ = decltype(HCc)::value;
    using T = decltype(Tc);
    const RowsLds l = rows_lds(m, rt, head, a.NTAIL, H_ ? rows_ring(sizeof(T), H_, R_) : 0);
    a.o_act = l.act; a.o_hid = l.hid; a.o_mods = l.mods; a.o_bias = l.bias; a.o_vrow = l.vrow; a.o_ring = l.ring;
    const dim3 g(cdiv(a.M, 16 * R_)), b(NT);
    if (head) hipLaunchKernelGGL((block_rows_kernel<T, R_, S_, ROWS_HEAD, H_>), g, b, l.total, st, a);
    else if (last) hipLaunchKernelGGL((block_rows_kernel<T, R_, S_, ROWS_LAST, H_>), g, b, l.total, st, a);
    else hipLaunchKernelGGL((block_rows_kernel<T, R_, S_, ROWS_BODY, H_>), g, b, l.total, st, a);
  };
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  // The form for the hidden size where it has one and everything fits (short samples have more modulation vectors), else the one for any sizes;
  // steps of 256 bytes where the rows of all weights are whole numbers of them (the patch vector is padded).
  auto form = [&](auto Tc, auto RTc, auto HCc) {
    constexpr int H_ = decltype(HCc)::value, ES = (int)sizeof(decltype(Tc));
    using SPSc = std::integral_constant<int, H_ * ES % 256 == 0 ? 2 : 1>;
    if (m->R == 4 && m->pd * ES <= 256 && m->pd <= 128 && rows_lds(m, rt, head, a.NTAIL, rows_ring(ES, H_, decltype(RTc)::value)).total <= LDS_LIMIT)
      go(Tc, RTc, SPSc{}, HCc);
    else go(Tc, RTc, SPSc{}, std::integral_constant<int, 0>{});
  };
  auto size = [&](auto Tc, auto RTc) {  // (H ES is 128, 256, 384 or 512: rows_fused_tiles)
    constexpr int U = 128 / (int)sizeof(decltype(Tc));
    if (H == U) form(Tc, RTc, std::integral_constant<int, U>{});
    else if (H == 2 * U) form(Tc, RTc, std::integral_constant<int, 2 * U>{});
    else if (H == 3 * U) form(Tc, RTc, std::integral_constant<int, 3 * U>{});
    else if (decltype(RTc)::value == 1) form(Tc, I1{}, std::integral_constant<int, 4 * U>{});
    else go(Tc, RTc, I2{}, std::integral_constant<int, 0>{});
  };
  auto rows = [&](auto Tc) { rt == 1 ? size(Tc, I1{}) : size(Tc, I2{}); };
  if (c.dtype == BR_BF16) rows(bf16{});
  else rows(float{});
  BR_LAUNCH_CHECK();
  return BR_OK;
}

}  // namespace br
