// Velocity-network internals: model handle, workspace plan, epilogues, launchers.
#pragma once
#include <type_traits>

#include "common.h"

typedef __bf16 bf16;

struct br_model {
  br_model_cfg cfg;
  const void* w[BR_W_COUNT];
  // derived
  int H, NB, NH, DH, R, n_img, pd, L, Nc, cd, A;  // A = NB*6H + 2H
  long long D;
  int gt, gh, gw;
};

namespace br {

// ---- epilogues of the GEMMs (fused bias / activation / gate / residual / scatter)
enum EpiMode {
  EPI_BIAS = 0,           // out[m, n] = acc + bias[n]                        (T out)
  EPI_BIAS_GELU = 1,      // out[m, n] = gelu_tanh(acc + bias[n])             (T out)
  EPI_BIAS_GATE_RES = 2,  // x[m, n] += gate[cond(m / L)][n] * (acc + bias)   (fp32 in place)
  EPI_PATCH_EMBED = 3,    // x[(m / n_img) L + m % n_img, n] = acc + bias + pos[m % n_img, n]
  EPI_BIAS_F32 = 4,       // out[m, n] = acc + bias[n]                        (fp32 out)
  EPI_UNPATCH = 5         // v[vrow(m / n_img)][latent index of (m % n_img, n)] = acc + bias
};

struct EpiArgs {
  const float* bias;
  void* out;
  int ldo;
  // gate / residual
  const float* mods;   // [n_cond, A]
  int A, gate_off;
  const int* condmap;  // [B]
  int L, n_img;
  const float* pos;    // [n_img, H]
  // unpatchify
  const int* vrows;    // [B] destination row of each sample in v
  long long D;
  int lt, lh, lw, pt, ph, pw, gh, gw;
  // EPI_BIAS: columns n < qcols (a multiple of 4) are multiplied by qscale after the bias.  The QKV
  // projection of the bf16 network writes q * log2(e) / sqrt(head dim) this way, rounded to bf16 once.
  int qcols;
  float qscale;
};

struct FwdBuffers {  // carved from the workspace
  int* modmap;    // sample -> modulation group (its adaLN vectors)
  int* vrows;     // sample -> row of v
  float *h1, *pooled, *cvec, *mods, *cond_emb, *x, *sde_partials;
  void *patches, *xn, *qkv, *hid;
  float* v;       // compact velocity [max_frontier, D] (rollout only)
  int* plan;      // br_logprob launch plan
  size_t total;
};

size_t plan_workspace(const br_model* m, int n_cond, int max_batch, long long v_rows, long long partial_floats,
                      long long plan_ints, FwdBuffers* fb, void* base);

// Times of the modulation groups: dev[g] (device array), or t[g / n_cond], several steps of n_cond conditions each.
constexpr int MAX_GROUP_STEPS = 64;
struct GroupTimes {
  const float* dev = nullptr;
  int n_cond = 1;
  float t[MAX_GROUP_STEPS] = {};
};
// adaLN vectors of the modulation groups g < G <= max(n_cond, max_batch) of the plan: condition gcond[g] (device
// array; nullptr: g % gt.n_cond) at the group's time.  They stay valid until the next call.  cond_tokens (the first call of an
// entry point; else nullptr): the tokens of all n_cond conditions, whose means every later call uses.
br_status conditioning(const br_model* m, const FwdBuffers& fb, const void* cond_tokens, int n_cond, const int* gcond, const GroupTimes& gt,
                       int G, hipStream_t st);
// One network evaluation of samples b0 .. b0 + B - 1 of `sm` (B <= max_batch of the plan): latent rows of z_base, groups of the
// last conditioning() call; v rows by v_rows_mode (1: the sample's row, 2: row of the batch, else: its index).
br_status forward(const br_model* m, const FwdBuffers& fb, const SampleMap& sm, int b0, int B, int v_rows_mode,
                  const float* z_base, float* v_out, hipStream_t st);
// Condition-token embedding, once per call.
br_status embed_cond(const br_model* m, const FwdBuffers& fb, const void* cond_tokens, int n_cond, hipStream_t st);

// ---- op launchers (dit_kernels.hip, gemm_bf16.hip, attn_bf16.hip)
br_status launch_gemm(int dtype, int mode, const void* A, int lda, const void* W, int ldw, int M, int N, int K,
                      const EpiArgs& ea, hipStream_t st);
// q_prescaled: the q third already carries the factor log2(e) / sqrt(DH) (bf16 only)
// next: memory that the launches behind this one read
struct WarmRows {
  static constexpr int RANGES = 4;
  const void* p[RANGES] = {};
  unsigned n16[RANGES] = {};  // 16-byte pieces
  int blocks = 0;
};
br_status launch_attention(int dtype, const void* qkv, void* out, int B, int L, int NH, int DH, int q_prescaled, const WarmRows& next,
                           hipStream_t st);
br_status launch_gemm_bf16(int mode, const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K,
                           const EpiArgs& ea, int variant, hipStream_t st);
br_status launch_gemm_small(int dtype, int mode, const void* A, int lda, const void* W, int ldw, int M, int N, int K,
                             const EpiArgs& ea, hipStream_t st);
br_status launch_gemm_f32(int mode, const float* A, int lda, const float* W, int ldw, int M, int N, int K,
                          const EpiArgs& ea, int variant, hipStream_t st);
bool gemm_f32_ring_supported(int mode, int K, int lda, int ldw);
// tiles of 16 rb rows (rb 2 .. 12) x 64 cb columns (cb 1, 2)
br_status launch_gemm_f32_ring(int mode, const float* A, int lda, const float* W, int ldw, int M, int N, int K, const EpiArgs& ea, int rb,
                               int cb, hipStream_t st);
// GEMM whose A operand is LayerNorm(x[src(r), :]) (1 + scale) + shift (rows as in launch_ln_modulate), for small problems.
struct LnArgs {
  const float* x;
  int rows_per_sample, L_in;
  const float* mods;
  int A, shift_off, scale_off;
  const int* condmap;
};
bool ln_gemm_fits(int dtype, int M, int N, int K, const void* x, const void* mods, int A, int shift_off, int scale_off);
br_status launch_ln_gemm(int dtype, int mode, const LnArgs& ln, const void* W, int M, int N, int K, const EpiArgs& ea,
                         hipStream_t st);
// The row-local part of a block (block_rows.hip): row tiles per workgroup for M rows (0: use the separate kernels), and the launch.
int rows_fused_tiles(const br_model* m, const FwdBuffers& fb, int M);
br_status launch_block_rows(const br_model* m, const FwdBuffers& fb, const SampleMap& sm, int b0, int B, int v_rows_mode,
                            const float* z, float* v_out, int block, int rt, hipStream_t st);
bool gemm_stream_supported(int mode, int K, size_t bytes_a, size_t bytes_w);
br_status launch_gemm_bf16_stream(int mode, const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K,
                                  const EpiArgs& ea, int height, int group_n, int row_block, hipStream_t st);
bool gemm_ring_supported(int mode, int height, int lda, int ldw);
br_status launch_gemm_bf16_ring(int mode, const bf16* A, int lda, const bf16* W, int ldw, int M, int N, int K,
                                const EpiArgs& ea, int height, int group_n, hipStream_t st);
br_status launch_attention_bf16(const bf16* qkv, bf16* out, int B, int L, int NH, int DH, int q_prescaled, const WarmRows& next, hipStream_t st);
br_status launch_attention_f32(const float* qkv, float* out, int B, int L, int NH, int DH, hipStream_t st);
br_status launch_ln_modulate(int dtype, const float* x, void* out, int n_rows, int rows_per_sample, int L_in, int H,
                             const float* mods, int A, int shift_off, int scale_off, const int* condmap,
                             hipStream_t st);

// Sum of the squares of four deviations from a row's mean, rounded in the same places wherever a row is normalised.
__device__ inline float sum_sq4(const float4& v, float mean) {
  const float a = v.x - mean, b = v.y - mean, c = v.z - mean, d = v.w - mean;
  return fmaf(a, a, b * b) + fmaf(c, c, d * d);
}

// Sum over groups of N consecutive lanes, at distances N / 2 ... 1 in turn (the order of __shfl_xor, without its trips to the LDS
// unit).  Rotations by 8, 4 of 16 lanes reach the lane that the exclusive-or reaches, or one that holds the same sum.
template <int N>
__device__ __forceinline__ float lanes_sum(float x) {
  static_assert(N >= 16, "whole rows of 16 lanes");
  if constexpr (N == 64) {
    const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    x = __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);
  }
  if constexpr (N >= 32) {
    const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    x = __builtin_bit_cast(float, (unsigned)p[0]) + __builtin_bit_cast(float, (unsigned)p[1]);
  }
  auto add = [&](auto CTRL) { x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(CTRL)::value, 0xf, 0xf, true)); };
  add(std::integral_constant<int, 0x128>{});  // row_ror:8
  add(std::integral_constant<int, 0x124>{});  // row_ror:4
  add(std::integral_constant<int, 0x4E>{});   // quad_perm [2,3,0,1]
  add(std::integral_constant<int, 0xB1>{});   // quad_perm [1,0,3,2]
  return x;
}

// ---- epilogue device code, shared by the fp32 and the MFMA GEMM
__device__ inline float gelu_tanh_f(float x) {
  // 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)), u = sqrt(2/pi) (x + 0.044715 x^3);
  // exp(-2u) = exp2(x (k1 + k3 x^2)), k1 = -2 sqrt(2/pi) log2(e), k3 = 0.044715 k1
  const float t = x * fmaf(x * x, -0.10294324f, -2.3022082f);
  return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(t));
}

template <typename T>
__device__ inline void store4(T* p, float a, float b, float c, float d);
template <>
__device__ inline void store4<float>(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
template <>
__device__ inline void store4<bf16>(bf16* p, float a, float b, float c, float d) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 v = {(bf16)a, (bf16)b, (bf16)c, (bf16)d};
  *reinterpret_cast<bf16x4*>(p) = v;
}

template <int MODE, typename T>
struct Epilogue {
  EpiArgs a;
  struct Row {
    long long o;       // element offset of the output row
    const float* aux;  // gate row / pos row
    int tok;
  };
  __device__ inline Row row(int m) const {
    Row r;
    r.aux = nullptr;
    r.tok = 0;
    if (MODE == EPI_BIAS_GATE_RES) {
      r.o = (long long)m * a.ldo;
      r.aux = a.mods + (size_t)a.condmap[m / a.L] * a.A + a.gate_off;
    } else if (MODE == EPI_PATCH_EMBED) {
      const int b = m / a.n_img, tok = m - b * a.n_img;
      r.o = ((long long)b * a.L + tok) * a.ldo;
      r.aux = a.pos + (size_t)tok * a.ldo;
    } else if (MODE == EPI_UNPATCH) {
      const int b = m / a.n_img;
      r.tok = m - b * a.n_img;
      r.o = (long long)a.vrows[b] * a.D;
    } else {
      r.o = (long long)m * a.ldo;
    }
    return r;
  }
  // rows per sample when the row mapping depends on the sample, else 0
  __device__ inline int rows_per_sample() const {
    return MODE == EPI_BIAS_GATE_RES ? a.L : (MODE == EPI_PATCH_EMBED || MODE == EPI_UNPATCH) ? a.n_img : 0;
  }
  // ---- staged interface of the MFMA GEMM epilogue.  One hardware counter tracks a wave's
  // loads and stores in issue order, so a load issued after a store cannot be waited for
  // without also waiting for the store's write acknowledgement.  Whatever a tile's rows need
  // from memory is therefore fetched ahead of the stores: column constants and per-sample
  // constants once per tile, the per-row addend a few rows ahead.
  struct SampleC {
    float4 gate;  // gate[b, n..n+3] of the gated residual
    long long o;  // output offset of the sample (patch embedding, unpatchify)
  };
  static constexpr bool kHasAddend = MODE == EPI_BIAS_GATE_RES || MODE == EPI_PATCH_EMBED;
  __device__ inline float4 bias4(int n) const { return *reinterpret_cast<const float4*>(a.bias + n); }
  // EPI_BIAS: factor of the four columns n..n+3 (n % 4 == 0)
  __device__ inline float colscale(int n) const { return n < a.qcols ? a.qscale : 1.f; }
  __device__ inline SampleC sample_consts(int b, int n) const {
    SampleC s;
    s.gate = make_float4(0.f, 0.f, 0.f, 0.f);
    s.o = 0;
    if (MODE == EPI_BIAS_GATE_RES)
      s.gate = *reinterpret_cast<const float4*>(a.mods + (size_t)a.condmap[b] * a.A + a.gate_off + n);
    else if (MODE == EPI_PATCH_EMBED)
      s.o = (long long)b * a.L * a.ldo;
    else if (MODE == EPI_UNPATCH)
      s.o = (long long)a.vrows[b] * a.D;
    return s;
  }
  // what is added to row m (token tok of its sample) at columns n..n+3: the residual stream
  // or the position embedding
  __device__ inline float4 addend(int m, int tok, int n) const {
    if (MODE == EPI_BIAS_GATE_RES)
      return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.out) + (long long)m * a.ldo + n);
    if (MODE == EPI_PATCH_EMBED) return *reinterpret_cast<const float4*>(a.pos + (size_t)tok * a.ldo + n);
    return make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // store() on operands already in registers
  __device__ inline void finish(int m, int tok, int n, float v0, float v1, float v2, float v3, const float4& bb,
                                const SampleC& sc, const float4& add) const {
    v0 += bb.x; v1 += bb.y; v2 += bb.z; v3 += bb.w;
    if (MODE == EPI_BIAS) {
      const float cs = colscale(n);
      store4<T>(reinterpret_cast<T*>(a.out) + (long long)m * a.ldo + n, v0 * cs, v1 * cs, v2 * cs, v3 * cs);
    } else if (MODE == EPI_BIAS_GELU) {
      store4<T>(reinterpret_cast<T*>(a.out) + (long long)m * a.ldo + n, gelu_tanh_f(v0), gelu_tanh_f(v1),
                gelu_tanh_f(v2), gelu_tanh_f(v3));
    } else if (MODE == EPI_BIAS_GATE_RES) {
      store4<float>(reinterpret_cast<float*>(a.out) + (long long)m * a.ldo + n, fmaf(sc.gate.x, v0, add.x),
                    fmaf(sc.gate.y, v1, add.y), fmaf(sc.gate.z, v2, add.z), fmaf(sc.gate.w, v3, add.w));
    } else if (MODE == EPI_PATCH_EMBED) {
      store4<float>(reinterpret_cast<float*>(a.out) + sc.o + (long long)tok * a.ldo + n, v0 + add.x, v1 + add.y,
                    v2 + add.z, v3 + add.w);
    } else if (MODE == EPI_BIAS_F32) {
      store4<float>(reinterpret_cast<float*>(a.out) + (long long)m * a.ldo + n, v0, v1, v2, v3);
    } else {
      Row r;
      r.o = sc.o;
      r.aux = nullptr;
      r.tok = tok;
      scatter_unpatch(r, n, v0, v1, v2, v3);
    }
  }
  // EPI_UNPATCH: token (tt, th, tw) raster, element (c, dt, dh, dw).  The place in the latent is a sum of
  // a part of the column and a part of the token, so a caller that walks rows at fixed columns keeps
  // the former.  Elements of one patch row are neighbours: with an even patch width they leave in pairs.
  __device__ inline void scatter_unpatch(const Row& r, int n, float v0, float v1, float v2, float v3) const {
    const int tw = r.tok % a.gw, th = (r.tok / a.gw) % a.gh, tt = r.tok / (a.gw * a.gh);
    float* v = reinterpret_cast<float*>(a.out) + r.o + ((long long)tt * a.pt * a.lh + th * a.ph) * a.lw + tw * a.pw;
    const float vals[4] = {v0, v1, v2, v3};
    long long at[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int el = n + e;
      const int dw = el % a.pw, dh = (el / a.pw) % a.ph, dt = (el / (a.pw * a.ph)) % a.pt,
                c = el / (a.pw * a.ph * a.pt);
      at[e] = (((long long)c * a.lt + dt) * a.lh + dh) * a.lw + dw;
    }
    if (a.pw % 2 == 0 && (reinterpret_cast<uintptr_t>(a.out) & 7) == 0) {
      *reinterpret_cast<float2*>(v + at[0]) = make_float2(vals[0], vals[1]);
      *reinterpret_cast<float2*>(v + at[2]) = make_float2(vals[2], vals[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[at[e]] = vals[e];
    }
  }
  // four consecutive output columns n..n+3 (n % 4 == 0)
  __device__ inline void store(const Row& r, int n, float v0, float v1, float v2, float v3) const {
    const float4 bb = *reinterpret_cast<const float4*>(a.bias + n);
    v0 += bb.x; v1 += bb.y; v2 += bb.z; v3 += bb.w;
    if (MODE == EPI_BIAS) {
      const float cs = colscale(n);
      store4<T>(reinterpret_cast<T*>(a.out) + r.o + n, v0 * cs, v1 * cs, v2 * cs, v3 * cs);
    } else if (MODE == EPI_BIAS_GELU) {
      store4<T>(reinterpret_cast<T*>(a.out) + r.o + n, gelu_tanh_f(v0), gelu_tanh_f(v1), gelu_tanh_f(v2),
                gelu_tanh_f(v3));
    } else if (MODE == EPI_BIAS_GATE_RES) {
      float* x = reinterpret_cast<float*>(a.out) + r.o + n;
      const float4 g = *reinterpret_cast<const float4*>(r.aux + n);
      float4 xv = *reinterpret_cast<float4*>(x);
      xv.x = fmaf(g.x, v0, xv.x); xv.y = fmaf(g.y, v1, xv.y); xv.z = fmaf(g.z, v2, xv.z); xv.w = fmaf(g.w, v3, xv.w);
      *reinterpret_cast<float4*>(x) = xv;
    } else if (MODE == EPI_PATCH_EMBED) {
      const float4 p = *reinterpret_cast<const float4*>(r.aux + n);
      store4<float>(reinterpret_cast<float*>(a.out) + r.o + n, v0 + p.x, v1 + p.y, v2 + p.z, v3 + p.w);
    } else if (MODE == EPI_BIAS_F32) {
      store4<float>(reinterpret_cast<float*>(a.out) + r.o + n, v0, v1, v2, v3);
    } else {
      scatter_unpatch(r, n, v0, v1, v2, v3);
    }
  }
};

}  // namespace br
