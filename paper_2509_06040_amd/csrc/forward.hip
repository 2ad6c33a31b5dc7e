// Model handle, workspace plan and one evaluation of the velocity network.
#include <algorithm>
#include <new>

#include "common.h"
#include "dispatch.h"
#include "dit.h"
#include "kernels.h"
#include "prof.h"

namespace br {
br_status launch_batch_prologue(const br_model* m, const FwdBuffers& fb, const SampleMap& sm, int b0, int B, int v_rows_mode,
                                const float* z, hipStream_t st);

static size_t esize(const br_model* m) { return m->cfg.dtype == BR_BF16 ? 2 : 4; }

size_t plan_workspace(const br_model* m, int n_cond, int max_batch, long long v_rows, long long partial_floats,
                      long long plan_ints, FwdBuffers* fb, void* base) {
  size_t o = 0;
  char* p = reinterpret_cast<char*>(base);
  auto take = [&](size_t bytes) {
    void* r = p ? p + o : nullptr;
    o += align_up(bytes ? bytes : 1, 256);
    return r;
  };
  const size_t B = (size_t)max_batch, H = m->H, L = m->L, es = esize(m);
  FwdBuffers f;
  const size_t G = std::max<size_t>(B, (size_t)n_cond);  // modulation groups: at most one per sample
  f.modmap = (int*)take(B * 4);
  f.vrows = (int*)take(B * 4);
  f.h1 = (float*)take(G * H * 4);
  f.pooled = (float*)take((size_t)n_cond * m->cd * 4);
  take((size_t)n_cond * H * 4);  // unused: the sizes that callers were given, and the batches that fit them, stay what they are
  f.cvec = (float*)take(G * H * 4);
  f.mods = (float*)take(G * m->A * 4);
  f.cond_emb = (float*)take((size_t)n_cond * m->Nc * H * 4);
  f.x = (float*)take(B * L * H * 4);
  f.patches = take(B * m->n_img * m->pd * es);
  f.xn = take(B * L * H * es);
  f.qkv = take(B * L * 3 * H * es);
  f.hid = take(B * L * (size_t)m->R * H * es);
  f.v = (float*)take((size_t)v_rows * m->D * 4);
  f.sde_partials = (float*)take((size_t)partial_floats * 4);
  f.plan = (int*)take((size_t)plan_ints * 4);
  f.total = o;
  if (fb) *fb = f;
  return o;
}

br_status embed_cond(const br_model* m, const FwdBuffers& fb, const void* cond_tokens, int n_cond, hipStream_t st) {
  EpiArgs ea{};
  ea.bias = (const float*)m->w[BR_W_COND_B];
  ea.out = fb.cond_emb;
  ea.ldo = m->H;
  return launch_gemm(m->cfg.dtype, EPI_BIAS_F32, cond_tokens, m->cd, m->w[BR_W_COND_W], m->cd, n_cond * m->Nc, m->H, m->cd, ea, st);
}

br_status forward(const br_model* m, const FwdBuffers& fb, const SampleMap& sm, int b0, int B, int v_rows_mode,
                  const float* z_base, float* v_out, hipStream_t st) {
  const int H = m->H, L = m->L, dt = m->cfg.dtype;
  const size_t es = esize(m);
  br_status s;
#define BR_TRY(x) do { if ((s = (x)) != BR_OK) return s; } while (0)
  if (const int rt = rows_fused_tiles(m, fb, B * L)) {
    ProfChain chain(dt == BR_BF16);
    for (int k = -1; k < m->NB; ++k) {
      if (k >= 0) BR_TRY(launch_attention(dt, fb.qkv, fb.xn, B, L, m->NH, m->DH, dt == BR_BF16 ? 1 : 0, WarmRows{}, st));
      BR_TRY(launch_block_rows(m, fb, sm, b0, B, v_rows_mode, z_base, v_out, k, rt, st));
    }
    return BR_OK;
  }
  BR_TRY(launch_batch_prologue(m, fb, sm, b0, B, v_rows_mode, z_base, st));
  {
    EpiArgs ea{};
    ea.bias = (const float*)m->w[BR_W_PATCH_B];
    ea.out = fb.x;
    ea.ldo = H;
    ea.L = L;
    ea.n_img = m->n_img;
    ea.pos = (const float*)m->w[BR_W_POS];
    BR_TRY(launch_gemm(dt, EPI_PATCH_EMBED, fb.patches, m->pd, m->w[BR_W_PATCH_W], m->pd, B * m->n_img, H, m->pd, ea, st));
  }
  const int M = B * L;
  // rows r of the normalised, modulated stream (rows_per_sample of every sample) times W, in one launch where it fits
  auto ln_gemm = [&](int mode, int rows_per_sample, int shift, const void* W, int N, const EpiArgs& ea) -> br_status {
    const int rows = B * rows_per_sample;
    if (ln_gemm_fits(dt, rows, N, H, fb.x, fb.mods, m->A, shift, shift + H)) {
      const LnArgs ln{fb.x, rows_per_sample, L, fb.mods, m->A, shift, shift + H, fb.modmap};
      return launch_ln_gemm(dt, mode, ln, W, rows, N, H, ea, st);
    }
    const br_status e = launch_ln_modulate(dt, fb.x, fb.xn, rows, rows_per_sample, L, H, fb.mods, m->A, shift, shift + H, fb.modmap, st);
    return e != BR_OK ? e : launch_gemm(dt, mode, fb.xn, H, W, H, rows, N, H, ea, st);
  };
  const bool cold_weights = dt == BR_BF16 && !rule::weights_stay(((4.0 + 2.0 * m->R) * m->NB * H * H + (double)m->A * H) * es);
  // the bf16 block stack launches only instrumented kernels, back to back
  ProfChain chain(dt == BR_BF16);
  for (int k = 0; k < m->NB; ++k) {
    const int mo = k * 6 * H;
    const char* qkv_w = (const char*)m->w[BR_W_QKV_W] + (size_t)k * 3 * H * H * es;
    const char* proj_w = (const char*)m->w[BR_W_PROJ_W] + (size_t)k * H * H * es;
    const char* fc1_w = (const char*)m->w[BR_W_FC1_W] + (size_t)k * m->R * H * H * es;
    const char* fc2_w = (const char*)m->w[BR_W_FC2_W] + (size_t)k * m->R * H * H * es;
    {
      EpiArgs ea{};
      ea.bias = (const float*)m->w[BR_W_QKV_B] + (size_t)k * 3 * H;
      ea.out = fb.qkv;
      ea.ldo = 3 * H;
      if (dt == BR_BF16) {  // the attention kernel takes the scores in units of log2 e / sqrt(head dim)
        ea.qcols = H;
        ea.qscale = (float)(1.4426950408889634 / sqrt((double)m->DH));
      }
      BR_TRY(ln_gemm(EPI_BIAS, L, mo, qkv_w, 3 * H, ea));
    }
    WarmRows next;  // the weights that the block's other products and the next block's first one are about to stream
    if (cold_weights) {
      auto range = [&](int i, const char* p, size_t bytes) {
        next.p[i] = p;
        next.n16[i] = (unsigned)std::min<size_t>(bytes / 16, 1u << 24);
      };
      range(0, proj_w, (size_t)H * H * es);
      range(1, fc1_w, (size_t)m->R * H * H * es);
      range(2, fc2_w, (size_t)m->R * H * H * es);
      if (k + 1 < m->NB) range(3, qkv_w + (size_t)3 * H * H * es, (size_t)3 * H * H * es);
    }
    BR_TRY(launch_attention(dt, fb.qkv, fb.xn, B, L, m->NH, m->DH, dt == BR_BF16 ? 1 : 0, next, st));  // xn is free again: attention output
    {
      EpiArgs ea{};
      ea.bias = (const float*)m->w[BR_W_PROJ_B] + (size_t)k * H;
      ea.out = fb.x;
      ea.ldo = H;
      ea.mods = fb.mods;
      ea.A = m->A;
      ea.gate_off = mo + 2 * H;
      ea.condmap = fb.modmap;
      ea.L = L;
      BR_TRY(launch_gemm(dt, EPI_BIAS_GATE_RES, fb.xn, H, proj_w, H, M, H, H, ea, st));
    }
    {
      EpiArgs ea{};
      ea.bias = (const float*)m->w[BR_W_FC1_B] + (size_t)k * m->R * H;
      ea.out = fb.hid;
      ea.ldo = m->R * H;
      BR_TRY(ln_gemm(EPI_BIAS_GELU, L, mo + 3 * H, fc1_w, m->R * H, ea));
    }
    {
      EpiArgs ea{};
      ea.bias = (const float*)m->w[BR_W_FC2_B] + (size_t)k * H;
      ea.out = fb.x;
      ea.ldo = H;
      ea.mods = fb.mods;
      ea.A = m->A;
      ea.gate_off = mo + 5 * H;
      ea.condmap = fb.modmap;
      ea.L = L;
      BR_TRY(launch_gemm(dt, EPI_BIAS_GATE_RES, fb.hid, m->R * H, fc2_w, m->R * H, M, H, m->R * H, ea, st));
    }
  }
  const int mo = m->NB * 6 * H;
  {
    EpiArgs ea{};
    const br_model_cfg& c = m->cfg;
    ea.bias = (const float*)m->w[BR_W_FINAL_B];
    ea.out = v_out;
    ea.n_img = m->n_img;
    ea.vrows = fb.vrows;
    ea.D = m->D;
    ea.lt = c.latent_t; ea.lh = c.latent_h; ea.lw = c.latent_w;
    ea.pt = c.patch_t; ea.ph = c.patch_h; ea.pw = c.patch_w;
    ea.gh = m->gh; ea.gw = m->gw;
    BR_TRY(ln_gemm(EPI_UNPATCH, m->n_img, mo, m->w[BR_W_FINAL_W], m->pd, ea));
  }
#undef BR_TRY
  return BR_OK;
}

}  // namespace br

using namespace br;

extern "C" br_status br_model_create(const br_model_cfg* cfg, const void* const* weight_ptrs, int32_t n_ptrs,
                                     br_model** out) {
  BR_REQUIRE(cfg && weight_ptrs && out, BR_EINVAL, "br_model_create: NULL argument");
  BR_REQUIRE(n_ptrs == BR_W_COUNT, BR_EINVAL, "br_model_create: n_ptrs must be BR_W_COUNT");
  const br_model_cfg& c = *cfg;
  BR_REQUIRE(c.dtype == BR_F32 || c.dtype == BR_BF16, BR_EINVAL, "br_model_create: unknown dtype");
  BR_REQUIRE(c.n_blocks >= 1 && c.hidden >= 1 && c.n_heads >= 1 && c.mlp_ratio >= 1 && c.latent_c >= 1 &&
                 c.latent_t >= 1 && c.latent_h >= 1 && c.latent_w >= 1 && c.patch_t >= 1 && c.patch_h >= 1 &&
                 c.patch_w >= 1 && c.n_cond_tokens >= 1 && c.cond_dim >= 1,
             BR_EINVAL, "br_model_create: sizes must be positive");
  BR_REQUIRE(c.hidden % c.n_heads == 0, BR_ESHAPE, "br_model_create: hidden must be divisible by n_heads");
  BR_REQUIRE(c.latent_t % c.patch_t == 0 && c.latent_h % c.patch_h == 0 && c.latent_w % c.patch_w == 0, BR_ESHAPE,
             "br_model_create: latent dims must be divisible by the patch");
  const long long D = (long long)c.latent_c * c.latent_t * c.latent_h * c.latent_w;
  const int pd = c.latent_c * c.patch_t * c.patch_h * c.patch_w, dh = c.hidden / c.n_heads;
  BR_REQUIRE(D % 4 == 0, BR_ESHAPE, "br_model_create: latent size must be a multiple of 4");
  BR_REQUIRE(c.hidden % 8 == 0 && c.cond_dim % 8 == 0 && pd % 4 == 0, BR_ESHAPE,
             "br_model_create: hidden and cond_dim must be multiples of 8, patch dim of 4");
  if (c.dtype == BR_BF16) {
    BR_REQUIRE(dh == 64 || dh == 128, BR_ESHAPE, "br_model_create: bf16 head dim must be 64 or 128");
    BR_REQUIRE(c.hidden % 64 == 0 && c.cond_dim % 64 == 0 && pd % 64 == 0, BR_ESHAPE,
               "br_model_create: bf16 needs hidden, cond_dim and patch dim divisible by 64");
  } else {
    BR_REQUIRE(dh == 16 || dh == 32 || dh == 64 || dh == 128, BR_ESHAPE,
               "br_model_create: fp32 head dim must be 16, 32, 64 or 128");
  }
  for (int i = 0; i < BR_W_COUNT; ++i) {
    BR_REQUIRE(weight_ptrs[i] != nullptr, BR_EINVAL, "br_model_create: NULL weight pointer");
    BR_REQUIRE(((uintptr_t)weight_ptrs[i] & 15) == 0, BR_EINVAL, "br_model_create: weight pointers must be 16-byte aligned");
  }
  br_model* m = new (std::nothrow) br_model();
  BR_REQUIRE(m != nullptr, BR_ENOMEM, "br_model_create: out of host memory");
  m->cfg = c;
  for (int i = 0; i < BR_W_COUNT; ++i) m->w[i] = weight_ptrs[i];
  m->H = c.hidden; m->NB = c.n_blocks; m->NH = c.n_heads; m->DH = dh; m->R = c.mlp_ratio;
  m->gt = c.latent_t / c.patch_t; m->gh = c.latent_h / c.patch_h; m->gw = c.latent_w / c.patch_w;
  m->n_img = m->gt * m->gh * m->gw;
  m->pd = pd; m->Nc = c.n_cond_tokens; m->cd = c.cond_dim;
  m->L = m->n_img + m->Nc;
  m->A = c.n_blocks * 6 * c.hidden + 2 * c.hidden;
  m->D = D;
  *out = m;
  return BR_OK;
}

extern "C" void br_model_free(br_model* m) { delete m; }
