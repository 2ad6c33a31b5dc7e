// Velocity network: the memory-bound and small kernels (batch prologue, conditioning path, LayerNorm-modulate) and the
// dispatch by type to the GEMMs (gemm_bf16.hip, gemm_f32.hip) and the attention (attn_bf16.hip, attn_f32.hip).
#include <type_traits>

#include "common.h"
#include "dit.h"
#include "prof.h"

namespace br {

template <typename T>
__device__ inline float to_f(T v) { return (float)v; }

// ------------------------------------------------------------ batch prologue
// What a batch needs before its first GEMM, in one launch (a launch costs about 4 us between dependent small kernels,
// the work of each of these parts less than one at a few samples):
//  - patches[(b n_img + tok) pd + el] = z[row of sample b][latent index]; tokens in (t,h,w) raster order, patch
//    vector in (c, dt, dh, dw) order (the first patch_blocks workgroups);
//  - x[b, n_img + j, :] = cond_emb[condition of b, j, :] (the others);
//  - per sample its modulation group and its row in v (workgroup 0).
template <typename T>
__global__ __launch_bounds__(256) void batch_prologue_kernel(SampleMap sm, int b0, int B, int v_rows_mode, int* __restrict__ modmap,
                                                             int* __restrict__ vrows, const float* __restrict__ z, long long D,
                                                             int n_img, int pd, int lt, int lh, int lw, int pt, int ph, int pw,
                                                             int gh, int gw, long long total, int patch_blocks,
                                                             T* __restrict__ out, const float* __restrict__ cond_emb, int L, int Nc,
                                                             int H, long long total4, float* __restrict__ x) {
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < B; i += 256) {
      const int b = b0 + i;
      modmap[i] = sm.group ? sm.group[b] : sm.group0 + sample_cond(sm, b);
      vrows[i] = v_rows_mode == 1 ? sample_row(sm, b) : (v_rows_mode == 2 ? i : b);  // arena row / row of this batch / frontier index
    }
  }
  if ((int)blockIdx.x < patch_blocks) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long long)patch_blocks * 256) {
      const int el = (int)(i % pd);
      const long long bt = i / pd;
      const int tok = (int)(bt % n_img), b = (int)(bt / n_img);
      const int tw = tok % gw, th = (tok / gw) % gh, tt = tok / (gw * gh);
      const int dw = el % pw, dh = (el / pw) % ph, dt = (el / (pw * ph)) % pt, c = el / (pw * ph * pt);
      const long long idx = (((long long)c * lt + tt * pt + dt) * lh + th * ph + dh) * lw + tw * pw + dw;
      out[i] = (T)z[(size_t)sample_row(sm, b0 + b) * D + idx];
    }
  } else {
    const int H4 = H >> 2;
    for (long long i = (long long)(blockIdx.x - patch_blocks) * 256 + threadIdx.x; i < total4;
         i += (long long)(gridDim.x - patch_blocks) * 256) {
      const int h4 = (int)(i % H4);
      const long long bj = i / H4;
      const int j = (int)(bj % Nc), b = (int)(bj / Nc);
      const float4 v = reinterpret_cast<const float4*>(cond_emb)[((size_t)sample_cond(sm, b0 + b) * Nc + j) * H4 + h4];
      reinterpret_cast<float4*>(x)[((size_t)b * L + n_img + j) * H4 + h4] = v;
    }
  }
}

// ------------------------------------------------------- conditioning path
__device__ inline float silu_f(float x) { return x / (1.f + __expf(-x)); }

// pooled[c, :] = mean over the condition tokens of condition c (depends on the prompt only), added in token order.  A
// workgroup takes 64 columns: its four waves fetch POOL_CHUNK tokens at a time, a quarter of them in flight per lane, and one
// wave adds them up from LDS (one lane down all 512 tokens of a column of 3072 by itself: 182 us, so: 8).
constexpr int POOL_CHUNK = 128;
template <typename T>
__device__ inline void pool_columns(const T* __restrict__ cond, int Nc, int cd, float* __restrict__ pooled, int c, int col_block,
                                    float (*tok)[64]) {
  const int col = threadIdx.x & 63, grp = threadIdx.x >> 6, d = col_block * 64 + col;
  const T* p = cond + (size_t)c * Nc * cd + min(d, cd - 1);
  float s = 0.f;
  for (int j0 = 0; j0 < Nc; j0 += POOL_CHUNK) {
    T v[POOL_CHUNK / 4];
#pragma unroll
    for (int k = 0; k < POOL_CHUNK / 4; ++k) v[k] = p[(size_t)min(j0 + 4 * k + grp, Nc - 1) * cd];
#pragma unroll
    for (int k = 0; k < POOL_CHUNK / 4; ++k) tok[4 * k + grp][col] = to_f(v[k]);
    __syncthreads();
    if (grp == 0) {
      const int n = min(POOL_CHUNK, Nc - j0);
#pragma unroll 16
      for (int j = 0; j < n; ++j) s += tok[j][col];
    }
    __syncthreads();
  }
  if (grp == 0 && d < cd) pooled[(size_t)c * cd + d] = s / (float)Nc;
}

template <typename TW>
struct WChunk;  // eight consecutive weights as floats
template <>
struct WChunk<float> {
  static __device__ inline void load(const float* p, float* w) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w; w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
  }
};
template <>
struct WChunk<bf16> {
  static __device__ inline void load(const bf16* p, float* w) {
    typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
    const bf16x8_t v = *reinterpret_cast<const bf16x8_t*>(p);
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = (float)v[e];
  }
};

// One weight row times R <= 8 input rows (row r at row(r)): lanes along k in 8-element chunks (K % 8 == 0, rows 16-byte aligned);
// every lane holds the sums.  (Lane permutations for them instead of the LDS unit: modulation vectors of the tiny network for eight groups 5.2 -> 3.7
// us, second layer 9.7 -> 9.1, small network's call 53.4 -> 52.9.)
template <typename TW, int R, typename ROW>
__device__ inline void skinny_dot(ROW&& row, const TW* __restrict__ wr, int K, int lane, float (&acc)[R]) {
  const float* in[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    acc[r] = 0.f;
    in[r] = row(r);
  }
  for (int k = lane * 8; k < K; k += 512) {
    float w[8];
    WChunk<TW>::load(wr + k, w);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float4 a0 = *reinterpret_cast<const float4*>(in[r] + k);
      const float4 a1 = *reinterpret_cast<const float4*>(in[r] + k + 4);
      const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[r] = fmaf(a[e], w[e], acc[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = lanes_sum<64>(acc[r]);
}

// The conditioning path is three dependent launches, each over groups of R <= 8 rows (modulation groups): the time MLP's first layer
// and, where asked for, the pooled conditions; its second layer with the pooled half of the vector; the modulation vectors.
// (Launches of their own for the pooled mean and its linear layer cost a small network 4 us each, and so did every eight rows.)

// h1[g, n] = silu(sum_k temb(t of group g)[k] W[n, k] + bias[n]), temb = [cos(1000 t f_k), sin(1000 t f_k)],
// f_k = 10000^(-k/128), formed by every workgroup for itself (1 us that runs once, against a launch).  The angle (up to
// 1000 rad) is formed and reduced to [-pi, pi] in fp64, then fp32 sin/cos suffice.  The workgroups behind these pool.
template <typename T, int R>
__global__ __launch_bounds__(256) void cond_first_kernel(GroupTimes gt, int G, const T* __restrict__ W, int N, const float* __restrict__ bias,
                                                         float* __restrict__ h1, int time_blocks, const T* __restrict__ cond, int Nc, int cd,
                                                         int col_blocks, float* __restrict__ pooled) {
  __shared__ __attribute__((aligned(16))) float lds[POOL_CHUNK * 64];
  static_assert(R * 256 <= POOL_CHUNK * 64, "embeddings fit");
  if ((int)blockIdx.x >= time_blocks) {
    const int i = blockIdx.x - time_blocks, c = i / col_blocks;
    pool_columns<T>(cond, Nc, cd, pooled, c, i - c * col_blocks, reinterpret_cast<float(*)[64]>(lds));
    return;
  }
  float(*temb)[256] = reinterpret_cast<float(*)[256]>(lds);
  const int per = (N + 3) / 4, ch = blockIdx.x / per, g0 = ch * R;
  const int k = threadIdx.x & 127;
  const double f = exp(-9.210340371976184 * (double)k / 128.0);  // ln 10000
  for (int r = threadIdx.x >> 7; r < R; r += 2) {
    const int g = min(g0 + r, G - 1);
    const float t = gt.dev ? gt.dev[g] : gt.t[g / gt.n_cond];
    double a = 1000.0 * (double)t * f;
    a -= 6.283185307179586 * rint(a * 0.15915494309189535);
    float sn, cs;
    sincosf((float)a, &sn, &cs);
    temb[r][k] = cs;
    temb[r][128 + k] = sn;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int n = (blockIdx.x - ch * per) * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  float acc[R];
  skinny_dot<T, R>([&](int r) { return &temb[r][0]; }, W + (size_t)n * 256, 256, lane, acc);
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (g0 + r < G) h1[(size_t)(g0 + r) * N + n] = silu_f(acc[r] + bias[n]);
  }
}

// cvec[g, n] = silu((sum_k pooled[condition of g, k] Wp[n, k] + bp[n]) + (sum_k h1[g, k] W[n, k] + bias[n])): the conditioning
// vector of a modulation group.
template <typename TW, int R>
__global__ __launch_bounds__(256) void cond_vector_kernel(const float* __restrict__ h1, const TW* __restrict__ W, const float* __restrict__ bias,
                                                          const float* __restrict__ pooled, const TW* __restrict__ Wp,
                                                          const float* __restrict__ bp, int cd, const int* __restrict__ gcond, int n_cond,
                                                          int G, int N, float* __restrict__ cvec) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6), g0 = blockIdx.y * R;
  if (n >= N) return;
  float acc[R], pool[R];
  skinny_dot<TW, R>([&](int r) { return h1 + (size_t)min(g0 + r, G - 1) * N; }, W + (size_t)n * N, N, lane, acc);
  skinny_dot<TW, R>([&](int r) {
    const int g = min(g0 + r, G - 1);
    return pooled + (size_t)(gcond ? gcond[g] : g % n_cond) * cd;
  }, Wp + (size_t)n * cd, cd, lane, pool);
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (g0 + r < G) cvec[(size_t)(g0 + r) * N + n] = silu_f((pool[r] + bp[n]) + (acc[r] + bias[n]));
  }
}

// out[g, n] = sum_k in[g, k] W[n, k] + bias[n]: a wavefront takes NC columns, and keeps to their weight rows for all groups (the second
// eight find them in cache: 448 000 columns of 3072 for 64 groups stream 2.7 GB once).
// What bounds it: the weights from memory with few groups, the input rows from the compute unit's cache with many.  Four columns a wave keep
// four pieces of the weights in flight instead of one and read the inputs a quarter as often:  444 000 columns of 3072 for two groups
// 736 -> 469 us (5.8 TB/s), 76 000 of 1024 for one 32.9 -> 27.9, for 80 751 -> 462.  Fewer than 64 columns a compute unit stay one to a
// wave: four would leave units idle.
template <typename TW, int R, int NC>
__global__ __launch_bounds__(256) void skinny_gemm_kernel(const float* __restrict__ in, int G, const TW* __restrict__ W, int K, int N,
                                                          const float* __restrict__ bias, float* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int n0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * NC;
  if (n0 >= N) return;
  const TW* wr[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) wr[c] = W + (size_t)min(n0 + c, N - 1) * K;
  for (int g0 = 0; g0 < G; g0 += R) {
    const float* row[R];
    float acc[NC][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      row[r] = in + (size_t)min(g0 + r, G - 1) * K;
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c][r] = 0.f;
    }
    for (int k = lane * 8; k < K; k += 512) {
      float w[NC][8];
#pragma unroll
      for (int c = 0; c < NC; ++c) WChunk<TW>::load(wr[c] + k, w[c]);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float4 a0 = *reinterpret_cast<const float4*>(row[r] + k);
        const float4 a1 = *reinterpret_cast<const float4*>(row[r] + k + 4);
        const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[c][r] = fmaf(a[e], w[c][e], acc[c][r]);
      }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (NC == 1) acc[c][r] = lanes_sum<64>(acc[c][r]);
        else  // (444 000 columns of 3072: 466 us, 494 with lanes_sum; the same bits)
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) acc[c][r] += __shfl_down(acc[c][r], o, 64);
      }
      if (lane == 0 && n0 + c < N) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (g0 + r < G) out[(size_t)(g0 + r) * N + n0 + c] = acc[c][r] + bias[n0 + c];
      }
    }
  }
}

// f(integral_constant R): the rows that a wavefront takes together: all of up to eight, more in equal parts.  (A last part of fewer rows
// costs as much as a whole one: a call of 9 conditions, hidden size 3072, one block, takes 436 us with 8 and 1, 376 with 5 and 4.)
template <typename F>
static void with_rows(int n, F&& f) {
  switch (cdiv(n, cdiv(n, 8))) {
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    default: f(std::integral_constant<int, 8>{}); break;
  }
}

// Per modulation group g: cvec = silu(t_mlp(temb(time of g)) + pool_lin(mean token of its condition)); mods = ada_lin(cvec).
template <typename T>
static br_status conditioning_t(const br_model* m, const FwdBuffers& fb, const T* cond_tokens, int n_cond, const int* gcond,
                                const GroupTimes& gt, int G, hipStream_t st) {
  const int H = m->H;
  auto w = [&](int id) { return (const T*)m->w[id]; };
  auto b = [&](int id) { return (const float*)m->w[id]; };
  with_rows(G, [&](auto Rc) {
    constexpr int R = decltype(Rc)::value;
    const int chunks = cdiv(G, R), time_blocks = chunks * cdiv(H, 4), col_blocks = cdiv(m->cd, 64);
    hipLaunchKernelGGL((cond_first_kernel<T, R>), dim3(time_blocks + (cond_tokens ? n_cond * col_blocks : 0)), dim3(256), 0, st, gt, G,
                       w(BR_W_T1_W), H, b(BR_W_T1_B), fb.h1, time_blocks, cond_tokens, m->Nc, m->cd, col_blocks, fb.pooled);
  });
  BR_LAUNCH_CHECK();
  with_rows(G, [&](auto Rc) {
    constexpr int R = decltype(Rc)::value;
    hipLaunchKernelGGL((cond_vector_kernel<T, R>), dim3(cdiv(H, 4), cdiv(G, R)), dim3(256), 0, st, fb.h1, w(BR_W_T2_W), b(BR_W_T2_B),
                       fb.pooled, w(BR_W_POOL_W), b(BR_W_POOL_B), m->cd, gcond, gt.n_cond, G, H, fb.cvec);
  });
  BR_LAUNCH_CHECK();
  // the modulation vectors of all blocks: a GEMV that streams the [A, H] weights
  ProfScope ps(st, PROF_ADALN, (double)m->A * H * sizeof(T));
  with_rows(G, [&](auto Rc) {
    constexpr int R = decltype(Rc)::value;
    if (m->A >= 64 * device_cu_count())
      hipLaunchKernelGGL((skinny_gemm_kernel<T, R, 4>), dim3(cdiv(m->A, 16)), dim3(256), 0, st, fb.cvec, G, w(BR_W_ADA_W), H, m->A, b(BR_W_ADA_B),
                         fb.mods);
    else
      hipLaunchKernelGGL((skinny_gemm_kernel<T, R, 1>), dim3(cdiv(m->A, 4)), dim3(256), 0, st, fb.cvec, G, w(BR_W_ADA_W), H, m->A, b(BR_W_ADA_B),
                         fb.mods);
  });
  BR_LAUNCH_CHECK();
  return BR_OK;
}

br_status conditioning(const br_model* m, const FwdBuffers& fb, const void* cond_tokens, int n_cond, const int* gcond,
                       const GroupTimes& gt, int G, hipStream_t st) {
  return m->cfg.dtype == BR_BF16 ? conditioning_t<bf16>(m, fb, (const bf16*)cond_tokens, n_cond, gcond, gt, G, st)
                                 : conditioning_t<float>(m, fb, (const float*)cond_tokens, n_cond, gcond, gt, G, st);
}

// ------------------------------------------------------- LayerNorm-modulate
// out[r, :] = LN(x[src(r), :]) (1 + scale) + shift; one wavefront per row, the row held in
// registers (VPL float4 per lane; VPL = 0: any H, the row is re-read from cache instead).
// r = b * rows_per_sample + tok, src = b * L_in + tok; LN without affine, eps 1e-6.
//
// What bounds it: a small launch, the chain of one row (row, group of its sample, modulation vectors, two sums of 64 lanes), a large one the
// memory.  The row's number is scalar, so the group comes by a scalar load beside the row's own; up to VPL = 4 the modulation vectors are
// under way with the row too (beyond, the compiler decides); the sums are exchanged without the LDS unit.  fp32 rows of more than 1024
// columns, and of large launches, fetch the vectors last (LATE): they lose by more registers or more loads in front of the row.  STREAM: rows that the caches cannot
// hold until the next launch reads them are stored past them.  Long rows of such launches keep the sums in the LDS unit (bf16 from 1536 columns: 22 020 x 2048
// 49.9 us without it, 49.1 with, 147 456 x 3072 462, 458), in fp32 from 1024 also the row number in a vector register and the vectors
// behind the sums (LONG: 9216 x 3072 45.0 us in the other form, 42.4; 147 456 x 3072 662, 647; 70 464 x 1024 96.8, 95.7; but 33 272 x 1536 71.2, 71.8).
// us before -> now (a graph over buffers in turn), bf16:  8808 x 1024 12.3 -> 11.1, 17 616 x 1024 21.2 -> 19.4, 26 424 x 1024 29.9 -> 27.5, 70 464 x 1024
// 74.1 -> 74.4, 38 336 x 512 22.9 -> 19.9, 36 864 x 3072 123.6 -> 117.0, 33 272 x 1536 53.8 -> 53.6; fp32: 8808 x 1024 15.2 -> 14.4, 17 616 x 1024
// 27.2 -> 24.8, 76 800 x 256 31.3 -> 28.1.  Plain stores below the line cost an isolated launch that writes the same rows again up to a
// tenth (4000 x 1536 7.8 -> 8.8), in a network they are worth 0 to 2 % of the call.
constexpr double LN_STREAM_FROM = 192e6;  // bytes of rows read and written
template <bool STREAM, typename T>
__device__ __forceinline__ void store4_row(T* p, float a, float b, float c, float d) {
  typedef T t4 __attribute__((ext_vector_type(4)));
  const t4 v = {(T)a, (T)b, (T)c, (T)d};
  if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<t4*>(p));
  else *reinterpret_cast<t4*>(p) = v;
}
template <typename T, int VPL, bool STREAM>
__global__ __launch_bounds__(256) void ln_modulate_kernel(const float* __restrict__ x, T* __restrict__ out, int n_rows,
                                                          int rows_per_sample, int L_in, int H,
                                                          const float* __restrict__ mods, int A, int shift_off,
                                                          int scale_off, const int* __restrict__ condmap) {
  constexpr int NV = VPL > 0 ? VPL : 1;
  constexpr bool F32 = std::is_same<T, float>::value, LONG = F32 && STREAM && VPL >= 4 && VPL != 6;
  constexpr bool LATE = F32 && !LONG && (STREAM || VPL > 4), EARLY = !LATE && !LONG && VPL > 0 && VPL <= 4;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6, r = blockIdx.x * 4 + (LONG ? wave : __builtin_amdgcn_readfirstlane(wave));
  if (r >= n_rows) return;
  const int b = r / rows_per_sample, tok = r - b * rows_per_sample;
  const float4* xr = reinterpret_cast<const float4*>(x + ((size_t)b * L_in + tok) * H);
  const int H4 = H >> 2;
  float4 v[NV], a[NV], g[NV];
  if (VPL > 0) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) v[i] = xr[lane + 64 * i];
  }
  const float4 *sh, *sc;
  auto vectors = [&] {
    const float* mrow = mods + (size_t)condmap[b] * A;
    sh = reinterpret_cast<const float4*>(mrow + shift_off);
    sc = reinterpret_cast<const float4*>(mrow + scale_off);
  };
  if (!LONG) vectors();
  if (EARLY) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      a[i] = sh[lane + 64 * i];
      g[i] = sc[lane + 64 * i];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  auto sum = [](float u) {
    if (!STREAM || !(F32 ? LONG : VPL >= 6)) return lanes_sum<64>(u);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) u += __shfl_xor(u, o, 64);
    return u;
  };
  float s = 0.f;
  if (VPL > 0) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  } else {
    for (int i = lane; i < H4; i += 64) {
      const float4 u = xr[i];
      s += (u.x + u.y) + (u.z + u.w);
    }
  }
  const float mean = sum(s) / (float)H;
  float q = 0.f;
  if (VPL > 0) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) q += sum_sq4(v[i], mean);
  } else {
    for (int i = lane; i < H4; i += 64) q += sum_sq4(xr[i], mean);
  }
  const float rstd = 1.0f / __builtin_sqrtf(sum(q) / (float)H + 1e-6f);
  if (LONG) vectors();
  T* orow = out + (size_t)r * H;
  if (LATE) asm volatile("" ::: "memory");
  if (VPL > 0) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
      const int c4 = lane + 64 * i;
      if (!EARLY) {
        a[i] = sh[c4];
        g[i] = sc[c4];
      }
      store4_row<STREAM, T>(orow + 4 * c4, fmaf((v[i].x - mean) * rstd, 1.f + g[i].x, a[i].x), fmaf((v[i].y - mean) * rstd, 1.f + g[i].y, a[i].y),
                fmaf((v[i].z - mean) * rstd, 1.f + g[i].z, a[i].z), fmaf((v[i].w - mean) * rstd, 1.f + g[i].w, a[i].w));
    }
  } else {
    for (int i = lane; i < H4; i += 64) {
      const float4 u = xr[i], m = sh[i], k = sc[i];
      store4_row<STREAM, T>(orow + 4 * i, fmaf((u.x - mean) * rstd, 1.f + k.x, m.x), fmaf((u.y - mean) * rstd, 1.f + k.y, m.y),
                fmaf((u.z - mean) * rstd, 1.f + k.z, m.z), fmaf((u.w - mean) * rstd, 1.f + k.w, m.w));
    }
  }
}

template <typename T, bool STREAM>
static void ln_launch(dim3 g, dim3 b, hipStream_t st, const float* x, T* out, int n_rows, int rows_per_sample, int L_in,
                      int H, const float* mods, int A, int shift_off, int scale_off, const int* condmap) {
#define BR_LN(V) hipLaunchKernelGGL((ln_modulate_kernel<T, V, STREAM>), g, b, 0, st, x, out, n_rows, rows_per_sample, L_in, H, \
                                    mods, A, shift_off, scale_off, condmap)
  switch (H % 256 == 0 ? H / 256 : 0) {
    case 1: BR_LN(1); break;
    case 2: BR_LN(2); break;
    case 3: BR_LN(3); break;
    case 4: BR_LN(4); break;
    case 6: BR_LN(6); break;
    case 8: BR_LN(8); break;
    case 12: BR_LN(12); break;
    default: BR_LN(0); break;
  }
#undef BR_LN
}

br_status launch_ln_modulate(int dtype, const float* x, void* out, int n_rows, int rows_per_sample, int L_in, int H,
                             const float* mods, int A, int shift_off, int scale_off, const int* condmap,
                             hipStream_t st) {
  if (n_rows == 0) return BR_OK;
  dim3 g(cdiv(n_rows, 4)), b(256);
  ProfScope ps(st, PROF_LN_MOD, (double)n_rows * H * (4.0 + (dtype == BR_BF16 ? 2.0 : 4.0)));
  auto go = [&](auto Tc, auto Sc) {
    using T = decltype(Tc);
    ln_launch<T, decltype(Sc)::value>(g, b, st, x, (T*)out, n_rows, rows_per_sample, L_in, H, mods, A, shift_off, scale_off, condmap);
  };
  const bool stream = (double)n_rows * H * (dtype == BR_BF16 ? 6.0 : 8.0) > LN_STREAM_FROM;
  auto type = [&](auto Tc) { stream ? go(Tc, std::true_type{}) : go(Tc, std::false_type{}); };
  if (dtype == BR_BF16) type(bf16{});
  else type(float{});
  BR_LAUNCH_CHECK();
  return BR_OK;
}

br_status launch_gemm(int dtype, int mode, const void* A, int lda, const void* W, int ldw, int M, int N, int K,
                      const EpiArgs& ea, hipStream_t st) {
  if (M == 0) return BR_OK;
  BR_REQUIRE(N % 4 == 0, BR_ESHAPE, "gemm: N must be a multiple of 4");
  if (dtype == BR_BF16)
    return launch_gemm_bf16(mode, (const bf16*)A, lda, (const bf16*)W, ldw, M, N, K, ea, -1, st);
  return launch_gemm_f32(mode, (const float*)A, lda, (const float*)W, ldw, M, N, K, ea, -1, st);
}

br_status launch_attention(int dtype, const void* qkv, void* out, int B, int L, int NH, int DH, int q_prescaled, const WarmRows& next,
                           hipStream_t st) {
  if (B == 0) return BR_OK;
  if (dtype == BR_BF16) return launch_attention_bf16((const bf16*)qkv, (bf16*)out, B, L, NH, DH, q_prescaled, next, st);
  BR_REQUIRE(!q_prescaled, BR_EINVAL, "attention: prescaled queries are a bf16 layout");
  return launch_attention_f32((const float*)qkv, (float*)out, B, L, NH, DH, st);
}

br_status launch_batch_prologue(const br_model* m, const FwdBuffers& fb, const SampleMap& sm, int b0, int B, int v_rows_mode,
                                const float* z, hipStream_t st) {
  const br_model_cfg& c = m->cfg;
  const long long total = (long long)B * m->n_img * m->pd, total4 = (long long)B * m->Nc * (m->H / 4);
  const int np = (int)std::min<long long>((total + 255) / 256, 65535 * 16), nc = (int)std::min<long long>((total4 + 255) / 256, 65535 * 16);
  auto go = [&](auto* patches) {
    using T = std::remove_pointer_t<decltype(patches)>;
    hipLaunchKernelGGL((batch_prologue_kernel<T>), dim3(np + nc), dim3(256), 0, st, sm, b0, B, v_rows_mode, fb.modmap, fb.vrows, z, m->D,
                       m->n_img, m->pd, c.latent_t, c.latent_h, c.latent_w, c.patch_t, c.patch_h, c.patch_w, m->gh, m->gw, total, np,
                       patches, fb.cond_emb, m->L, m->Nc, m->H, total4, fb.x);
  };
  if (c.dtype == BR_BF16) go((bf16*)fb.patches);
  else go((float*)fb.patches);
  BR_LAUNCH_CHECK();
  return BR_OK;
}

}  // namespace br
