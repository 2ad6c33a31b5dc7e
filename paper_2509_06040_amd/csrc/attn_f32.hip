// fp32 attention on the matrix cores (v_mfma_f32_32x32x2_f32: full fp32): softmax(Q K^T / sqrt(d)) V over
// all L tokens of a sample, one workgroup per (32 queries, head, sample), whose four waves take every
// fourth tile of 32 keys each and merge their partial results at the end.
//
// The matrix pipe is the bound: one key tile of a wave is DH products of 64 cycles, against 0.25 KB of
// K and V per head channel, so sharing tiles between waves would save nothing that is short, and a wave that
// fetches its own tiles (global -> LDS directly) needs no barrier in the loop.  Splitting the keys instead
// of the queries keeps four waves busy at any sequence length above 96.  At L = 1101, 4 samples of 16
// heads of 64 channels: 222 us (90 TFLOP/s; one query per lane with vector arithmetic took 880 us).
//
// Scores are computed transposed, S^T = K Q^T: register r of a lane then holds key
// 8 (r / 4) + 4 (lane / 32) + r % 4 of query lane % 32, the reference / sum / rescale of the online
// softmax are per-lane scalars, and step r of O^T = V^T P^T contracts over exactly the two keys that
// register r holds in the two halves of the wave: P needs no exchange between lanes.
#include "common.h"
#include "dit.h"

namespace br {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

#define BR_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

namespace {
constexpr int NW = 4;        // waves per workgroup
constexpr int KT = 32;       // keys of a tile
}  // namespace

// 16-byte chunk c of row r of a K tile (and of the merged output rows) sits in slot c ^ swz(r), which spreads
// 16 consecutive rows at one chunk index over all LDS banks; CH = chunks of a row.
template <int CH>
__device__ inline int row_swz(int r) { return CH >= 16 ? (r & 15) : CH == 8 ? ((r >> 1) & 7) : ((r >> 2) & 3); }

template <int DH>
__global__ __launch_bounds__(NW * 64, DH == 128 ? 1 : 2) void attn_f32_kernel(const float* __restrict__ qkv, float* __restrict__ out,
                                                                              int L, int H, int NH, int n_pairs, int grouped,
                                                                              float scale_log2) {
  constexpr int CH = DH / 4, RB = DH * 4;   // chunks and bytes of a row
  constexpr int RPI = 1024 / RB;            // rows covered by one 1 KB load
  constexpr int NI = KT / RPI;              // loads per operand and tile
  constexpr int KP = DH / 8;                // chunk pairs of the score product
  constexpr int DB = (DH + 31) / 32;        // 32-row blocks of O^T (rows past DH repeat and are dropped)
  constexpr int TILE_B = KT * RB;
  __shared__ __attribute__((aligned(1024))) char slots[NW][2 * TILE_B];
  __shared__ float part_m[NW][32], part_l[NW][32];

  // query tiles of one (sample, head) share that head's keys and values: they run on one compute die when
  // there are enough pairs to occupy all eight
  const int nq = (L + 31) / 32;
  int pair, qt;
  if (grouped) {
    const int x = blockIdx.x & 7, slot = blockIdx.x >> 3;
    pair = (slot / nq) * 8 + x;
    qt = slot - (slot / nq) * nq;
  } else {
    pair = blockIdx.x / nq;
    qt = blockIdx.x - pair * nq;
  }
  if (pair >= n_pairs) return;
  const int b = pair / NH, h = pair - b * NH;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t ld = (size_t)3 * H;
  const float* base = qkv + (size_t)b * L * ld + (size_t)h * DH;
  const int nkt = (L + KT - 1) / KT;

  // queries, in units of log2 e / sqrt(d): the exponent is then a power of two
  f32x4 q[KP];
  {
    const float* qr = base + (size_t)min(qt * 32 + l32, L - 1) * ld;
#pragma unroll
    for (int p = 0; p < KP; ++p) q[p] = *reinterpret_cast<const f32x4*>(qr + (2 * p + lh) * 4) * scale_log2;
  }
  f32x16 o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  const unsigned ldb = (unsigned)(ld * 4);
  const int lrow = lane / CH, slot = lane % CH;
  char* mine = slots[wv];
  auto issue = [&](int kt) {
    const char* kp = reinterpret_cast<const char*>(base + (size_t)kt * KT * ld + H);
    const char* vp = kp + (size_t)H * 4;
    const unsigned dst = (unsigned)(uintptr_t)BR_LPTR(mine);
    const int last = L - 1 - kt * KT;  // rows past the end read the last key (their scores and values are masked)
#pragma unroll
    for (int t = 0; t < NI; ++t) {
      const int row = t * RPI + lrow;
      const unsigned off = (unsigned)min(row, last) * ldb + ((slot ^ row_swz<CH>(row)) << 4);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst + t * 1024), "v"(off), "s"(kp) : "memory", "m0");
    }
#pragma unroll
    for (int t = 0; t < NI; ++t) {
      const unsigned off = (unsigned)min(t * RPI + lrow, last) * ldb + (slot << 4);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst + TILE_B + t * 1024), "v"(off), "s"(vp) : "memory", "m0");
    }
  };

  if (wv < nkt) issue(wv);
  for (int kt = wv; kt < nkt; kt += NW) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    f32x4 kf[KP];
    float vf[DB][16];
#pragma unroll
    for (int p = 0; p < KP; ++p)
      kf[p] = *reinterpret_cast<const f32x4*>(mine + l32 * RB + (((2 * p + lh) ^ row_swz<CH>(l32)) << 4));
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        vf[d][r] = *reinterpret_cast<const float*>(mine + TILE_B + (8 * (r >> 2) + 4 * lh + (r & 3)) * RB + ((d * 32 + l32) % DH) * 4);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (kt + NW < nkt) issue(kt + NW);  // the tile is in registers: its slot is free
    __builtin_amdgcn_sched_barrier(0);

    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int p = 0; p < KP; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[p][e], q[p][e], s, 0, 0, 0);
    if (kt == nkt - 1) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (kt * KT + 8 * (r >> 2) + 4 * lh + (r & 3) >= L) {
          s[r] = -INFINITY;
#pragma unroll
          for (int d = 0; d < DB; ++d) vf[d][r] = 0.f;  // (0 times an infinite value would be a NaN)
        }
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // the reference: the largest score so far, 0 while all of them are -inf (the wave holds only a part of the keys)
    const float m_new = fmaxf(m_run, mx), m_ref = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_ref);
    m_run = m_new;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = __builtin_amdgcn_exp2f(s[r] - m_ref);
      sum += s[r];
    }
    l_run = l_run * alpha + sum;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int d = 0; d < DB; ++d) o[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[d][r], s[r], o[d], 0, 0, 0);
  }

  // merge of the four partial results: bring them to the common reference, add them up in wave order
  l_run += __shfl_xor(l_run, 32, 64);
  if (lh == 0) part_m[wv][l32] = m_run;
  __syncthreads();  // (every wave is done with its slots too)
  float m_all = part_m[0][l32];
#pragma unroll
  for (int w = 1; w < NW; ++w) m_all = fmaxf(m_all, part_m[w][l32]);
  const float f = __builtin_amdgcn_exp2f(m_run - m_all);  // 0 for a wave without keys; (NaN if every score is -inf)
  if (lh == 0) part_l[wv][l32] = l_run * f;
  static_assert(32 * RB <= 2 * TILE_B, "a partial output reuses the wave's slot");
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int c = d * 8 + 2 * g + lh;
      if (c < CH) {
        const f32x4 v = {o[d][4 * g] * f, o[d][4 * g + 1] * f, o[d][4 * g + 2] * f, o[d][4 * g + 3] * f};
        *reinterpret_cast<f32x4*>(mine + l32 * RB + ((c ^ row_swz<CH>(l32)) << 4)) = v;
      }
    }
  __syncthreads();
  for (int e = tid; e < 32 * CH; e += NW * 64) {
    const int row = e / CH, c = e % CH, qi = qt * 32 + row;
    if (qi >= L) break;
    const int at = row * RB + ((c ^ row_swz<CH>(row)) << 4);
    f32x4 v = *reinterpret_cast<const f32x4*>(slots[0] + at);
    float l = part_l[0][row];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      v += *reinterpret_cast<const f32x4*>(slots[w] + at);
      l += part_l[w][row];
    }
    const float inv = 1.f / l;
    *reinterpret_cast<f32x4*>(out + ((size_t)b * L + qi) * H + h * DH + c * 4) = v * inv;
  }
}

// Any alignment of the buffers (the kernel above fetches 16 bytes at a time): one thread per query, streaming over all keys with an online softmax.
template <int DH>
__global__ __launch_bounds__(64) void attn_f32_any_kernel(const float* __restrict__ qkv, float* __restrict__ out, int L,
                                                      int H, float scale) {
  const int b = blockIdx.z, h = blockIdx.y, qi = blockIdx.x * 64 + threadIdx.x;
  const float* base = qkv + (size_t)b * L * 3 * H + h * DH;
  const bool live = qi < L;
  float q[DH], o[DH];
#pragma unroll
  for (int d = 0; d < DH; ++d) {
    q[d] = live ? base[(size_t)qi * 3 * H + d] * scale : 0.f;
    o[d] = 0.f;
  }
  float mx = -INFINITY, den = 0.f;
  for (int j = 0; j < L; ++j) {
    const float* kr = base + (size_t)j * 3 * H + H;
    const float* vr = kr + H;
    float s = 0.f;
#pragma unroll
    for (int d = 0; d < DH; ++d) s = fmaf(q[d], kr[d], s);
    const float mn = fmaxf(mx, s);
    const float alpha = __expf(mx - mn), p = __expf(s - mn);
    den = den * alpha + p;
#pragma unroll
    for (int d = 0; d < DH; ++d) o[d] = fmaf(p, vr[d], o[d] * alpha);
    mx = mn;
  }
  if (live) {
    float* orow = out + ((size_t)b * L + qi) * H + h * DH;
    const float inv = 1.f / den;
#pragma unroll
    for (int d = 0; d < DH; ++d) orow[d] = o[d] * inv;
  }
}

#define BR_AT_SWITCH                                                                      \
  switch (DH) {                                                                           \
    case 16: BR_AT(16); break;                                                            \
    case 32: BR_AT(32); break;                                                            \
    case 64: BR_AT(64); break;                                                            \
    case 128: BR_AT(128); break;                                                          \
    default: return fail(BR_ESHAPE, "attention: head dim must be 16, 32, 64 or 128");     \
  }

br_status launch_attention_f32(const float* qkv, float* out, int B, int L, int NH, int DH, hipStream_t st) {
  const int H = NH * DH;
  if ((((uintptr_t)qkv | (uintptr_t)out) & 15) != 0) {
    BR_REQUIRE(NH <= 65535 && B <= 65535, BR_ESHAPE, "attention: too many heads or samples for one launch");
    const float scale = 1.0f / sqrtf((float)DH);
#define BR_AT(D_) hipLaunchKernelGGL((attn_f32_any_kernel<D_>), dim3(cdiv(L, 64), NH, B), dim3(64), 0, st, qkv, out, L, H, scale)
    BR_AT_SWITCH
#undef BR_AT
    BR_LAUNCH_CHECK();
    return BR_OK;
  }
  const long long n_pairs = (long long)B * NH;
  BR_REQUIRE(n_pairs <= 0x7FFFFFFFLL, BR_ESHAPE, "attention: too many heads and samples for one launch");
  const int grouped = n_pairs >= 32 ? 1 : 0;
  const long long n_blocks = (grouped ? (n_pairs + 7) / 8 * 8 : n_pairs) * cdiv(L, 32);
  BR_REQUIRE(n_blocks <= 0x7FFFFFFFLL, BR_ESHAPE, "attention: too many workgroups for one launch");
  const float scale_log2 = (float)(1.4426950408889634 / sqrt((double)DH));
#define BR_AT(D_) \
  hipLaunchKernelGGL((attn_f32_kernel<D_>), dim3((unsigned)n_blocks), dim3(NW * 64), 0, st, qkv, out, L, H, NH, (int)n_pairs, grouped, scale_log2)
  BR_AT_SWITCH
#undef BR_AT
  BR_LAUNCH_CHECK();
  return BR_OK;
}

}  // namespace br
