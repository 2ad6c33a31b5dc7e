// Epilogue of the persistent bf16 GEMM, whose waves own 16 RB x 128 outputs in the accumulators of 16x16 matrix
// instructions: block (i, j) of acc gives lane l the columns 16 i + 4 (l >> 4) .. + 3 of row 16 j + (l & 15).
// Each wave passes its blocks through a private 8 KB LDS buffer and stores whole 512-byte (fp32) or 256-byte
// (bf16) row segments.  The rules for loads and stores are those of gemm_epilogue.h: what a row needs from memory
// is fetched before the stores that would otherwise have to be acknowledged first.
#pragma once
#include "gemm_epilogue.h"

namespace br {

constexpr int WIDE_EPI_BYTES = 8192;  // LDS of a wave

// Four accumulators, read from the accumulation registers where they are used: as ordinary values the compiler
// copies all of a tile's to vector registers at once, and spills.
__device__ __forceinline__ f32x4_e acc_read(const f32x4_e& a) {
  f32x4_e v;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x = a[e], y;
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(y) : "a"(x));
    v[e] = y;
  }
  return v;
}

// 16 rows (block row j) of the wave's outputs into its buffer: row r is 512 bytes, 16-byte chunk c in slot c ^ r.
template <int RB>
__device__ __forceinline__ void wide_stage_rows(const f32x4_e (&acc)[8][RB], char* ebuf, int j, int lane) {
  const int r = lane & 15, c = lane >> 4;
  epilogue_wave_fence();
#pragma unroll
  for (int i = 0; i < 8; ++i) *reinterpret_cast<f32x4_e*>(ebuf + r * 512 + (((i * 4 + c) ^ r) << 4)) = acc_read(acc[i][j]);
  epilogue_wave_fence();
}

// Rows of a wave tile that spans more than two samples: every row looks its sample up by itself.
template <int RB, int MODE, typename TOUT>
__device__ __forceinline__ void wide_epilogue_rows(const f32x4_e (&acc)[8][RB], char* ebuf, int m_base, int n_base, int M, int N,
                                                   const Epilogue<MODE, TOUT>& epi, int lane) {
  const int c = lane & 31, rq = lane >> 5, n = n_base + c * 4;
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    wide_stage_rows(acc, ebuf, j, lane);
    for (int q = 0; q < 8; ++q) {
      const int r = rq + 2 * q, m = m_base + j * 16 + r;
      const f32x4_e v = *reinterpret_cast<const f32x4_e*>(ebuf + r * 512 + ((c ^ r) << 4));
      if (m < M && n < N) epi.store(epi.row(m), n, v[0], v[1], v[2], v[3]);
    }
  }
}

// FULL: every row and column of the wave tile lies inside the matrix (no branches: the compiler then counts the
// outstanding memory operations exactly).  The residual rows are fetched AHEAD passes of 16 rows before their use:
// a compute unit has one wave per SIMD here, so what is in flight has to come from each of them.
template <bool FULL, int RB, int MODE, typename TOUT>
__device__ __forceinline__ void wide_epilogue_pair(const f32x4_e (&acc)[8][RB], char* ebuf, int m_base, int n_base, int M, int N,
                                                   const Epilogue<MODE, TOUT>& epi, int lane) {
  using Epi = Epilogue<MODE, TOUT>;
  constexpr int AHEAD = Epi::kHasAddend ? 3 : 0, NBUF = AHEAD + 1;
  const int rps = epi.rows_per_sample();
  const int c = lane & 31, rq = lane >> 5, n = n_base + c * 4;
  const bool n_ok = FULL || n < N;
  // the wave's rows lie in sample b0 (first row lo0) and, from row lo1 on, in sample b0 + 1
  int lo0 = 0, lo1 = 0x7fffffff;
  typename Epi::SampleC s0 = {}, s1 = {};
  float4 bb = make_float4(0.f, 0.f, 0.f, 0.f);
  if (n_ok) {
    bb = epi.bias4(n);
    if (rps > 0 && (FULL || m_base < M)) {
      const int b0 = m_base / rps;
      lo0 = b0 * rps;
      lo1 = lo0 + rps;
      s0 = epi.sample_consts(b0, n);
      s1 = epi.sample_consts(lo1 < M ? b0 + 1 : b0, n);
    }
  }
  float4 add[NBUF][8];
  auto fetch_addend = [&](int pass, float4* dst) {
    if (!Epi::kHasAddend) return;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int m = m_base + pass * 16 + rq + 2 * q;
      const int tok = m - (m >= lo1 ? lo1 : lo0);
      if (FULL)
        dst[q] = epi.addend(m, tok, n);
      else
        dst[q] = (m < M && n_ok) ? epi.addend(m, tok, n) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
#pragma unroll
  for (int pass = 0; pass < AHEAD; ++pass) fetch_addend(pass, add[pass % NBUF]);
#pragma unroll
  for (int pass = 0; pass < RB; ++pass) {
    if (pass + AHEAD < RB) fetch_addend(pass + AHEAD, add[(pass + AHEAD) % NBUF]);
    wide_stage_rows(acc, ebuf, pass, lane);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = rq + 2 * q, m = m_base + pass * 16 + r;
      const f32x4_e v = *reinterpret_cast<const f32x4_e*>(ebuf + r * 512 + ((c ^ r) << 4));
      if (FULL || (m < M && n_ok)) {
        const bool second = m >= lo1;
        epi.finish(m, m - (second ? lo1 : lo0), n, v[0], v[1], v[2], v[3], bb, second ? s1 : s0, add[pass % NBUF][q]);
      }
    }
  }
}

// bf16 outputs of a wave tile wholly inside the matrix: bias and activation in the accumulator layout, rounded before
// the trip through LDS, 32 rows of 256 bytes per pass (16-byte chunk c of row r in slot c ^ (r & 15)).
// KEEP: plain stores, which leave the rows in the caches for the launch that reads them; else past the caches (persistent_output_stays).
template <int RB, int MODE, bool KEEP>
__device__ __forceinline__ void wide_epilogue_bf16(const f32x4_e (&acc)[8][RB], char* ebuf, int m_base, int n_base,
                                                   const Epilogue<MODE, bf16>& epi, int lane) {
  typedef __bf16 bf16x4_e __attribute__((ext_vector_type(4)));
  typedef unsigned int u32x4_e __attribute__((ext_vector_type(4)));
  const int l16 = lane & 15, lq = lane >> 4;
  float4 bias[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) bias[i] = epi.bias4(n_base + i * 16 + lq * 4);
  bf16* const obase = reinterpret_cast<bf16*>(epi.a.out) + (long long)(m_base + lq) * epi.a.ldo + n_base + l16 * 8;
#pragma unroll
  for (int p = 0; p < (RB + 1) / 2; ++p) {
    epilogue_wave_fence();
#pragma unroll
    for (int h = 0; h < 2 && 2 * p + h < RB; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const f32x4_e a = acc_read(acc[i][2 * p + h]);
        float v0 = a[0] + bias[i].x, v1 = a[1] + bias[i].y, v2 = a[2] + bias[i].z, v3 = a[3] + bias[i].w;
        if (MODE == EPI_BIAS_GELU) {
          v0 = gelu_tanh_f(v0);
          v1 = gelu_tanh_f(v1);
          v2 = gelu_tanh_f(v2);
          v3 = gelu_tanh_f(v3);
        } else {
          const float cs = epi.colscale(n_base + i * 16 + lq * 4);
          v0 *= cs;
          v1 *= cs;
          v2 *= cs;
          v3 *= cs;
        }
        const bf16x4_e pk = {(bf16)v0, (bf16)v1, (bf16)v2, (bf16)v3};
        *reinterpret_cast<bf16x4_e*>(ebuf + (h * 16 + l16) * 256 + (((i * 2 + (lq >> 1)) ^ l16) << 4) + (lq & 1) * 8) = pk;
      }
    epilogue_wave_fence();
#pragma unroll
    for (int q = 0; q < (2 * p + 1 < RB ? 8 : 4); ++q) {
      const int r = lq + 4 * q;
      const u32x4_e v = *reinterpret_cast<const u32x4_e*>(ebuf + r * 256 + ((l16 ^ (r & 15)) << 4));
      u32x4_e* const dst = reinterpret_cast<u32x4_e*>(obase + (long long)(p * 32 + 4 * q) * epi.a.ldo);
      if constexpr (KEEP) *dst = v;
      else __builtin_nontemporal_store(v, dst);
    }
  }
}

// Returns a lower bound on the number of store instructions the wave has issued (0 on the guarded paths).
template <int RB, int MODE, typename TOUT, bool KEEP>
__device__ __forceinline__ int wide_epilogue(const f32x4_e (&acc)[8][RB], char* ebuf, int m_base, int n_base, int M, int N,
                                             const Epilogue<MODE, TOUT>& epi, int lane) {
  const int rps = epi.rows_per_sample();
  if (rps > 0 && rps < 16 * RB) {
    wide_epilogue_rows<RB, MODE, TOUT>(acc, ebuf, m_base, n_base, M, N, epi, lane);
  } else if (m_base + 16 * RB <= M && n_base + 128 <= N) {
    if constexpr (std::is_same<TOUT, bf16>::value) {
      wide_epilogue_bf16<RB, MODE, KEEP>(acc, ebuf, m_base, n_base, epi, lane);
      return 4 * RB;
    } else {
      wide_epilogue_pair<true, RB, MODE, TOUT>(acc, ebuf, m_base, n_base, M, N, epi, lane);
      return 8 * RB;
    }
  } else {
    wide_epilogue_pair<false, RB, MODE, TOUT>(acc, ebuf, m_base, n_base, M, N, epi, lane);
  }
  return 0;
}

}  // namespace br
