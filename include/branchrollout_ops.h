/*
 * libbranchrollout -- op-level entry points of the velocity network, for checking
 * single kernels against a reference and for timing them in isolation.  They are
 * not part of the rollout API; conventions as in branchrollout.h.
 */
#ifndef BRANCHROLLOUT_OPS_H
#define BRANCHROLLOUT_OPS_H

#include "branchrollout.h"

#ifdef __cplusplus
extern "C" {
#endif

/* C[m, n] = epilogue(sum_k A[m, k] W[n, k] + bias[n]); A dev [M, lda], W dev [N, ldw]
 * in `dtype` (BR_F32 / BR_BF16), bias dev [N] fp32.
 *   epilogue 0: out[m, n] = acc                  out in `dtype`  [M, ldo]
 *            1: out[m, n] = gelu_tanh(acc)       out in `dtype`
 *            2: out[m, n] += gate[cond[m / L]][n] * acc    out fp32 in place;
 *               gate row r at mods + r*mods_stride + gate_off, cond dev [M / L]
 *            4: out[m, n] = acc                  out fp32
 * BR_BF16 needs K % 64 == 0, lda % 8 == 0, ldw % 8 == 0; N % 4 == 0 always.
 * variant: bits 0..3 = kernel (-1 = automatic; 0 = 32x32 tiles; 1 / 2 / 3 / 4 / 5 = 128x128 in eight waves /
 * 64x64 / 64x128 / 256x256 / 128x128 tile per workgroup; 6 = one 16h x 128 tile per workgroup with a deep ring, h in bits
 * 24..30: 2, 4, 6, 8, 10 or 12, otherwise (or where 16h rows of A or 128 of W span 4 GiB) as 5; 7 = persistent streaming
 * kernel with tiles of 256 rows x 256 columns, 8 / 9 / 10 / 11 = the same with 128 / 160 / 192 / 224 rows, need
 * K % 128 == 0.  BR_F32 has 0 and, where K % 32 == 0, 6 with h from 2 to 12 and 64 columns, 128 with bit 4, and takes its own
 * choice where another is asked for or does not apply.  bf16 only:
 * bits 4..11 = column-group width of the tile walk, 0 = the kernel's own choice; for the persistent kernel bits 24..30 =
 * rows of a row block of the tile walk in units of 8 tile rows, 0 = the kernel's own choice; bits 12..23, start delays
 * of workgroups in earlier versions, are accepted and have no effect.  All of them give the same
 * results, bit for bit: every output is the sum over k in ascending order. */
br_status br_op_gemm(int32_t dtype, int32_t epilogue, const void* A, int32_t lda, const void* W,
                     int32_t ldw, int32_t M, int32_t N, int32_t K, const float* bias, void* out,
                     int32_t ldo, const float* mods, int32_t mods_stride, int32_t gate_off,
                     const int32_t* cond, int32_t L, int32_t variant, void* stream);

/* out[b, l, h*DH + d] = softmax_j(q_l . k_j / sqrt(DH)) v_j for every sample b and
 * head h; qkv dev [B, L, 3*NH*DH] (q | k | v), out dev [B, L, NH*DH], both `dtype`.
 * BR_BF16: DH 64 or 128, qkv 16-byte aligned, L*3*NH*DH*2 below 4 GiB (BR_ESHAPE otherwise).
 * BR_BF16: a query that is not finite, or that scores +inf with a key or -inf with all, has NaN in its own row of that head; others keep theirs.
 * q_prescaled = 1 (BR_BF16 only, BR_EINVAL otherwise): the q third holds q * log2(e) / sqrt(DH)
 * instead of q -- the layout the network's QKV projection writes, which spares the kernel one
 * multiplication per score; the result is the same function of the unscaled q. */
br_status br_op_attention(int32_t dtype, const void* qkv, void* out, int32_t B, int32_t L,
                          int32_t NH, int32_t DH, int32_t q_prescaled, void* stream);

/* out[r, :] = LayerNorm(x[src(r), :]) * (1 + scale) + shift, eps 1e-6, no affine;
 * r = b*rows_per_sample + tok, src(r) = b*L_in + tok; shift / scale are the rows
 * mods + cond[b]*mods_stride + {shift_off, scale_off}.  x dev fp32, out dev `dtype`. */
br_status br_op_ln_modulate(int32_t dtype, const float* x, void* out, int32_t n_rows,
                            int32_t rows_per_sample, int32_t L_in, int32_t H, const float* mods,
                            int32_t mods_stride, int32_t shift_off, int32_t scale_off,
                            const int32_t* cond, void* stream);

/* Per-launch timing of the main kernels with HIP events recorded on the launch
 * stream around each launch (off by default; single-threaded use).  While enabled
 * every instrumented launch adds one record; br_profile_read waits for the
 * recorded events, sums work (flops for GEMM and attention, bytes for the others)
 * and milliseconds per kernel id, clears the records and returns up to max_ids
 * entries.  Ids: GEMM = epilogue*8 + tile variant; attention = 100 + head dim;
 * 200 SDE step, 201 log-prob re-evaluation, 300 LayerNorm-modulate, 301 adaLN modulation GEMV
 * (bytes = the weights it streams), 400 / 401 / 402 the fused rows of a narrow bf16 network: head, a block, the last
 * block (flops). */
br_status br_profile_enable(int32_t on);
br_status br_profile_read(int32_t max_ids, int32_t* ids, double* work, double* ms,
                          int64_t* launches, int32_t* n_ids);

#ifdef __cplusplus
}
#endif
#endif
