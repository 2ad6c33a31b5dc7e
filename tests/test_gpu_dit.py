"""GPU parity of the velocity network: single ops against numpy fp64 on the same
inputs, and the whole forward against the oracle, teacher-forced (fp32: relative
L2 error <= 1e-4; bf16: <= 2e-2)."""
import numpy as np
import pytest
import torch

from oracle import dit
from paper_2509_06040_amd import binding as br
from paper_2509_06040_amd import synth
from gpu_util import DEV, assert_velocity, bytes_buffer, cond_dev, dev, host, make_model, rel_l2

pytestmark = pytest.mark.gpu


def _bf(a):
    return synth.from_bf16_bits(synth.to_bf16_bits(a))


@pytest.mark.parametrize("M,N,K", [(37, 64, 16), (130, 192, 64), (300, 100, 256)])
def test_gemm_fp32(lib, M, N, K):
    rng = np.random.default_rng(M)
    A, W, b = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K), (N,)))
    ref = A.astype(np.float64) @ W.astype(np.float64).T + b
    out = torch.empty((M, N), device=DEV)
    br.op_gemm(br.F32, 0, dev(A), dev(W), dev(b), out)
    assert rel_l2(host(out), ref) < 1e-6
    br.op_gemm(br.F32, 1, dev(A), dev(W), dev(b), out)
    assert rel_l2(host(out), dit.gelu_tanh(ref)) < 1e-5


@pytest.mark.parametrize("variant", [4, 5, 6, 7, 7 | (2 << 4), 4 | (3 << 4), 6 | (1 << 4), -1])
@pytest.mark.parametrize("M,N,K", [(1, 128, 64), (129, 64, 64), (1101, 384, 128), (2 * 1101 + 5, 1024, 256), (700, 36, 192), (515, 640, 320), (5000, 4096, 128), (9000, 1280, 384)])
def test_gemm_bf16_every_tile_shape(lib, variant, M, N, K):
    rng = np.random.default_rng(M + N)
    A, W = _bf(rng.standard_normal((M, K)).astype(np.float32)), _bf(rng.standard_normal((N, K)).astype(np.float32) * 0.05)
    b = rng.standard_normal(N).astype(np.float32)
    ref = A.astype(np.float64) @ W.astype(np.float64).T + b
    Ad, Wd = dev(A, torch.bfloat16), dev(W, torch.bfloat16)
    out32 = torch.full((M, N), -9.0, device=DEV)
    if variant >= 0 and (variant & 15) == 7 and K % 128:
        with pytest.raises(br.BranchRolloutError) as e:      # the streaming kernel needs K % 128 == 0
            br.op_gemm(br.BF16, 4, Ad, Wd, dev(b), out32, variant=variant)
        assert e.value.code == -3
        return
    br.op_gemm(br.BF16, 4, Ad, Wd, dev(b), out32, variant=variant)
    assert rel_l2(host(out32), ref) < 1e-5, rel_l2(host(out32), ref)
    out16 = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    br.op_gemm(br.BF16, 0, Ad, Wd, dev(b), out16, variant=variant)
    assert np.array_equal(host(out16), _bf(host(out32)))          # same accumulators, rounded once
    br.op_gemm(br.BF16, 1, Ad, Wd, dev(b), out16, variant=variant)
    assert rel_l2(host(out16), dit.gelu_tanh(ref)) < 4e-3


def test_gemm_gated_residual_epilogue(lib):
    rng = np.random.default_rng(0)
    L, B, N, K, C, Astr = 50, 3, 128, 64, 2, 700
    M = L * B
    A, W = _bf(rng.standard_normal((M, K)).astype(np.float32)), _bf(rng.standard_normal((N, K)).astype(np.float32) * 0.1)
    b, x0 = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    mods = rng.standard_normal((C, Astr)).astype(np.float32)
    cond = np.array([1, 0, 1], np.int32)
    gate = mods[cond][:, 256:256 + N]
    ref = x0 + np.repeat(gate, L, axis=0) * (A.astype(np.float64) @ W.astype(np.float64).T + b)
    for dt, tol in ((br.BF16, 1e-5), (br.F32, 1e-6)):
        x = dev(x0.copy())
        tdt = torch.bfloat16 if dt == br.BF16 else torch.float32
        br.op_gemm(dt, 2, dev(A, tdt), dev(W, tdt), dev(b), x, mods=dev(mods), gate_off=256, cond=dev(cond), L=L)
        assert rel_l2(host(x), ref) < tol


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_gemm_tile_height_of_a_sparse_last_round_matches_full_height_and_fp64(lib, mode):
    """16 samples of 1101 tokens and 1024 output columns are 1.08 rounds of 256x256 tiles on 256 compute units: the library takes
    tiles of 160 rows.  Same bits as tiles of 256 rows, and right against fp64 on sampled rows around tile and sample
    boundaries (each sample with its own gate)."""
    rng = np.random.default_rng(mode)
    L, B, N, K, C = 1101, 16, 1024, 256, 5
    M = L * B
    A, W = _bf(rng.standard_normal((M, K)).astype(np.float32)), _bf(rng.standard_normal((N, K)).astype(np.float32) * 0.05)
    b = rng.standard_normal(N).astype(np.float32)
    Ad, Wd, bd = dev(A, torch.bfloat16), dev(W, torch.bfloat16), dev(b)
    rows = np.concatenate([np.arange(0, 3), np.arange(14 * L - 2, 14 * L + 3), np.arange(15 * L - 2, 15 * L + 2), np.arange(16382, 16387), np.arange(M - 3, M)])
    lin = A[rows].astype(np.float64) @ W.astype(np.float64).T + b
    if mode == 2:
        x0 = rng.standard_normal((M, N)).astype(np.float32)
        mods = rng.standard_normal((C, N)).astype(np.float32)
        cond = (np.arange(B) * 3 % C).astype(np.int32)
        outs = []
        for variant in (-1, 7):
            x = dev(x0.copy())
            br.op_gemm(br.BF16, 2, Ad, Wd, bd, x, mods=dev(mods), gate_off=0, cond=dev(cond), L=L, variant=variant)
            outs.append(x)
        ref = x0[rows] + mods[cond[rows // L]] * lin
        tol = 1e-5
    else:
        outs = []
        for variant in (-1, 7):
            out = torch.full((M, N), 3.0, dtype=torch.bfloat16, device=DEV)
            br.op_gemm(br.BF16, mode, Ad, Wd, bd, out, variant=variant)
            outs.append(out)
        ref = dit.gelu_tanh(lin) if mode == 1 else lin
        tol = 4e-3
    assert torch.equal(outs[0], outs[1])
    assert rel_l2(host(outs[0].float())[rows], ref) < tol


STREAM = {4: 8, 5: 9, 6: 10, 7: 11, 8: 7}  # variant of the persistent kernel by rows of a tile in units of 32


@pytest.mark.parametrize("height", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("M,N,K,L", [(32, 256, 128, 32), (255, 260, 256, 255), (1290, 772, 384, 129), (2 * 1101, 1024, 256, 1101), (640, 128, 128, 20)])
def test_gemm_persistent_tile_heights(lib, height, M, N, K, L):
    """Every tile height: one stage pair and more, ragged rows and columns, samples that end inside a wave's
    rows (L 129, 1101) and more than two of them (L 20), nothing written past the last row."""
    rng = np.random.default_rng(M + N + height)
    A, W = _bf(rng.standard_normal((M, K)).astype(np.float32)), _bf(rng.standard_normal((N, K)).astype(np.float32) * 0.05)
    b, x0 = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    mods = rng.standard_normal((M // L, N)).astype(np.float32)
    Ad, Wd, bd = dev(A, torch.bfloat16), dev(W, torch.bfloat16), dev(b)
    lin = A.astype(np.float64) @ W.astype(np.float64).T + b
    variant = STREAM[height]
    out = torch.full((M + 8, N), -9.0, device=DEV)
    br.op_gemm(br.BF16, 4, Ad, Wd, bd, out[:M], variant=variant)
    assert rel_l2(host(out[:M]), lin) < 1e-5 and bool((out[M:] == -9.0).all())
    for mode, ref in ((0, lin), (1, dit.gelu_tanh(lin))):
        o16 = torch.full((M + 8, N), -9.0, dtype=torch.bfloat16, device=DEV)
        br.op_gemm(br.BF16, mode, Ad, Wd, bd, o16[:M], variant=variant)
        assert rel_l2(host(o16[:M].float()), ref) < 4e-3 and bool((o16[M:] == -9.0).all())
    x = torch.full((M + 8, N), -9.0, device=DEV)
    x[:M] = dev(x0)
    cond = np.arange(M // L, dtype=np.int32)[::-1].copy()
    br.op_gemm(br.BF16, 2, Ad, Wd, bd, x[:M], mods=dev(mods), gate_off=0, cond=dev(cond), L=L, variant=variant)
    assert rel_l2(host(x[:M]), x0 + np.repeat(mods[cond], L, axis=0) * lin) < 1e-5 and bool((x[M:] == -9.0).all())


def _attention_ref(qkv, nh):
    B, L, H3 = qkv.shape
    H = H3 // 3
    return np.stack([dit.attention(qkv[b, :, :H], qkv[b, :, H:2 * H], qkv[b, :, 2 * H:], nh) for b in range(B)])


@pytest.mark.parametrize("dh,nh,L,B", [(16, 4, 24, 2), (32, 2, 100, 1), (64, 2, 77, 1), (128, 1, 130, 2)])
def test_attention_fp32(lib, dh, nh, L, B):
    rng = np.random.default_rng(dh + L)
    qkv = rng.standard_normal((B, L, 3 * nh * dh)).astype(np.float32)
    out = torch.empty((B, L, nh * dh), device=DEV)
    br.op_attention(br.F32, dev(qkv), out, nh)
    assert rel_l2(host(out), _attention_ref(qkv.astype(np.float64), nh)) < 2e-6


# the last four: enough (sample, head) pairs for the XCD-grouped tile order, with ragged query
# and key tiles, one key tile only, and the last sample ending at the end of the buffer
@pytest.mark.parametrize("dh,nh,L,B", [(64, 2, 1, 1), (64, 3, 77, 2), (64, 2, 1101, 1), (128, 2, 130, 2), (128, 1, 640, 1),
                                        (64, 1, 128, 1), (64, 16, 203, 3), (128, 8, 150, 5), (64, 12, 63, 3),
                                        (128, 9, 257, 4)])
def test_attention_bf16(lib, dh, nh, L, B):
    rng = np.random.default_rng(dh + L)
    qkv = _bf(rng.standard_normal((B, L, 3 * nh * dh)).astype(np.float32) * 1.5)
    out = torch.full((B, L, nh * dh), 3.0, dtype=torch.bfloat16, device=DEV)
    br.op_attention(br.BF16, dev(qkv, torch.bfloat16), out, nh)
    ref = _attention_ref(qkv.astype(np.float64), nh)
    err = rel_l2(host(out), ref)
    assert err < 3e-3, err                       # bf16 probabilities and output rounding (measured 1.8e-3)


@pytest.mark.parametrize("dh,nh,L,B", [(64, 2, 77, 2), (64, 4, 1101, 1), (128, 2, 130, 2), (128, 9, 257, 4), (64, 12, 63, 3)])
def test_attention_bf16_prescaled_queries(lib, dh, nh, L, B):
    """The layout the network's QKV projection writes: q * log2(e) / sqrt(dh) in the q third.  The
    result is softmax attention of the q that these bf16 values stand for."""
    rng = np.random.default_rng(dh + L)
    H = nh * dh
    c = np.log2(np.e) / np.sqrt(dh)
    qkv = rng.standard_normal((B, L, 3 * H)).astype(np.float32) * 1.5
    qkv[..., :H] *= c
    qkv = _bf(qkv)
    out = torch.full((B, L, H), 3.0, dtype=torch.bfloat16, device=DEV)
    br.op_attention(br.BF16, dev(qkv, torch.bfloat16), out, nh, q_prescaled=1)
    plain = qkv.astype(np.float64)
    plain[..., :H] /= c
    err = rel_l2(host(out), _attention_ref(plain, nh))
    assert err < 3e-3, err
    raw = br.load()
    import ctypes as C
    p = C.c_void_p(out.data_ptr())
    assert raw.br_op_attention(br.F32, p, p, 1, 16, 2, 64, 1, None) == -1     # fp32 has no prescaled layout


@pytest.mark.parametrize("jump", [40.0, -200.0])
def test_attention_bf16_reference_follows_the_scores(lib, jump):
    """jump > 0: keys 300.. score about `jump` (in powers of two) above everything before them, so
    the kernel's softmax reference has to move mid-sequence.  jump < 0: every score sits that far
    below zero, so the first tile must not start from a reference of zero."""
    rng = np.random.default_rng(7)
    dh, nh, L, B = 64, 2, 400, 1
    H = nh * dh
    qkv = rng.standard_normal((B, L, 3 * H)).astype(np.float32)
    u = rng.standard_normal(dh).astype(np.float32)
    u /= np.linalg.norm(u)
    a = 4.0
    b = jump * np.sqrt(dh) / np.log2(np.e) / a          # a b / sqrt(dh) * log2(e) = jump
    for h in range(nh):
        qkv[0, :, h * dh:(h + 1) * dh] += a * u
        first = 300 if jump > 0 else 0
        qkv[0, first:, H + h * dh:H + (h + 1) * dh] += b * u
    qkv = _bf(qkv)
    out = torch.full((B, L, H), 3.0, dtype=torch.bfloat16, device=DEV)
    br.op_attention(br.BF16, dev(qkv, torch.bfloat16), out, nh)
    got = host(out)
    assert np.isfinite(got).all()
    err = rel_l2(got, _attention_ref(qkv.astype(np.float64), nh))
    assert err < 3e-3, err


def test_attention_bf16_rejects_what_it_cannot_address(lib):
    import ctypes as C
    raw = br.load()
    buf = torch.zeros(64, dtype=torch.bfloat16, device=DEV)
    p = C.c_void_p(buf.data_ptr())
    # rows of one sample beyond 4 GiB (the check precedes any launch; the buffers are never touched)
    assert raw.br_op_attention(br.BF16, p, p, 1, 400000, 16, 128, 0, None) == -3
    assert b"4 GiB" in raw.br_last_error()
    assert raw.br_op_attention(br.BF16, p, p, 1, 16, 2, 32, 0, None) == -3          # head dim 32 in bf16
    assert raw.br_op_attention(br.BF16, p, p, 1, 0, 2, 64, 0, None) == -1


@pytest.mark.parametrize("dt", [br.F32, br.BF16])
def test_ln_modulate(lib, dt):
    rng = np.random.default_rng(1)
    B, L, n_img, H, C, Astr = 3, 9, 7, 192, 2, 1000
    x = (rng.standard_normal((B * L, H)) * 3 + 1).astype(np.float32)
    mods = rng.standard_normal((C, Astr)).astype(np.float32) * 0.3
    cond = np.array([0, 1, 1], np.int32)
    tdt = torch.bfloat16 if dt == br.BF16 else torch.float32
    tol = 4e-3 if dt == br.BF16 else 2e-6
    for rows, so, co in ((L, 0, H), (n_img, 400, 600)):
        out = torch.empty((B * rows, H), dtype=tdt, device=DEV)
        br.op_ln_modulate(dt, dev(x), out, rows, L, dev(mods), so, co, dev(cond))
        xs = x.reshape(B, L, H)[:, :rows].astype(np.float64)
        m = mods[cond].astype(np.float64)
        ref = dit.layer_norm(xs) * (1 + m[:, None, co:co + H]) + m[:, None, so:so + H]
        assert rel_l2(host(out).reshape(B, rows, H), ref) < tol


@pytest.mark.parametrize("dt", [br.F32, br.BF16])
@pytest.mark.parametrize("B,L,H", [(1, 1, 256), (3, 5, 512), (2, 3, 768), (5, 7, 1024), (2, 9, 1536), (1, 3, 2048), (2, 2, 3072), (3, 11, 260),
                                   (1, 9765, 3072), (4, 7813, 1024)])
def test_ln_modulate_row_lengths(lib, dt, B, L, H):
    """Each way a row is held, with samples that share a workgroup, and launches on both sides of the size from which rows are stored past
    the caches (192 MB read and written).  The bound: one rounding to bf16 (2^-9), fp32 sums elsewhere."""
    g = torch.Generator(device=DEV)
    g.manual_seed(H + L)
    x = torch.randn((B * L, H), generator=g, device=DEV) * 2 + 0.5
    mods = torch.randn((B, 2 * H + 8), generator=g, device=DEV) * 0.3
    cond = torch.arange(B - 1, -1, -1, dtype=torch.int32, device=DEV)
    out = torch.empty((B * L, H), dtype=torch.bfloat16 if dt == br.BF16 else torch.float32, device=DEV)
    br.op_ln_modulate(dt, x, out, L, L, mods, 0, H + 8, cond)
    for b in range(B):
        m, xs = mods[B - 1 - b].double(), x[b * L:(b + 1) * L].double()
        xs = xs - xs.mean(1, keepdim=True)
        ref = xs / (xs.square().mean(1, keepdim=True) + 1e-6).sqrt() * (1 + m[H + 8:2 * H + 8]) + m[:H]
        err = (out[b * L:(b + 1) * L].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert float(err.max()) < (2.0 ** -9 if dt == br.BF16 else 2e-6), b


@pytest.mark.parametrize("dt", [br.F32, br.BF16])
@pytest.mark.parametrize("rows,H", [(125004, 256), (62505, 512), (41700, 768), (31270, 1024), (20900, 1536), (15700, 2048), (10500, 3072), (33000, 992)])
def test_ln_modulate_bits_do_not_depend_on_the_launch(lib, dt, rows, H):
    """A launch whose rows are stored past the caches (long ones summed through the LDS unit) and the same rows in small launches: the same bits."""
    g = torch.Generator(device=DEV)
    g.manual_seed(H)
    x, mods = torch.randn((rows, H), generator=g, device=DEV) * 2 + 0.5, torch.randn((1, 2 * H), generator=g, device=DEV)
    cond, tdt = torch.zeros(1, dtype=torch.int32, device=DEV), torch.bfloat16 if dt == br.BF16 else torch.float32
    out = torch.empty((rows, H), dtype=tdt, device=DEV)
    br.op_ln_modulate(dt, x, out, rows, rows, mods, 0, H, cond)
    for lo in range(0, rows, 2500):
        part = torch.empty((min(2500, rows - lo), H), dtype=tdt, device=DEV)
        br.op_ln_modulate(dt, x[lo:lo + 2500], part, len(part), len(part), mods, 0, H, cond)
        assert torch.equal(out[lo:lo + 2500], part), lo


def _velocity_case(cfg, n_cond, B, t, seed, std=0.02):
    W = synth.make_weights(cfg, seed, std)
    D = synth.model_sizes(cfg)["D"]
    z = synth.random_latents(B, D, seed + 1)
    cond = synth.cond_tokens(cfg, n_cond, seed + 2)
    cidx = np.arange(B) % n_cond
    model = make_model(cfg, W)
    ws = bytes_buffer(br.workspace_bytes(None, model, B))
    v = torch.full((B, D), 5.0, device=DEV)
    br.velocity(model, dev(z), t, cond_dev(cfg, cond), cidx, v, ws)
    rnd = dit.round_bf16 if cfg["dtype"] == synth.BF16 else dit.identity
    ref = dit.forward(cfg, W, z, t, cond, cidx, act_round=rnd)
    return host(v), ref, (model, W, z, cond, cidx)


def test_velocity_tiny_fp32_matches_oracle(lib):
    cfg = synth.WORKLOADS["tiny"]["model"]
    for t, std in ((1.0, 0.02), (0.37, 0.02), (0.05, 0.2)):
        got, ref, _ = _velocity_case(cfg, 2, 5, t, 0, std)
        for b in range(5):
            assert_velocity(cfg, got[b], ref[b], 1e-4, "tiny t=%g b=%d" % (t, b))   # stated fp32 tolerance


def test_velocity_fp32_other_shapes(lib):
    # temporal patches, head dim 32, ragged token count
    cfg = synth.model_cfg(2, 64, 2, (3, 4, 6, 10), (2, 2, 2), 5, synth.F32)
    got, ref, _ = _velocity_case(cfg, 3, 4, 0.6, 3, 0.1)
    for b in range(4):
        assert_velocity(cfg, got[b], ref[b], 1e-4, "fp32 shapes b=%d" % b)


def test_velocity_small_bf16_matches_oracle(lib):
    for cfg in (synth.model_cfg(2, 128, 2, (16, 1, 16, 20), (1, 2, 2), 13, synth.BF16),          # d_h 64, L = 93
                synth.model_cfg(1, 256, 2, (16, 2, 8, 12), (1, 2, 2), 70, synth.BF16)):         # d_h 128, L = 166
        got, ref, _ = _velocity_case(cfg, 2, 3, 0.5, 1, 0.05)
        for b in range(3):
            assert_velocity(cfg, got[b], ref[b], 2e-2, "small bf16 b=%d" % b)                   # stated bf16 tolerance


@pytest.mark.parametrize("hidden,heads,dtype,B", [(48, 3, synth.F32, 1), (32, 2, synth.F32, 9), (256, 8, synth.F32, 2), (272, 17, synth.F32, 1),
                                                  (64, 1, synth.BF16, 2), (192, 3, synth.BF16, 3), (512, 4, synth.BF16, 1), (576, 9, synth.BF16, 1)])
def test_velocity_normalisation_inside_the_gemm(lib, hidden, heads, dtype, B):
    """Hidden sizes of a part of a stage, of whole stages, the largest whose rows fit beside the operands (256 in fp32,
    512 in bf16) and the next; rows that end inside a tile."""
    cfg = synth.model_cfg(2, hidden, heads, (16, 1, 6, 10), (1, 2, 2), 5, dtype)
    got, ref, _ = _velocity_case(cfg, min(2, B), B, 0.4, 2, 0.05)
    for b in range(B):
        assert_velocity(cfg, got[b], ref[b], 1e-4 if dtype == synth.F32 else 2e-2, "hidden %d b=%d" % (hidden, b))


@pytest.mark.parametrize("dtype,B", [(synth.F32, 1), (synth.BF16, 3), (synth.F32, 9)])
def test_velocity_modulation_vectors_four_columns_a_wave(lib, dtype, B):
    """6 x 6 x 512 + 2 x 512 modulation columns, above 64 a compute unit; one group, a few, and more than the eight that a wave takes together."""
    cfg = synth.model_cfg(6, 512, 4, (16, 1, 4, 6), (1, 2, 2), 5, dtype)
    got, ref, _ = _velocity_case(cfg, B, B, 0.4, 6, 0.05)
    for b in range(B):
        assert_velocity(cfg, got[b], ref[b], 1e-4 if dtype == synth.F32 else 2e-2, "modulation b=%d" % b)


def test_velocity_chunked_batches_agree(lib):
    cfg = synth.WORKLOADS["tiny"]["model"]
    got, ref, (model, W, z, cond, cidx) = _velocity_case(cfg, 2, 5, 0.5, 4)
    small = bytes_buffer(br.workspace_bytes(None, model, 2) + 64)       # forces chunks of <= 2
    v2 = torch.empty_like(torch.from_numpy(got)).to(DEV)
    br.velocity(model, dev(z), 0.5, cond_dev(cfg, cond), cidx, v2, small)
    assert np.array_equal(host(v2), got)
    with pytest.raises(br.BranchRolloutError) as e:
        br.velocity(model, dev(z), 0.5, cond_dev(cfg, cond), cidx, v2, bytes_buffer(256))
    assert e.value.code == -4


# every form of the fp32 GEMM (32x32 tiles, the ring kernel in 64 and 128 columns; its choice, which the last shape gives to the ring) at tile
# edges, with K of less than one stage, one to 32 whole stages of 32 (the ring has two slots; where K is not
# a multiple of 32 the 32x32 tiles take over) and a stage that ends inside a 16-byte chunk pair
@pytest.mark.parametrize("variant", [-1, 0, 6 | (3 << 24), 6 | (8 << 24) | 16])
@pytest.mark.parametrize("M,N,K", [(1, 4, 4), (31, 36, 12), (33, 132, 16), (64, 128, 20), (65, 124, 32), (129, 260, 144),
                                   (257, 128, 1040), (1000, 516, 96), (129, 132, 64), (65, 260, 128), (257, 124, 160), (130, 388, 1024), (1005, 1028, 96)])
def test_gemm_fp32_every_form(lib, variant, M, N, K):
    rng = np.random.default_rng(M * 7 + K)
    A, W, b = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K), (N,)))
    ref = A.astype(np.float64) @ W.astype(np.float64).T + b
    out = torch.full((M + 1, N), -9.0, device=DEV)
    br.op_gemm(br.F32, 0, dev(A), dev(W), dev(b), out[:M], variant=variant)
    # fp32 sums of K products: rounding errors of 2^-24 each add up to about sqrt(K) 2^-24 < 2e-6 of the norm
    assert rel_l2(host(out)[:M], ref) < 2e-6
    assert (host(out)[M] == -9.0).all()
    L = 1 if M % 5 else 5
    x0, mods = rng.standard_normal((M, N)).astype(np.float32), rng.standard_normal((3, N)).astype(np.float32)
    cond = (np.arange(M // L) % 3).astype(np.int32)
    x = dev(x0.copy())
    br.op_gemm(br.F32, 2, dev(A), dev(W), dev(b), x, mods=dev(mods), gate_off=0, cond=dev(cond), L=L, variant=variant)
    assert rel_l2(host(x), x0 + np.repeat(mods[cond], L, axis=0) * ref) < 2e-6


@pytest.mark.parametrize("off,K", [(1, 64), (0, 30), (2, 33)])
def test_gemm_fp32_operands_that_are_not_16_byte_aligned(lib, off, K):
    rng = np.random.default_rng(K)
    M, N = 70, 72
    A, W, b = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K), (N,)))
    buf = torch.zeros(M * K + off, device=DEV)
    buf[off:] = dev(A).reshape(-1)
    out = torch.empty((M, N), device=DEV)
    br.op_gemm(br.F32, 0, buf[off:].view(M, K), dev(W), dev(b), out)
    assert rel_l2(host(out), A.astype(np.float64) @ W.astype(np.float64).T + b) < 1e-6


@pytest.mark.parametrize("patch,latent", [((1, 1, 1), (4, 1, 5, 7)), ((1, 3, 3), (4, 2, 6, 9)), ((2, 1, 4), (2, 4, 3, 8))])
def test_velocity_fp32_patch_widths(lib, patch, latent):
    """Odd and even patch widths: the unpatchify epilogue stores single elements or pairs."""
    cfg = synth.model_cfg(1, 32, 2, latent, patch, 3, synth.F32)
    got, ref, _ = _velocity_case(cfg, 2, 2, 0.4, 5, 0.1)
    for b in range(2):
        assert_velocity(cfg, got[b], ref[b], 1e-4, "patch %s b=%d" % (patch, b))


# one key, one tile of 32 keys and its neighbours, fewer tiles than waves, every wave with a different
# number of tiles; the last two have enough (sample, head) pairs for the grouped order
@pytest.mark.parametrize("dh,nh,L,B", [(16, 1, 1, 1), (32, 2, 31, 1), (64, 1, 32, 2), (128, 2, 33, 1), (16, 3, 97, 2),
                                       (64, 2, 161, 1), (128, 1, 290, 1), (32, 8, 70, 4), (16, 11, 40, 3)])
def test_attention_fp32_tile_edges(lib, dh, nh, L, B):
    rng = np.random.default_rng(dh + L)
    qkv = (rng.standard_normal((B, L, 3 * nh * dh)) * 1.5).astype(np.float32)
    out = torch.full((B, L, nh * dh), 3.0, device=DEV)
    br.op_attention(br.F32, dev(qkv), out, nh)
    assert rel_l2(host(out), _attention_ref(qkv.astype(np.float64), nh)) < 2e-6


def test_attention_fp32_reference_moves_and_unaligned_buffers(lib):
    """Scores that jump by hundreds between key tiles, in either direction; and the same call on buffers
    that are only 4-byte aligned."""
    rng = np.random.default_rng(2)
    nh, dh, L = 2, 32, 200
    qkv = rng.standard_normal((1, L, 3 * nh * dh)).astype(np.float32)
    H = nh * dh
    qkv[0, :, :H] += 3.0
    qkv[0, 64:96, H:2 * H] += 20.0
    qkv[0, 96:128, H:2 * H] -= 20.0
    ref = _attention_ref(qkv.astype(np.float64), nh)
    out = torch.empty((1, L, H), device=DEV)
    br.op_attention(br.F32, dev(qkv), out, nh)
    # exponents reach 340: a relative rounding of 2^-24 of the score is 4e-5 of the probability
    assert rel_l2(host(out), ref) < 1e-4
    buf, obuf = torch.zeros(qkv.size + 1, device=DEV), torch.zeros(L * H + 1, device=DEV)
    buf[1:] = dev(qkv).reshape(-1)
    br.op_attention(br.F32, buf[1:].view(1, L, 3 * H), obuf[1:].view(1, L, H), nh)
    assert rel_l2(host(obuf)[1:].reshape(1, L, H), ref) < 1e-4


# the bf16 forms for small and middle sizes: 32x32, 64x64 and 64x128 tiles, 128x128 in eight waves; K of one
# stage, fewer stages than the ring or than waves, and more; ragged rows and columns
@pytest.mark.parametrize("variant", [0, 1, 2, 3, 2 | (1 << 4), 3 | (3 << 4)])
@pytest.mark.parametrize("M,N,K", [(1, 4, 64), (31, 64, 128), (33, 132, 192), (65, 36, 256), (127, 192, 320), (130, 260, 1088)])
def test_gemm_bf16_small_tiles(lib, variant, M, N, K):
    rng = np.random.default_rng(M + K)
    A, W = _bf(rng.standard_normal((M, K)).astype(np.float32)), _bf(rng.standard_normal((N, K)).astype(np.float32) * 0.05)
    b = rng.standard_normal(N).astype(np.float32)
    ref = A.astype(np.float64) @ W.astype(np.float64).T + b
    Ad, Wd, bd = dev(A, torch.bfloat16), dev(W, torch.bfloat16), dev(b)
    out = torch.full((M + 1, N), -9.0, device=DEV)
    br.op_gemm(br.BF16, 4, Ad, Wd, bd, out[:M], variant=variant)
    # exact products, fp32 sums of K of them: about sqrt(K) 2^-24 < 2e-6 of the norm
    assert rel_l2(host(out)[:M], ref) < 2e-6 and (host(out)[M] == -9.0).all()
    out16 = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    br.op_gemm(br.BF16, 0, Ad, Wd, bd, out16, variant=variant)
    assert np.array_equal(host(out16), _bf(host(out)[:M]))        # same accumulators, rounded once
    L = 1 if M % 5 else 5
    x0, mods = rng.standard_normal((M, N)).astype(np.float32), rng.standard_normal((3, N)).astype(np.float32)
    cond = (np.arange(M // L) % 3).astype(np.int32)
    x = dev(x0.copy())
    br.op_gemm(br.BF16, 2, Ad, Wd, bd, x, mods=dev(mods), gate_off=0, cond=dev(cond), L=L, variant=variant)
    assert rel_l2(host(x), x0 + np.repeat(mods[cond], L, axis=0) * ref) < 2e-6


# Every kernel of either dtype adds k in ascending order, so a result has the same bits whichever a problem size selects.
# K of one stage, of less or more whole stages than a ring holds, and (fp32) ends inside a stage; ragged rows and columns.
@pytest.mark.parametrize("dt,M,N,K", [(br.BF16, 93, 128, 256), (br.BF16, 1101, 260, 1024), (br.BF16, 40, 64, 3072), (br.BF16, 300, 132, 64),
                                      (br.BF16, 70, 512, 1088), (br.F32, 33, 36, 20), (br.F32, 65, 132, 32), (br.F32, 70, 64, 144),
                                      (br.F32, 300, 260, 256), (br.F32, 1101, 132, 1024), (br.F32, 40, 64, 1056)])
def test_gemm_bits_do_not_depend_on_the_kernel(lib, dt, M, N, K):
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)
    tdt = torch.bfloat16 if dt == br.BF16 else torch.float32
    A, W = (torch.randn(s, generator=g, device=DEV).to(tdt) for s in ((M, K), (N, K)))
    b = torch.randn(N, generator=g, device=DEV)
    mode = 4 if dt == br.BF16 else 0          # fp32 outputs; (fp32 operands: bias, which has every tile form)

    def run(A, variant):
        out = torch.full((A.shape[0], N), -9.0, device=DEV)
        br.op_gemm(dt, mode, A, W, b, out, variant=variant)
        return out
    ref = run(A, 0)
    variants = [-1, 1, 2, 3, 4, 5, 6] + ([7] if K % 128 == 0 else [])
    if dt == br.F32:  # (3 and 5, kernels of earlier versions, are the library's choice; so is the ring where it does not apply)
        variants = [-1, 3, 5] + [6 | (h << 24) | cols for h in (2, 5, 9, 12) for cols in (0, 16)]
    for v in variants:
        assert torch.equal(run(A, v), ref), v
    # the automatic choice for a few rows alone, and for the same rows at the end of a large problem
    lone = run(A[:31], -1)
    assert torch.equal(lone, ref[:31])
    large = torch.cat([A.repeat(12000 // M, 1), A[:31]])
    assert torch.equal(run(large, -1)[-31:], lone)
    if dt == br.F32:  # operands that only the vector kernel takes
        buf = torch.empty(M * K + 1, device=DEV)
        buf[1:] = A.reshape(-1)
        assert torch.equal(run(buf[1:].view(M, K), -1), ref)


@pytest.mark.parametrize("hidden,heads,lat,cond,dtype,B", [(1024, 16, (16, 1, 64, 64), 77, synth.BF16, 13), (1536, 12, (16, 3, 20, 24), 512, synth.BF16, 36),
                                                           (1024, 16, (16, 1, 32, 32), 77, synth.F32, 5)])
def test_velocity_does_not_depend_on_the_batch(lib, hidden, heads, lat, cond, dtype, B):
    """A sample alone, in a whole batch and in chunks of one and two (small workspaces): the same bits."""
    cfg = synth.model_cfg(2, hidden, heads, lat, (1, 2, 2), cond, dtype)
    model = make_model(cfg, synth.make_weights(cfg, 3, 0.03))
    D = synth.model_sizes(cfg)["D"]
    z, c = dev(synth.random_latents(B, D, 4)), cond_dev(cfg, synth.cond_tokens(cfg, 2, 5))
    idx = np.arange(B) % 2

    def run(z, idx, ws_batch):
        v = torch.empty_like(z)
        br.velocity(model, z, 0.4, c, idx, v, bytes_buffer(br.workspace_bytes(None, model, ws_batch)))
        return v
    whole = run(z, idx, B)
    assert torch.equal(run(z, idx, 2), whole)
    alone = torch.cat([run(z[b:b + 1].clone(), idx[b:b + 1], 2) for b in range(B)])
    assert torch.equal(alone, whole)


def test_velocity_bits_where_the_mlp_moves_to_the_ring(lib):
    """The first MLP product (GELU) of one sample of 93 rows runs in 32x32 tiles, that of eight in the ring kernel: the same bits."""
    cfg = synth.model_cfg(2, 768, 12, (16, 1, 16, 20), (1, 2, 2), 13, synth.BF16)
    model = make_model(cfg, synth.make_weights(cfg, 3, 0.03))
    D = synth.model_sizes(cfg)["D"]
    z, c = dev(synth.random_latents(8, D, 4)), cond_dev(cfg, synth.cond_tokens(cfg, 2, 5))

    def run(first, n):
        v = torch.empty((n, D), device=DEV)
        br.profile_enable(True)
        try:
            br.velocity(model, z[first:first + n].contiguous(), 0.4, c, np.arange(first, first + n) % 2, v,
                        bytes_buffer(br.workspace_bytes(None, model, max(n, 2))))
            torch.cuda.synchronize()
            gelu = [i - 8 for i in br.profile_read() if 8 <= i < 16]
        finally:
            br.profile_enable(False)
        return v, gelu
    whole, kernel = run(0, 8)
    assert kernel == [6]
    for b in (0, 7):
        v, kernel = run(b, 1)
        assert kernel == [0]
        assert torch.equal(v[0], whole[b])


# (narrow networks of whole 128-byte rows run the row-local part of a block in one launch: 64 in fp32, 64 and 128 in bf16 for one sample and
# for many, in one row tile and in two; 192 in bf16 for one)
@pytest.mark.parametrize("hidden,heads,dtype", [(48, 3, synth.F32), (64, 4, synth.F32), (256, 8, synth.F32), (64, 1, synth.BF16), (128, 2, synth.BF16),
                                                (192, 3, synth.BF16), (512, 4, synth.BF16), (80, 5, synth.F32), (160, 5, synth.F32), (192, 6, synth.F32),
                                                (320, 5, synth.BF16), (384, 6, synth.BF16)])
def test_velocity_bits_where_the_normalisation_moves_into_the_gemm(lib, hidden, heads, dtype):
    """A sample alone (its rows normalised by the GEMM that reads them, or by the fused row kernel) and among enough others that every
    GEMM has more tiles than compute units (normalised by a launch of its own, or by the fused row kernel): the same bits."""
    cfg = synth.model_cfg(2, hidden, heads, (16, 1, 14, 18), (1, 2, 2), 6, dtype)
    model = make_model(cfg, synth.make_weights(cfg, 3, 0.05))
    sizes = synth.model_sizes(cfg)
    B = 256 * 32 // sizes["n_img"] + 2                    # rows of the narrowest call: the final projection, 64 columns
    z, c = dev(synth.random_latents(1, sizes["D"], 4)), cond_dev(cfg, synth.cond_tokens(cfg, 1, 5))
    fused = hidden in {synth.F32: (64,), synth.BF16: (64, 128)}[dtype]
    out = []
    for n in (1, B):
        v = torch.empty((n, sizes["D"]), device=DEV)
        br.profile_enable(True)
        try:
            br.velocity(model, z.repeat(n, 1), 0.4, c, np.zeros(n, np.int32), v, bytes_buffer(br.workspace_bytes(None, model, n)))
            torch.cuda.synchronize()
            launched = 300 in br.profile_read()           # LayerNorm launches
        finally:
            br.profile_enable(False)
        assert launched == (n > 1 and not fused)
        out.append(v)
    assert torch.equal(out[1], out[0].expand(B, -1))


@pytest.mark.parametrize("hidden,heads,lat,pt,cond,dtype,Bs", [
    (64, 1, (16, 1, 14, 18), 1, 6, synth.BF16, (1, 70, 950)), (128, 1, (16, 2, 14, 18), 2, 7, synth.BF16, (3, 200, 940)),
    (192, 3, (16, 1, 8, 6), 1, 3, synth.BF16, (1, 280)), (256, 2, (16, 1, 14, 18), 1, 6, synth.BF16, (2, 61)),
    (32, 2, (4, 1, 6, 10), 1, 2, synth.F32, (1, 300)), (64, 4, (4, 1, 8, 8), 1, 8, synth.F32, (1, 171, 2740)),
    (96, 3, (4, 2, 10, 6), 2, 5, synth.F32, (5, 250, 415)), (128, 2, (4, 1, 14, 18), 1, 6, synth.F32, (1, 61))])
def test_velocity_of_narrow_networks_with_fused_rows(lib, hidden, heads, lat, pt, cond, dtype, Bs):
    """Narrow networks run the row-local part of a block in one launch, with one or two tiles of 16 rows a workgroup (the last one
    ragged, tiles across samples), in steps of 128 or 256 bytes, patch vectors shorter than a step; from the last batch size on
    some fall back on the separate kernels.  A sample has the same bits in every batch, and is right against the oracle."""
    cfg = synth.model_cfg(2, hidden, heads, lat, (pt, 2, 2), cond, dtype)
    W = synth.make_weights(cfg, 3, 0.05)
    model = make_model(cfg, W)
    D = synth.model_sizes(cfg)["D"]
    n = max(Bs)
    z, tok = synth.random_latents(5, D, 4), synth.cond_tokens(cfg, 2, 5)
    zd, c = dev(z)[torch.arange(n, device=DEV) % 5], cond_dev(cfg, tok)
    outs = []
    for B in Bs:
        v = torch.empty((B, D), device=DEV)
        br.velocity(model, zd[:B].contiguous(), 0.4, c, np.arange(B) % 5 % 2, v, bytes_buffer(br.workspace_bytes(None, model, max(B, 2))))
        outs.append(v)
    assert_velocity(cfg, host(outs[0])[0], dit.forward(cfg, W, z[:1], 0.4, tok, np.zeros(1, np.int32))[0], 2e-2 if dtype == synth.BF16 else 1e-4)
    for v in outs[1:]:
        first = v[:min(5, len(v))]
        assert torch.equal(first[:len(outs[0])], outs[0][:len(first)])
        assert torch.equal(v, first[torch.arange(len(v), device=DEV) % 5])


# The fused rows have a form for each hidden size (MLP ratio 4, patch vectors of up to 256 bytes and 128 elements) and one for anything else: patch vectors that are
# not whole column blocks, or a step and a half of weights; just beyond the form's limits; another ratio; samples so short that their modulation vectors
# need the room.
@pytest.mark.parametrize("hidden,heads,lat,patch,cond,dtype,ratio", [
    (64, 4, (3, 1, 6, 10), (1, 2, 2), 5, synth.F32, 4), (64, 4, (5, 1, 6, 10), (1, 2, 2), 5, synth.F32, 4), (32, 2, (16, 1, 6, 10), (1, 2, 2), 5, synth.F32, 4),
    (96, 3, (12, 1, 6, 10), (1, 2, 2), 5, synth.F32, 4), (64, 4, (17, 1, 6, 10), (1, 2, 2), 5, synth.F32, 4), (128, 2, (16, 1, 6, 10), (1, 2, 2), 5, synth.F32, 2),
    (64, 1, (32, 1, 6, 10), (1, 2, 2), 5, synth.BF16, 4), (128, 1, (16, 1, 6, 10), (1, 2, 2), 5, synth.BF16, 3), (64, 1, (48, 1, 6, 10), (1, 2, 2), 5, synth.BF16, 4),
    (128, 2, (16, 1, 2, 2), (1, 2, 2), 1, synth.BF16, 4), (64, 4, (4, 1, 2, 4), (1, 2, 2), 1, synth.F32, 4), (256, 4, (16, 1, 6, 10), (1, 2, 2), 1, synth.BF16, 4)])
def test_velocity_of_fused_rows_in_either_form(lib, hidden, heads, lat, patch, cond, dtype, ratio):
    cfg = synth.model_cfg(2, hidden, heads, lat, patch, cond, dtype, ratio)
    W = synth.make_weights(cfg, 3, 0.05)
    model = make_model(cfg, W)
    D = synth.model_sizes(cfg)["D"]
    n = 4200 // synth.model_sizes(cfg)["L"] + 3             # rows in two tiles a workgroup
    z, tok = synth.random_latents(5, D, 4), synth.cond_tokens(cfg, 2, 5)
    zd, c = dev(z)[torch.arange(n, device=DEV) % 5], cond_dev(cfg, tok)
    outs = []
    for B in (5, n):
        v = torch.full((B + 1, D), 7.0, device=DEV)
        br.velocity(model, zd[:B].contiguous(), 0.4, c, np.arange(B) % 5 % 2, v[:B], bytes_buffer(br.workspace_bytes(None, model, B)))
        assert bool((v[B] == 7.0).all())
        outs.append(v[:B])
    for b in range(5):
        assert_velocity(cfg, host(outs[0])[b], dit.forward(cfg, W, z[b:b + 1], 0.4, tok, np.array([b % 2], np.int32))[0], 2e-2 if dtype == synth.BF16 else 1e-4)
    assert torch.equal(outs[1], outs[0][torch.arange(n, device=DEV) % 5])


# Rows, modulation vectors, biases and weights in flight of 160 KB to the byte: the form for any sizes, one row tile and two.
@pytest.mark.parametrize("hidden,heads,lat,ratio,n", [(128, 2, (16, 1, 6, 6), 16, 30), (192, 3, (16, 1, 6, 10), 3, 230)])
def test_velocity_of_rows_that_fill_the_lds_stays_fused(lib, hidden, heads, lat, ratio, n):
    cfg = synth.model_cfg(2, hidden, heads, lat, (1, 2, 2), 5, synth.BF16, ratio)
    W = synth.make_weights(cfg, 3, 0.05)
    model = make_model(cfg, W)
    D = synth.model_sizes(cfg)["D"]
    z, tok = synth.random_latents(3, D, 4), synth.cond_tokens(cfg, 2, 5)
    v = torch.empty((n, D), device=DEV)
    br.profile_enable(True)
    br.profile_read()
    try:
        br.velocity(model, dev(z)[torch.arange(n, device=DEV) % 3], 0.4, cond_dev(cfg, tok), np.arange(n) % 3 % 2, v, bytes_buffer(br.workspace_bytes(None, model, n)))
        assert {400, 401, 402} <= set(br.profile_read())     # head, block, last block
    finally:
        br.profile_enable(False)
    for b in range(3):
        assert_velocity(cfg, host(v)[b], dit.forward(cfg, W, z[b:b + 1], 0.4, tok, np.array([b % 2], np.int32))[0], 2e-2)
    assert torch.equal(v, v[torch.arange(n, device=DEV) % 3])


@pytest.mark.parametrize("n_cond", [1, 8, 11])
def test_velocity_conditions_passed_with_the_launch_or_transferred(lib, n_cond):
    """Up to 64 samples carry their conditions in the launch, more in a buffer; up to eight conditions share a pass over the
    weights of the conditioning path.  Each sample as it is by itself under its condition, and one right against the oracle."""
    cfg = synth.model_cfg(1, 64, 4, (4, 1, 8, 8), (1, 2, 2), 8, synth.F32)
    W = synth.make_weights(cfg, 1, 0.1)
    model, D = make_model(cfg, W), synth.model_sizes(cfg)["D"]
    z, tok = synth.random_latents(65, D, 2), synth.cond_tokens(cfg, n_cond, 3)
    idx = ((np.arange(65) * 7 + 3) % n_cond).astype(np.int32)
    out = {}
    for B in (64, 65):
        out[B] = torch.empty((B, D), device=DEV)
        br.velocity(model, dev(z[:B]), 0.6, dev(tok), idx[:B], out[B], bytes_buffer(br.workspace_bytes(None, model, B)))
    assert torch.equal(out[64], out[65][:64])
    for b in (0, 37, 64):
        one = torch.empty((1, D), device=DEV)
        br.velocity(model, dev(z[b:b + 1]), 0.6, dev(tok[idx[b]:idx[b] + 1]), np.zeros(1, np.int32), one, bytes_buffer(br.workspace_bytes(None, model, 1)))
        assert torch.equal(one[0], out[65][b])
    assert_velocity(cfg, host(out[65])[64], dit.forward(cfg, W, z[64:], 0.6, tok, idx[64:])[0], 1e-4)


@pytest.mark.parametrize("n_tok", [64, 300])
def test_condition_mean_adds_the_tokens_in_order(lib, n_tok):
    """1 + 2^-24 rounds to 1 in fp32, so in token order the small tokens behind the first one leave no trace; added among
    themselves first, they would.  The tokens' own embeddings are switched off (zero weights)."""
    cfg = synth.model_cfg(1, 64, 4, (4, 1, 8, 8), (1, 2, 2), n_tok, synth.F32)
    W = synth.make_weights(cfg, 1, 0.1)
    W["cond_w"][:] = 0.0
    cond = np.zeros((2, n_tok, cfg["cond_dim"]), np.float32)
    cond[:, 0] = 1.0
    cond[1, 1:] = 2.0 ** -24
    model = make_model(cfg, W)
    z = dev(np.repeat(synth.random_latents(1, synth.model_sizes(cfg)["D"], 2), 2, axis=0))
    v = torch.empty_like(z)
    br.velocity(model, z, 0.6, dev(cond), np.array([0, 1], np.int32), v, bytes_buffer(br.workspace_bytes(None, model, 2)))
    assert torch.equal(v[0], v[1])


@pytest.mark.parametrize("dh,L", [(16, 33), (64, 45), (128, 70), (32, 131)])
def test_attention_fp32_infinite_values_and_scores(lib, dh, L):
    """An infinite value is an infinite output where its key is not masked, the last key of a ragged tile among them; keys that
    score -inf throughout the first tile of a wave (or of all but one) have no weight; only where all keys do there is no result."""
    rng = np.random.default_rng(L)
    qkv = rng.standard_normal((1, L, 3 * dh)).astype(np.float32)
    qkv[0, :, 0] = 1.0                                     # every query scores key j with k[j, 0] + finite
    def run(qkv):
        out = torch.empty((1, L, dh), device=DEV)
        br.op_attention(br.F32, dev(qkv), out, 1)
        return host(out)[0]
    a = qkv.copy()
    a[0, L - 1, 2 * dh + 3] = np.inf
    got, plain = run(a), run(qkv)
    assert np.isposinf(got[:, 3]).all()
    rest = np.arange(dh) != 3
    assert np.array_equal(got[:, rest], plain[:, rest])
    for masked in (np.arange(0, 32), np.arange(0, L - 2), np.arange(L - 3, L)):
        b = qkv.copy()
        b[0, masked, dh] = -np.inf
        keep = np.setdiff1d(np.arange(L), masked)
        c = qkv.astype(np.float64)
        s = (c[0, :, :dh] @ c[0, keep, dh:2 * dh].T) / np.sqrt(dh)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        assert rel_l2(run(b), (p / p.sum(axis=1, keepdims=True)) @ c[0, keep, 2 * dh:]) < 2e-6, masked
    b = qkv.copy()
    b[0, :, dh] = -np.inf
    assert np.isnan(run(b)).all()


@pytest.mark.parametrize("prescaled", [0, 1])
@pytest.mark.parametrize("dh,L", [(64, 100), (64, 300), (128, 100), (128, 257)])
def test_attention_bf16_queries_without_a_result(lib, dh, L, prescaled):
    """A query that is not finite, or that a key scores +inf, has no result in its head; every other query keeps its own, also one
    whose row sums come out of the same matrix instruction, and the queries next to the last one, which fills the rows past the end."""
    rng = np.random.default_rng(dh + L)
    H, c = 2 * dh, np.log2(np.e) / np.sqrt(dh)
    qkv = rng.standard_normal((1, L, 3 * H)).astype(np.float32)
    if prescaled:
        qkv[..., :H] *= c
    qkv = _bf(qkv)

    def check(a, lost):
        out = torch.full((1, L, H), 3.0, dtype=torch.bfloat16, device=DEV)
        br.op_attention(br.BF16, dev(a, torch.bfloat16), out, 2, q_prescaled=prescaled)
        got = host(out)[0]
        x = a.astype(np.float64)
        x[0, lost, :dh] = 0.0                                        # (their own rows are not compared)
        if prescaled:
            x[..., :H] /= c
        s = x[0].reshape(L, 3, 2, dh).transpose(1, 2, 0, 3)
        with np.errstate(invalid="ignore"):
            sc = np.nan_to_num(s[0] @ s[1].transpose(0, 2, 1) / np.sqrt(dh), nan=0.0, neginf=-np.inf)
        p = np.exp(sc - sc.max(axis=2, keepdims=True))
        ref = (p / p.sum(axis=2, keepdims=True) @ s[2]).transpose(1, 0, 2).reshape(L, H)
        kept = np.setdiff1d(np.arange(L), lost)
        assert np.isnan(got[lost, :dh]).all(), lost
        assert rel_l2(got[kept, :dh], ref[kept, :dh]) < 3e-3, lost   # as in test_attention_bf16
        assert rel_l2(got[:, dh:], ref[:, dh:]) < 3e-3, lost

    for lost in ([3], [L - 1], [1, 17, 40], list(range(64, 80))):
        for bad in (np.nan, np.inf, -np.inf):
            a = qkv.copy()
            a[0, lost, 5] = bad
            check(a, np.array(lost))
    a = qkv.copy()                                                   # key 70 scores +inf or -inf, by the sign of the query
    a[0, 70, H + 5] = np.inf
    check(a, np.flatnonzero(a[0, :, 5] > 0))


# A query's reference comes from the first half tile of keys in which one scores above -inf: the first, one of the next, the last; in the kernel of short
# sequences, the one with a loop, whole tiles (of 256 queries at head dim 128 beyond 2048 tokens, else two workgroups a unit) and parts.
# The other keys score about -210, which a reference of zero would lose, in some heads and samples.
@pytest.mark.parametrize("prescaled", [0, 1])
@pytest.mark.parametrize("dh,L,leading", [(dh, L, n) for dh in (64, 128) for L, n in ((20, 7), (34, 32), (34, 33), (65, 64), (100, 31), (100, 32), (100, 33), (100, 63),
                                                                                      (190, 65), (300, 32), (300, 64), (300, 65), (333, 320), (470, 200), (2100, 70))])
def test_attention_bf16_leading_keys_that_score_minus_infinity(lib, dh, L, leading, prescaled):
    rng = np.random.default_rng(dh + L + leading)
    H, c = 2 * dh, np.log2(np.e) / np.sqrt(dh)
    qkv = rng.standard_normal((3, L, 3 * H)).astype(np.float32)
    qkv[..., 5:H:dh] = np.abs(qkv[..., 5:H:dh]) + 0.1        # by element 5 of every key of `leading`, whatever the query
    qkv[1, ..., 5:dh:dh] *= np.where(np.arange(L) % 3 == 0, -1, 1)[:, None]   # (sample 1, head 0: +inf for every third query)
    qkv[..., 6:H:dh], qkv[1:, :, H + 6:2 * H:dh] = 4.0, -52.5 * np.sqrt(dh)
    if prescaled:
        qkv[..., :H] *= c
    qkv = _bf(qkv)
    x = qkv.astype(np.float64)
    if prescaled:
        x[..., :H] /= c
    q, k, v = x.reshape(3, L, 3, 2, dh).transpose(2, 0, 3, 1, 4)
    s = q @ k.transpose(0, 1, 3, 2) / np.sqrt(dh)
    s[..., :leading] = -np.inf
    p = np.exp(s - s.max(axis=3, keepdims=True))
    ref = (p / p.sum(axis=3, keepdims=True) @ v).transpose(0, 2, 1, 3)
    lost = np.zeros((3, L, 2), bool)
    lost[1, ::3, 0] = True
    a = dev(qkv, torch.bfloat16)
    a[:, :leading, H + 5:2 * H:dh] = -np.inf
    n = -(-(2 * 256 * 256 + 1) // (2 * L))                   # samples of at least two rounds of whole tiles
    outs = []
    for rows in (torch.arange(3, device=DEV), torch.arange(n, device=DEV) % 3):
        out = torch.full((len(rows), L, H), 3.0, dtype=torch.bfloat16, device=DEV)
        br.op_attention(br.BF16, a[rows].contiguous(), out, 2, prescaled)
        outs.append(out)
    got = host(outs[0].float()).reshape(3, L, 2, dh)
    assert np.isnan(got[lost]).all() and np.isfinite(got[~lost]).all()
    assert rel_l2(got[~lost], ref[~lost]) < 8e-3             # probabilities and outputs rounded to bf16, 2^-9 each
    assert torch.equal(torch.nan_to_num(outs[1], nan=7.0), torch.nan_to_num(outs[0], nan=7.0)[torch.arange(n, device=DEV) % 3])


def test_attention_bf16_rows_far_apart(lib):
    """One token of 190 000 heads of 128: rows 29 to 31 of the first half of its tile of keys would lie 4 GiB and more from row 0 (modulo that, the values of
    row 29 are the query of the head 132 784 further).  The softmax of one key is 1, so the outputs are the values; queries that are not numbers
    reach their own heads alone."""
    nh, dh = 190000, 128
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    qkv = torch.randn((1, 1, 3 * nh * dh), generator=g, device=DEV).bfloat16()
    qkv[0, 0].view(3, nh, dh)[0, ::7] = float("nan")
    out = torch.full((1, 1, nh * dh), 3.0, dtype=torch.bfloat16, device=DEV)
    br.op_attention(br.BF16, qkv, out, nh)
    got, v = out.view(nh, dh), qkv[0, 0].view(3, nh, dh)[2]
    lost = torch.zeros(nh, dtype=torch.bool, device=DEV)
    lost[::7] = True
    assert bool(got[lost].isnan().all()) and torch.equal(got[~lost], v[~lost])


def test_gemm_bf16_rows_far_apart(lib):
    """192 rows of 832 values, 24 MB apart: the last rows of a tile are beyond 4 GiB from its first one.  Same bits as packed rows."""
    import ctypes as C
    M, N, K, lda = 192, 32768, 832, 12 << 20
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    A, W = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((M, K), (N, K)))
    b = torch.randn(N, generator=g, device=DEV)
    far = torch.empty((M, lda), dtype=torch.bfloat16, device=DEV)
    far[:, :K] = A
    ref, out = torch.empty((M, N), device=DEV), torch.empty((M, N), device=DEV)
    br.op_gemm(br.BF16, 4, A, W, b, ref)
    torch.cuda.synchronize()
    i = C.c_int32
    p = [C.c_void_p(t.data_ptr()) for t in (far, W, b, out)]
    assert br.load().br_op_gemm(i(br.BF16), i(4), p[0], i(lda), p[1], i(K), i(M), i(N), i(K), p[2], p[3], i(N), None, i(0), i(0), None, i(1), i(-1), None) == 0
    torch.cuda.synchronize()
    assert torch.equal(out, ref)


@pytest.mark.parametrize("M,N,K,kernel", [(1638, 2048, 256, 3), (1400, 2304, 576, 3), (4424, 192, 1536, 2), (32424, 96, 384, 3), (8831, 640, 192, 1),  # not the ring
                                           (4404, 512, 512, 6), (2202, 2048, 512, 6), (1101, 3072, 1024, 6), (4404, 1024, 4096, 6)])
def test_gemm_bf16_ring_where_it_is_the_faster_one(lib, M, N, K, kernel):
    """The choice on 256 compute units: a short K stays with the tiles that come two to a unit unless they are a little more than a
    round."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sizes are for 256 compute units")
    A, W = (torch.zeros(s, dtype=torch.bfloat16, device=DEV) for s in ((M, K), (N, K)))
    out = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    br.profile_enable(True)
    try:
        br.op_gemm(br.BF16, 0, A, W, torch.zeros(N, device=DEV), out)
        torch.cuda.synchronize()
        ids = br.profile_read()
    finally:
        br.profile_enable(False)
    assert list(ids) == [kernel]


def test_gemm_variant_word(lib):
    """Heights of the persistent kernel are kernel numbers of their own; what callers pass as start delays (bits 12..23) stays
    accepted and changes nothing; numbers beyond are refused."""
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    M, N, K = 700, 512, 256
    A, W = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((M, K), (N, K)))
    b = torch.randn(N, generator=g, device=DEV)
    ref = torch.empty((M, N), device=DEV)
    br.op_gemm(br.BF16, 4, A, W, b, ref, variant=5)
    for variant in [7, 8, 9, 10, 11] + [v | (d << 12) for v in (7, 9) for d in (4, 6, 255, 4095)]:
        out = torch.empty((M, N), device=DEV)
        br.op_gemm(br.BF16, 4, A, W, b, out, variant=variant)
        assert torch.equal(out, ref), variant
    for variant in (12, 13, 14, 15):
        with pytest.raises(br.BranchRolloutError) as e:
            br.op_gemm(br.BF16, 4, A, W, b, ref, variant=variant)
        assert e.value.code == -1


@pytest.mark.parametrize("M,N,K,mode", [(4404, 1024, 1024, 1), (1101, 3072, 1024, 0), (1101, 1024, 4096, 2), (6144, 768, 192, 1), (599, 768, 768, 1)])
def test_gemm_fp32_automatic_choice_of_every_form(lib, M, N, K, mode):
    """Shapes that the size rule gives to the ring kernel (the last one: to 32x32 tiles), against the other kernel (32x32 tiles, or a ring tile) bit for bit,
    and right against fp64."""
    rng = np.random.default_rng(N + M)
    A, W, b, x0 = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (N, K), (N,), (M, N)))
    mods, cond = rng.standard_normal((1, N)).astype(np.float32), np.zeros(1, np.int32)
    outs = []
    for variant in (-1, 0, 6 | (5 << 24) | 16):
        out = dev(x0.copy())
        br.op_gemm(br.F32, mode, dev(A), dev(W), dev(b), out, mods=dev(mods) if mode == 2 else None, cond=dev(cond) if mode == 2 else None, L=M, variant=variant)
        outs.append(out)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    rows = np.r_[0:3, 63:66, 127:130, M - 130:M - 126, M - 3:M]
    ref = A[rows].astype(np.float64) @ W.astype(np.float64).T + b
    # fp32 sums of K products: about sqrt(K) 2^-24 of the norm
    assert rel_l2(host(outs[0])[rows], dit.gelu_tanh(ref) if mode == 1 else x0[rows] + mods * ref if mode == 2 else ref) < 3e-6


@pytest.mark.parametrize("height", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("M,N,K,L", [(37 * 1101, 1024, 128, 1101), (438 * 93, 1020, 384, 93), (2037 * 20, 1024, 256, 20)])
def test_gemm_persistent_tiles_after_the_first(lib, height, M, N, K, L):
    """Every workgroup takes two to five tiles: the operand stream crosses tile boundaries, the next tile's first stages are
    waited for with the epilogue's stores in flight.  Every element of every output form against the 128x128 kernel, which has one
    tile per workgroup, bit for bit; samples longer and shorter than a wave's rows."""
    g = torch.Generator(device=DEV)
    g.manual_seed(height + K)
    A, W = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((M, K), (N, K)))
    b, x0 = torch.randn(N, generator=g, device=DEV), torch.randn((M, N), generator=g, device=DEV)
    mods = torch.randn((7, N), generator=g, device=DEV)
    cond = (torch.arange(M // L, device=DEV) % 7).int()
    for mode, dt in ((4, torch.float32), (0, torch.bfloat16), (1, torch.bfloat16), (2, torch.float32)):
        outs = []
        for variant in (STREAM[height], 5):
            out = x0.clone() if mode == 2 else torch.full((M, N), -9.0, dtype=dt, device=DEV)
            br.op_gemm(br.BF16, mode, A, W, b, out, mods=mods if mode == 2 else None, cond=cond if mode == 2 else None, L=L, variant=variant)
            outs.append(out)
        assert torch.equal(outs[0], outs[1]), (mode, height)


def test_profile_lists_gemms_of_bf16_networks_only(lib):
    """Ids 0..47 are bf16 GEMMs (epilogue * 8 + kernel); an fp32 network has none, whether or not its small GEMMs normalise
    their rows themselves."""
    for dtype, expect in ((synth.F32, False), (synth.BF16, True)):
        cfg = synth.model_cfg(1, 64, 1, (16, 1, 8, 8), (1, 2, 2), 5, dtype)
        br.profile_enable(True)
        try:
            _velocity_case(cfg, 1, 2, 0.5, 1)
            torch.cuda.synchronize()
            ids = br.profile_read()
        finally:
            br.profile_enable(False)
        assert any(i < 48 for i in ids) == expect, ids


# 128-column tiles of 32 to 192 rows with a ring of four to seven stages: one stage, fewer than a ring holds, more; one row, ragged rows and
# columns, samples shorter and longer than a wave's rows.  Same bits as the 32x32 tiles, nothing past the end.
@pytest.mark.parametrize("height", [2, 4, 6, 8, 10, 12])
@pytest.mark.parametrize("M,N,K,L", [(1, 4, 64, 1), (160, 128, 128, 160), (161, 132, 320, 7), (333, 260, 448, 111), (480, 384, 1088, 240)])
def test_gemm_bf16_ring_tiles(lib, height, M, N, K, L):
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)
    A, W = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((M, K), (N, K)))
    b, mods, x0 = (torch.randn(s, generator=g, device=DEV) for s in ((N,), (3, N), (M + 1, N)))
    cond = torch.arange(M // L, device=DEV, dtype=torch.int32) % 3
    for mode in (0, 1, 2, 4):
        outs = []
        for variant in (0, 6 | (height << 24)):
            out = x0.clone() if mode in (2, 4) else x0.bfloat16()
            br.op_gemm(br.BF16, mode, A, W, b, out[:M], mods=mods if mode == 2 else None, cond=cond if mode == 2 else None, L=L, variant=variant)
            outs.append(out)
        assert torch.equal(outs[0], outs[1]), mode
        assert torch.equal(outs[1][M], x0[M].to(outs[1].dtype))


# fp32 tiles of 16 h rows x 64 or 128 columns: one stage of 32 k, two (both slots), an odd and an even number more; one row, ragged rows and
# columns, samples shorter and longer than a tile.  Same bits as the 32x32 tiles, nothing past the end.
@pytest.mark.parametrize("height", range(2, 13))
@pytest.mark.parametrize("M,N,K,L", [(1, 4, 32, 1), (160, 128, 64, 160), (203, 132, 160, 7), (390, 260, 96, 195), (577, 384, 1056, 577)])
def test_gemm_fp32_ring_tiles(lib, height, M, N, K, L):
    g = torch.Generator(device=DEV)
    g.manual_seed(M + K)
    A, W, b, mods, x0 = (torch.randn(s, generator=g, device=DEV) for s in ((M, K), (N, K), (N,), (3, N), (M + 1, N)))
    cond = torch.arange(M // L, device=DEV, dtype=torch.int32) % 3
    for mode in (0, 1, 2):
        outs = []
        for variant in (0, 6 | (height << 24), 6 | (height << 24) | 16):
            out = x0.clone()
            br.op_gemm(br.F32, mode, A, W, b, out[:M], mods=mods if mode == 2 else None, cond=cond if mode == 2 else None, L=L, variant=variant)
            outs.append(out)
        assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]), mode
        assert torch.equal(outs[0][M], x0[M])


# Head dim 64: three samples, whose tiles are cut in two, and nine workgroups a compute unit, whole.  One to seven tiles of keys (up to two in the kernel of short
# sequences; three fill the buffers of keys and of values, from the fourth on they are refilled), last tiles of 1, 32, 33 and 64 keys; a
# reference that moves mid-sequence in some queries; waves without queries.  The same bits.
@pytest.mark.parametrize("prescaled", [0, 1])
@pytest.mark.parametrize("L", [1, 32, 33, 64, 65, 96, 128, 161, 192, 224, 256, 257, 300, 352, 384, 417])
def test_attention_bf16_head_dim_64_does_not_depend_on_the_kernel(lib, L, prescaled):
    nh, n = 2, 9 * 256 // (2 * ((L + 127) // 128)) + 1     # nine workgroups a compute unit
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    qkv = torch.randn((3, L, 3 * nh * 64), generator=g, device=DEV)
    qkv[1, L // 2:, nh * 64:2 * nh * 64] *= 12.0           # later keys score far above the first tiles'
    qkv = qkv.bfloat16()
    few, many = torch.empty((3, L, nh * 64), device=DEV).bfloat16(), torch.empty((n, L, nh * 64), device=DEV).bfloat16()
    br.op_attention(br.BF16, qkv, few, nh, prescaled)
    br.op_attention(br.BF16, qkv[torch.arange(n, device=DEV) % 3].contiguous(), many, nh, prescaled)
    assert torch.equal(many, few[torch.arange(n, device=DEV) % 3])
    q, k, v = (t.float().reshape(3, L, nh, 64).transpose(1, 2).double().cpu() for t in qkv.split(nh * 64, dim=2))
    s = (q @ k.transpose(2, 3).contiguous()) * (0.6931471805599453 if prescaled else 0.125)
    ref = (torch.softmax(s, dim=3) @ v).transpose(1, 2).reshape(3, L, nh * 64)
    assert rel_l2(host(few.float()), ref.numpy()) < 8e-3   # probabilities and outputs rounded to bf16, 2^-9 each


# Tiles whole, in two and in four parts, and the kernel of short sequences, which is left at 193 tokens (128; with more tiles, at 129) and 129 (64): tiles of keys up to
# the fifth, where the four or three buffers have been refilled; whole rounds of 256 queries in front of parts, which head dim 128 has beyond 2048 tokens;
# last tiles of 1, 31, 32, 33 and 64 keys; parts without queries; a reference that moves mid-sequence.
@pytest.mark.parametrize("prescaled", [0, 1])
@pytest.mark.parametrize("dh,L", [(128, L) for L in (1, 31, 64, 65, 128, 129, 191, 192, 193, 224, 225, 255, 256, 257, 320, 321, 449, 577, 2081, 2304)] + [(64, 129), (64, 160), (64, 193)])
def test_attention_bf16_does_not_depend_on_the_parts(lib, dh, L, prescaled):
    nh, rows = 2, 128 if dh == 64 or L <= 192 else 256
    tiles = nh * ((L + rows - 1) // rows)                   # of a sample
    # a part of a round (in four parts at head dim 128), a third (in two; 128: two workgroups a unit), and full rounds behind which few are left
    counts = [3, -(-90 // tiles), -(-(3 * 256 + 8) // tiles)]
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    qkv = torch.randn((3, L, 3 * nh * dh), generator=g, device=DEV)
    qkv[1, L // 2:, nh * dh:2 * nh * dh] *= 12.0            # later keys score far above the first tiles'
    qkv = qkv.bfloat16()
    outs = []
    for n in counts:
        out = torch.full((n + 1, L, nh * dh), 3.0, device=DEV).bfloat16()
        br.op_attention(br.BF16, qkv[torch.arange(n, device=DEV) % 3].contiguous(), out[:n], nh, prescaled)
        assert bool((out[n] == 3.0).all())
        outs.append(out[:n])
    for n, out in zip(counts, outs):
        assert torch.equal(out, outs[0][torch.arange(n, device=DEV) % 3]), n
    q, k, v = (t.float().reshape(3, L, nh, dh).transpose(1, 2).double().cpu() for t in qkv.split(nh * dh, dim=2))
    s = (q @ k.transpose(2, 3).contiguous()) * (0.6931471805599453 if prescaled else dh ** -0.5)
    ref = (torch.softmax(s, dim=3) @ v).transpose(1, 2).reshape(3, L, nh * dh)
    assert rel_l2(host(outs[0].float()), ref.numpy()) < 8e-3   # probabilities and outputs rounded to bf16, 2^-9 each


# Head dim 128 has tiles of 128 queries, two workgroups a compute unit with two buffers of keys and of values, beside those of 256: few samples (in parts), three quarters
# of a workgroup a unit (128), just under a round of 256, just above one and three (128; 256 and a cut last round beyond 2048 tokens).  Two to five tiles of keys and
# long loops, which end in either buffer; last tiles of 1, 31, 32, 33 and 64 keys; waves without queries; a reference that moves mid-sequence.  The same bits.
@pytest.mark.parametrize("prescaled", [0, 1])
@pytest.mark.parametrize("L", [129, 160, 161, 192, 193, 223, 224, 225, 256, 257, 320, 449, 577, 1101, 4095, 4097])
def test_attention_bf16_head_dim_128_does_not_depend_on_the_form(lib, L, prescaled):
    nh, dh = 2, 128
    t128, t256 = nh * ((L + 127) // 128), nh * ((L + 255) // 256)           # tiles of a sample
    counts = [3] + [max(3, n) for n in (192 // t128, 256 // t256, 256 // t256 + 9, 3 * 256 // t256 + 9)]
    g = torch.Generator(device=DEV)
    g.manual_seed(L)
    qkv = torch.randn((3, L, 3 * nh * dh), generator=g, device=DEV)
    qkv[1, L // 2:, nh * dh:2 * nh * dh] *= 12.0            # later keys score far above the first tiles'
    qkv = qkv.bfloat16()
    first = None
    for n in counts:
        which = torch.arange(n, device=DEV) % 3
        out = torch.full((n + 1, L, nh * dh), 3.0, device=DEV).bfloat16()
        br.op_attention(br.BF16, qkv[which].contiguous(), out[:n], nh, prescaled)
        assert bool((out[n] == 3.0).all()), n
        first = out[:3] if first is None else first
        assert torch.equal(out[:n], first[which]), n
    q, k, v = (t.float().reshape(3, L, nh, dh).transpose(1, 2) for t in qkv.split(nh * dh, dim=2))
    s = torch.matmul(q, k.transpose(2, 3).contiguous()) * (0.6931471805599453 if prescaled else dh ** -0.5)   # (fp32: 1e-6 of the sum)
    ref = torch.matmul(torch.softmax(s, dim=3), v).transpose(1, 2).reshape(3, L, nh * dh)
    assert rel_l2(host(first.float()), host(ref)) < 8e-3   # probabilities and outputs rounded to bf16, 2^-9 each


# Outputs of 32 to 112 MB, with GELU 100, are stored plainly by the persistent kernel at this K, smaller and larger ones past the caches: below, at and
# above the lines, full and ragged tiles, against the 128x128 kernel, bit for bit (which stores plainly up to 160 MB).
@pytest.mark.parametrize("M,N", [(8191, 2048), (8192, 2048), (8200, 2060), (24414, 2048), (24415, 2048), (27343, 2048), (27344, 2048), (40960, 2048), (40961, 2048)])
def test_gemm_persistent_outputs_that_stay_in_the_caches(lib, M, N):
    g = torch.Generator(device=DEV)
    g.manual_seed(M)
    A, W = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((M, 128), (N, 128)))
    b = torch.randn(N, generator=g, device=DEV)
    for mode in (0, 1):
        outs = []
        for variant in (STREAM[7], 5):
            out = torch.full((M + 1, N), -9.0, device=DEV).bfloat16()
            br.op_gemm(br.BF16, mode, A, W, b, out[:M], variant=variant)
            outs.append(out)
        assert torch.equal(outs[0], outs[1]), mode


# Outputs above 160 MB go past the caches in the kernels of 128x128 and 256x256 tiles: at and above the line, full and ragged tiles, against the
# 64x64 kernel, whose stores are always plain, bit for bit; and nothing past the end.
@pytest.mark.parametrize("variant", [1, 4, 5])
@pytest.mark.parametrize("M,N", [(40960, 2048), (40961, 2048), (40963, 2060)])
def test_gemm_tile_outputs_past_the_caches(lib, variant, M, N):
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N)
    A, W = (torch.randn(s, generator=g, device=DEV).bfloat16() for s in ((M, 64), (N, 64)))
    b = torch.randn(N, generator=g, device=DEV)
    for mode in (0, 1):
        outs = []
        for v in (variant, 2):
            out = torch.full((M + 1, N), -9.0, device=DEV).bfloat16()
            br.op_gemm(br.BF16, mode, A, W, b, out[:M], variant=v)
            outs.append(out)
        assert torch.equal(outs[0], outs[1]), mode


# Up to 192 tokens an attention that reads weights ahead has all its keys under way at once, beyond it has a loop over four buffers: 72, 139, 193, 257, 321 and 389
# tokens; last tiles of keys of 1 and 5, which come into each of the buffers; waves of 16 queries without any; heads of 64 (grouped by die) and 128 (dealt out in order).
@pytest.mark.parametrize("heads,lat_h,lat_w", [(32, 14, 18), (16, 20, 26)] + [(h, *hw) for h in (32, 16) for hw in ((16, 46), (16, 62), (24, 52), (38, 40))])
def test_velocity_where_attention_leaves_units_to_the_weights(lib, heads, lat_h, lat_w):
    """Networks too large for the memory-side cache read the next weights in front of an attention that leaves compute units idle (one
    sample: 16 to 128 workgroups), and not where it does not (eighteen): the same bits, right against the oracle."""
    cfg = synth.model_cfg(3, 2048, heads, (16, 1, lat_h, lat_w), (1, 2, 2), 9, synth.BF16)
    W = synth.make_weights(cfg, 3, 0.03)
    model = make_model(cfg, W)
    D = synth.model_sizes(cfg)["D"]
    z, tok = synth.random_latents(1, D, 4), synth.cond_tokens(cfg, 1, 5)
    out = []
    for n in (1, 18):
        v = torch.empty((n, D), device=DEV)
        br.velocity(model, dev(z).repeat(n, 1), 0.4, cond_dev(cfg, tok), np.zeros(n, np.int32), v, bytes_buffer(br.workspace_bytes(None, model, n)))
        out.append(v)
    assert torch.equal(out[1], out[0].expand(18, -1))
    assert_velocity(cfg, host(out[0])[0], dit.forward(cfg, W, z, 0.4, tok, np.zeros(1, np.int32))[0], 2e-2)
