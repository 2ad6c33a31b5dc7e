"""Performance cases of the tree-rollout library: what its callers run, through the entry points of
`paper_2509_06040_amd.binding`, from calls that only cost launches to the largest frontiers.

A case is a dict of plain values.  `kind` names what one pass calls:
  velocity  br_velocity: the network on a batch of latents (the core of every rollout; also called by itself)
  rollout   br_rollout: root noise, one network batch per depth, SDE step into the children
  logprob   br_logprob: kept edges re-evaluated under updated weights (Extreme-b selection, 4 of T depths dropped)
  sde       br_sde_step: one step of a frontier with a velocity that the caller computed
  post      what follows a rollout: leaf rewards, fusion and advantages, pruning, and the read-back of the kept edges
  step      a whole policy iteration: rollout, post, logprob on the kept edges, clipped objective
The network is `blocks, heads, head_dim, lat_c/t/h/w, patch 1x2x2 (pt x 2 x 2), cond tokens, dtype`.
"""
import math

import numpy as np
import torch

from paper_2509_06040_amd import binding as br
from paper_2509_06040_amd import synth

DEV = "cuda"
DTYPES = {"f32": synth.F32, "bf16": synth.BF16}


def _net(blocks, heads, head_dim, lat, cond, dtype, pt=1):
    c, t, h, w = lat
    return dict(blocks=blocks, heads=heads, head_dim=head_dim, lat_c=c, lat_t=t, lat_h=h, lat_w=w, pt=pt, cond=cond,
                dtype=dtype)


def _tree(T, splits, K, n_tree, kappa=3.0):
    return dict(T=T, splits=",".join(str(s) for s in splits), K=K, n_tree=n_tree, kappa=kappa)


_TINY = _net(2, 4, 16, (4, 1, 8, 8), 8, "f32")
_IMAGE = _net(12, 16, 64, (16, 1, 64, 64), 77, "bf16")
_LARGE = _net(24, 24, 128, (16, 1, 128, 128), 512, "bf16")
_VIDEO = _net(30, 12, 128, (16, 21, 60, 104), 512, "bf16")


def listed():
    return [
        # the fp32 reference workload: every call is a few kilobytes, so latency and launch count are all there is
        dict(name="tiny_step", kind="step", **_TINY, **_tree(8, (2, 4, 6), 2, 1, 1.0), reward="linear"),
        # a small bf16 network with ragged token counts (L = 93): quick experiments
        dict(name="small_velocity", kind="velocity", **_net(2, 2, 64, (16, 1, 16, 20), 13, "bf16"), B=3),
        # one image sample: the root of a single prompt's tree, sampling for inspection
        dict(name="image_velocity_1", kind="velocity", **_IMAGE, B=1),
        # the image workload's rollout: 4 prompts x 16 leaves, frontiers of 4 to 64 samples
        dict(name="image_rollout", kind="rollout", **_IMAGE, **_tree(20, (4, 8, 12, 16), 2, 4)),
        # its log-prob re-evaluation: ragged batches that mix steps
        dict(name="image_logprob", kind="logprob", **_IMAGE, **_tree(20, (4, 8, 12, 16), 2, 4)),
        # the same network in fp32 (numerical checks of a run), one sample per prompt
        dict(name="image_velocity_f32", kind="velocity", **{**_IMAGE, "dtype": "f32"}, B=4),
        # the large-image network: the narrowest frontier of a 2-prompt rollout, and the widest
        dict(name="large_velocity_2", kind="velocity", **_LARGE, B=2),
        dict(name="large_velocity_32", kind="velocity", **_LARGE, B=32),
        # video: one sample of 33 272 tokens with full attention
        dict(name="video_velocity_1", kind="velocity", **_VIDEO, B=1),
        # the split step of the video tree (4 parents, 8 children of 2.1 million elements)
        dict(name="video_sde_split", kind="sde", D=2096640, step=12, **_tree(16, (4, 8, 12), 2, 1)),
        # after the rollout: image rewards and tree; video rewards (plane means) over the largest leaves
        dict(name="image_post", kind="post", lat_c=16, lat_t=1, lat_h=64, lat_w=64, reward="tanh",
             **_tree(20, (4, 8, 12, 16), 2, 4)),
        dict(name="video_post", kind="post", lat_c=16, lat_t=21, lat_h=60, lat_w=104, reward="video",
             **_tree(16, (4, 8, 12), 2, 1)),
    ]


# ------------------------------------------------------------------------------------------ draws
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_tree(rng, max_leaves, max_T, n_tree):
    T = rng.randint(3, max_T)
    K = rng.choice((2, 2, 2, 3, 4))
    n = rng.randint(1, max(1, min(T, int(math.log(max_leaves) / math.log(K) + 1e-9))))
    return _tree(T, sorted(rng.sample(range(T), n)), K, n_tree, rng.choice((1.0, 3.0)))


def _draw_net(rng, dtype):
    head_dim = rng.choice((64, 128)) if dtype == "bf16" else rng.choice((16, 32, 64, 128))
    top = 3072 if dtype == "bf16" else 1024
    heads = max(1, _log_int(rng, 64, top) // head_dim)
    video = rng.random() < 0.2
    lat = (16 if dtype == "bf16" else rng.choice((4, 16)), rng.randint(2, 21) if video else 1,
           2 * _log_int(rng, 4, 64), 2 * _log_int(rng, 4, 64))
    return _net(rng.randint(1, 24), heads, head_dim, lat, _log_int(rng, 5, 512), dtype)


def draw(rng):
    """Another case of the listed ones' ranges."""
    kind = rng.choice(("velocity",) * 4 + ("velocity_f32",) * 2 + ("rollout", "logprob", "sde", "post", "step"))
    if kind in ("sde", "post"):
        tree = _draw_tree(rng, 64, 28, rng.randint(1, 4))
        lat = dict(lat_c=16, lat_t=rng.choice((1, 1, rng.randint(2, 21))), lat_h=2 * _log_int(rng, 4, 64),
                   lat_w=2 * _log_int(rng, 4, 64))
        D = lat["lat_c"] * lat["lat_t"] * lat["lat_h"] * lat["lat_w"]
        nodes = _shape(tree)
        while tree["n_tree"] * nodes["n_nodes"] * D > 1.5e9:   # (a 6 GB arena)
            lat["lat_h"] = lat["lat_w"] = 8
            D = lat["lat_c"] * lat["lat_t"] * 64
        if kind == "sde":
            return dict(kind="sde", D=D, step=rng.randrange(tree["T"]), **tree)
        return dict(kind="post", reward="video" if lat["lat_t"] > 1 else rng.choice(("linear", "tanh")), **lat, **tree)
    f32 = kind in ("velocity_f32", "step")
    # flops of a pass: log-uniform up to a third of the largest listed case (fp32: up to a large fp32 batch)
    low, high = (1e6, 5e12) if f32 else (1e8, 3e14)
    goal = math.exp(rng.uniform(math.log(low), math.log(high)))
    best, best_off = None, math.inf
    for _ in range(400):
        case = dict(kind="velocity" if kind == "velocity_f32" else kind, **_draw_net(rng, "f32" if f32 else "bf16"))
        if case["kind"] == "velocity":
            case["B"] = _log_int(rng, 1, 64)
        else:
            case.update(_draw_tree(rng, 16, 20, rng.randint(1, 4)))
            if kind == "step":
                case["reward"] = rng.choice(("linear", "tanh"))
        off = abs(math.log(work(case)["flops"] / goal))
        if off < best_off and _state_bytes(case) < 40e9:
            best, best_off = case, off
        if best_off < 0.3:
            break
    return best


# ------------------------------------------------------------------------------------------ shapes
def _splits(case):
    return [int(s) for s in case["splits"].split(",") if s]


def _shape(case):
    width = [1]
    for i in range(case["T"]):
        width.append(width[-1] * (case["K"] if i in _splits(case) else 1))
    return dict(width=width, n_nodes=sum(width), n_leaves=width[-1], frontier=max(width[:-1]))


def _cfg(case):
    return synth.model_cfg(case["blocks"], case["heads"] * case["head_dim"], case["heads"],
                           (case["lat_c"], case["lat_t"], case["lat_h"], case["lat_w"]), (case["pt"], 2, 2),
                           case["cond"], DTYPES[case["dtype"]])


def _net_flops(cfg):
    s = synth.model_sizes(cfg)
    H, L = cfg["hidden"], s["L"]
    return cfg["n_blocks"] * (24.0 * L * H * H + 4.0 * L * L * H) + 4.0 * s["n_img"] * s["patch_dim"] * H


def _weight_bytes(cfg):
    e = 2 if cfg["dtype"] == synth.BF16 else 4
    return sum(math.prod(shape) * (e if mat else 4) for _, shape, mat in synth.weight_shapes(cfg))


def _state_bytes(case):
    cfg = _cfg(case)
    s = synth.model_sizes(cfg)
    B = case["B"] if "B" in case else case["n_tree"] * _shape(case)["frontier"]
    rows = B if "B" in case else case["n_tree"] * _shape(case)["n_nodes"]
    return 2 * _weight_bytes(cfg) + B * s["L"] * cfg["hidden"] * 40.0 + rows * s["D"] * 8.0


def _pick_edges(tree, case, rewards):
    """Extreme-b selection of a quarter of the leaves from each end, four of every T = 16 depths dropped."""
    mask = br.depth_mask_seeded(case["T"], case["T"] // 4, synth.DATA_SEED)
    kept = torch.empty(tree.n_tree * tree.n_edges, dtype=torch.int32, device=DEV)
    nk = torch.zeros(1, dtype=torch.int32, device=DEV)
    br.prune(tree, rewards, br.PRUNE_EXTREME, max(1, tree.n_leaves // 4), mask, kept, nk)
    return kept[:int(nk)].cpu().numpy()


def _kept_counts(case):
    """(network evaluations, edges) of the kept set: Parent-Top1 for `step` (a fixed count), about half of
    the leaves for `logprob`."""
    sh = _shape(case)
    mask = br.depth_mask_seeded(case["T"], case["T"] // 4, synth.DATA_SEED)
    leaves = sh["n_leaves"] // case["K"] if case["kind"] == "step" else 2 * max(1, sh["n_leaves"] // 4)
    live = [i for i in range(case["T"]) if not mask[i]]
    evals = sum(min(sh["width"][i], leaves) for i in live)
    edges = sum(min(sh["width"][i + 1], leaves) for i in live)
    return case["n_tree"] * evals, case["n_tree"] * edges


def work(case):
    kind = case["kind"]
    if kind in ("sde", "post"):
        sh = _shape(case)
        n_tree = case["n_tree"]
        if kind == "sde":  # parents' latent and velocity read, children written; about 60 operations a normal
            p, c = n_tree * sh["width"][case["step"]], n_tree * sh["width"][case["step"] + 1]
            return {"bytes": 4.0 * case["D"] * (2 * p + c), "flops": 60.0 * case["D"] * c}
        D = case["lat_c"] * case["lat_t"] * case["lat_h"] * case["lat_w"]
        return {"bytes": 4.0 * (n_tree * sh["n_leaves"] * D + n_tree * sh["n_nodes"] * 4),
                "flops": 2.0 * n_tree * sh["n_leaves"] * D}
    cfg = _cfg(case)
    s = synth.model_sizes(cfg)
    f, wb, D4 = _net_flops(cfg), _weight_bytes(cfg), 4.0 * s["D"]
    if kind == "velocity":
        return {"bytes": wb + 2 * case["B"] * D4, "flops": f * case["B"]}
    sh = _shape(case)
    evals = case["n_tree"] * sum(sh["width"][:-1])
    arena = case["n_tree"] * sh["n_nodes"] * D4
    if kind == "rollout":
        return {"bytes": wb + arena, "flops": f * evals}
    again, edges = _kept_counts(case)
    if kind == "logprob":
        return {"bytes": wb + (again + edges) * D4, "flops": f * again}
    return {"bytes": 2 * wb + 2 * arena, "flops": f * (evals + again)}


def tolerance(case):
    """About four times what was measured: fp32 networks against the same network in fp64 (7e-7, largest
    element 9e-6 of the rms), bf16 ones against fp64 arithmetic on the same weights (1.7e-3 to 2.6e-3,
    largest element 1.2e-2), bf16 log-probs against those of the fp32 network (7e-6 at D = 65536; a mean
    over fewer elements averages less)."""
    kind = case["kind"]
    if kind in ("sde", "post"):
        return {"rel": 5e-6, "max": 1e-4}
    if kind == "step":      # advantages divide differences of fused rewards by their spread
        return {"rel": 2e-5, "max": 2e-3}
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4}
    if kind == "logprob":
        return {"rel": 2e-4, "max": 2e-3}
    if kind == "rollout":   # the velocity errors, weighted by the step sizes, on latents of rms about 1
        return {"rel": 4e-3, "max": 5e-2}
    return {"rel": 1e-2, "max": 5e-2}


# ------------------------------------------------------------------------------------------ states
def _randn(shape, g, std=1.0):
    return torch.randn(shape, generator=g, device=DEV) * std


def _weights(cfg, g):
    mat = torch.bfloat16 if cfg["dtype"] == synth.BF16 else torch.float32
    W = {}
    for name, shape, is_mat in synth.weight_shapes(cfg):
        if name == "pos":  # the sine-cosine table of synth.positional_table
            n, H = shape
            k = torch.arange(H // 2, device=DEV, dtype=torch.float64)
            ang = torch.arange(n, device=DEV, dtype=torch.float64)[:, None] / 10000.0 ** (2.0 * k / H)
            W[name] = torch.stack((ang.sin(), ang.cos()), dim=2).reshape(n, H).float()
        else:
            w = _randn(shape, g, 0.02)
            W[name] = w.to(mat) if is_mat else w
    return W


def _cond(cfg, n, g):
    return _randn((n, cfg["n_cond_tokens"], cfg["cond_dim"]), g).to(
        torch.bfloat16 if cfg["dtype"] == synth.BF16 else torch.float32)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _model(cfg, g, extra=None):
    W = _weights(cfg, g)
    model = br.Model(cfg, W)
    if extra is None:
        return model, None
    return model, br.Model(cfg, synth.device_perturb_weights(cfg, W, extra, 0.002, DEV))


def _post_buffers(st, case, tree, latent):
    n = tree.n_tree * tree.n_nodes
    st.update(latent=latent, kind_r={"linear": br.REWARD_LINEAR, "tanh": br.REWARD_TANH, "video": br.REWARD_VIDEO}[case["reward"]],
              rewards=torch.empty(tree.n_tree * tree.n_leaves, device=DEV), rbar=torch.empty(n, device=DEV),
              adv=torch.empty(n, device=DEV), kept=torch.empty(tree.n_tree * tree.n_edges, dtype=torch.int32, device=DEV),
              n_kept=torch.zeros(1, dtype=torch.int32, device=DEV),
              mask=br.depth_mask_seeded(case["T"], case["T"] // 4, synth.DATA_SEED))
    st["reward_scratch"] = _bytes(br.reward_scratch_bytes(tree, st["kind_r"], latent))


def prepare(case, seed):
    kind = case["kind"]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    st = dict(case=case, seed=seed)
    if kind == "velocity":
        cfg, B = _cfg(case), case["B"]
        n_cond = min(B, 4)
        st["model"], _ = _model(cfg, g)
        D = synth.model_sizes(cfg)["D"]
        st.update(z=_randn((B, D), g), cond=_cond(cfg, n_cond, g), index=np.arange(B, dtype=np.int32) % n_cond,
                  t=0.05 + 0.9 * float(torch.rand(1, generator=g, device=DEV)), v=torch.empty((B, D), device=DEV),
                  ws=_bytes(br.workspace_bytes(None, st["model"], B)))
        return st
    tree = br.Tree(case["T"], _splits(case), case["K"], n_tree=case["n_tree"]).upload()
    sched = synth.schedule(case["T"], case["kappa"])
    n = tree.n_tree * tree.n_nodes
    st.update(tree=tree, sched=sched, groups=list(range(tree.n_tree)), logp=torch.zeros(n, device=DEV))
    if kind == "sde":
        D, width = case["D"], tree.n_tree * int(tree.width[case["step"]])
        st.update(v=_randn((width, D), g), z=torch.zeros((n, D), device=DEV), scratch=_bytes(br.sde_scratch_bytes(tree, D)))
        rows = _rows(tree, case["step"])
        st["z"][rows] = _randn((len(rows), D), g)
        return st
    if kind == "post":
        latent = tuple(case["lat_" + a] for a in "cthw")
        D = math.prod(latent)
        st.update(z=torch.zeros((n, D), device=DEV), w=_randn((latent[0] * latent[1] if case["reward"] == "video" else D,), g))
        st["z"][_rows(tree, tree.T)] = _randn((tree.n_tree * tree.n_leaves, D), g)
        st["logp"] = 1.2 + _randn((n,), g, 0.02)
        _post_buffers(st, case, tree, latent)
        return st
    cfg = _cfg(case)
    D = synth.model_sizes(cfg)["D"]
    st["model"], st["model2"] = _model(cfg, g, None if kind == "rollout" else seed + 1)
    st.update(cond=_cond(cfg, tree.n_tree, g), z=torch.zeros((n, D), device=DEV),
              ws=_bytes(br.workspace_bytes(tree, st["model"], tree.n_tree * _shape(case)["frontier"])))
    if kind == "logprob":  # transitions of a rollout whose velocities are of the network's magnitude
        scratch = _bytes(br.sde_scratch_bytes(tree, D))
        br.root_noise(tree, seed, st["groups"], D, st["z"])
        for i in range(tree.T):
            br.sde_step(tree, sched, seed, i, D, _randn((tree.n_tree * int(tree.width[i]), D), g, 0.6), st["z"], st["logp"], scratch)
        st["ids"] = _pick_edges(tree, case, _randn((tree.n_tree * tree.n_leaves,), g))
        st["out"] = torch.zeros(tree.n_tree * tree.n_edges, device=DEV)
    elif kind == "step":
        st["w"] = _randn((D,), g)
        _post_buffers(st, case, tree, tuple(case["lat_" + a] for a in "cthw"))
        st["logp_new"] = torch.empty(tree.n_tree * tree.n_edges, device=DEV)
        st["J"] = torch.empty(1, device=DEV)
    return st


def _rows(tree, depth):
    lo, hi = int(tree.off[depth]), int(tree.off[depth + 1])
    return torch.cat([torch.arange(c * tree.n_nodes + lo, c * tree.n_nodes + hi, device=DEV) for c in range(tree.n_tree)])


# ------------------------------------------------------------------------------------------ passes
def _post(st):
    tree = st["tree"]
    br.leaf_reward(tree, st["z"], st["kind_r"], st["w"], 0.1, st["latent"], st["rewards"], st["reward_scratch"])
    br.fuse_advantage(tree, st["rewards"], st["logp"], 1.0, 1e-8, 0, synth.ADV_CLIP, st["rbar"], st["adv"])
    br.prune(tree, st["rewards"], br.PRUNE_PARENT_TOP1, 0, st["mask"], st["kept"], st["n_kept"])
    # the one read-back of an iteration: the kept edges size the batches of the re-evaluation
    return st["kept"][:int(st["n_kept"])]


def run(st):
    kind = st["case"]["kind"]
    if kind == "velocity":
        br.velocity(st["model"], st["z"], st["t"], st["cond"], st["index"], st["v"], st["ws"])
        return st["v"]
    tree, sched = st["tree"], st["sched"]
    if kind == "sde":
        br.sde_step(tree, sched, st["seed"], st["case"]["step"], st["case"]["D"], st["v"], st["z"], st["logp"], st["scratch"])
        return st["z"], st["logp"]
    if kind == "post":
        kept = _post(st)
        return st["rewards"], st["rbar"], st["adv"], kept
    if kind == "logprob":
        out = st["out"]
        br.logprob(tree, st["model2"], sched, st["cond"], st["z"], st["ids"], out, st["ws"])
        return out
    br.rollout(tree, st["model"], sched, st["seed"], st["groups"], st["cond"], st["z"], st["logp"], None, st["ws"])
    if kind == "rollout":
        return st["z"], st["logp"]
    kept = _post(st)
    new = st["logp_new"][:len(kept)]
    br.logprob(tree, st["model2"], sched, st["cond"], st["z"], kept.cpu().numpy(), new, st["ws"])
    br.grpo_objective(new, st["logp"], st["adv"], kept, len(kept), synth.CLIP_RANGE, st["J"])
    return st["z"], st["logp"], st["rewards"], st["rbar"], st["adv"], kept, new, st["J"]
