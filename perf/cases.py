"""The calls whose time matters, as data: what users of the library have it do, through its Python entry points.

A case is a dict of plain values.  `listed()` holds the named ones, `draw(rng)` gives another one of the same ranges,
`prepare` makes what a program holds before the call (weights and handle, inputs, reusable outputs and workspaces), `run`
is one call, `work` what the call cannot do without and `tolerance` how far a correct result may be from another one.

Model shapes are the class-conditional DiT ones the library is built for: patch 2 on 4-channel latents, widths 384 / 768 /
1152 (6 / 12 / 16 heads, 12 / 12 / 28 blocks), latents of 256^2 (32 x 32) and 512^2 (64 x 64) images and other even sizes.
"""
import math

import numpy as np
import torch

from paper_2511_20390_amd import binding, synth

# hidden width -> blocks, heads
WIDTHS = {384: (12, 6), 768: (12, 12), 1152: (28, 16)}
CHANNELS = 4
POOL = 1 << 24


def listed():
    xl, s = dict(hidden=1152, mode="bf16"), dict(hidden=384, mode="bf16")
    return [
        # one trajectory's drafts checked inside a sampling loop at 256^2: all latency
        dict(name="verify_one_256", op="verify", n_traj=1, K=6, d=4096, relaxed=False),
        # many trajectories checked in one call at 512^2, uncertainty-relaxed rule: the streaming rate
        dict(name="verify_64_512", op="verify", n_traj=64, K=6, d=16384, relaxed=True),
        # one variance per element, odd counts and a latent that is no multiple of anything large
        dict(name="verify_diag_ragged", op="verify_diag", n_traj=23, K=5, d=4 * 33 * 47, relaxed=False),
        # one guided step of the sequential sampler at 256^2 (conditional and null state): few rows, all weights
        dict(name="forward_256_pair", op="forward", lat_h=32, lat_w=32, B=2, feat=False, **xl),
        # the same step in full precision
        dict(name="forward_256_pair_fp32", op="forward", lat_h=32, lat_w=32, B=2, feat=False, hidden=1152, mode="fp32"),
        # a batch of a small model on a latent that is neither square nor a power of two, features kept
        dict(name="forward_small_ragged", op="forward", lat_h=36, lat_w=50, B=5, feat=True, **s),
        # drafting round of a guided 512^2 chain: six dependent steps of the one-block drafter
        dict(name="draft_512", op="draft", lat_h=64, lat_w=64, K=6, cfg_scale=4.0, **xl),
        # drafting round of an unguided 256^2 chain
        dict(name="draft_256", op="draft", lat_h=32, lat_w=32, K=4, cfg_scale=1.0, **xl),
        # verification round without guidance at 256^2: four states in one pack
        dict(name="round_256", op="round", lat_h=32, lat_w=32, K=4, cfg_scale=1.0, relaxed=False, **xl),
        # a long speculation at 256^2 with guidance: 32 states in one pack
        dict(name="round_256_long", op="round", lat_h=32, lat_w=32, K=16, cfg_scale=1.5, relaxed=True, **xl),
        # the headline verification round: six guided states at 512^2
        dict(name="round_512", op="round", lat_h=64, lat_w=64, K=6, cfg_scale=4.0, relaxed=True, **xl),
        # a whole (respaced) sampler run at 256^2 with guidance: target steps, drafting, rounds, host decisions
        dict(name="sample_256", op="sample", lat_h=32, lat_w=32, S=10, L=4, cfg_scale=4.0, **xl),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["verify", "verify_diag", "forward", "forward", "draft", "round", "round", "sample"])
    if op in ("verify", "verify_diag"):
        K = rng.randint(1, 8)
        d = CHANNELS * rng.randint(16, 72) * rng.randint(16, 72)
        n_max = max(1, min(64, 64 * 6 * 16384 // (K * d * (4 if op == "verify_diag" else 3) // 3)))
        return dict(op=op, n_traj=_log_int(rng, 1, n_max), K=K, d=d, relaxed=rng.random() < 0.5)
    case = dict(op=op, lat_h=2 * rng.randint(8, 34), lat_w=2 * rng.randint(8, 34), hidden=1152, mode="bf16")
    tok = case["lat_h"] * case["lat_w"] // 4
    guided = rng.random() < 0.6
    if op == "forward":
        case["hidden"] = rng.choice([384, 768, 1152, 1152])
        case["mode"] = "fp32" if rng.random() < 0.2 else "bf16"
        rows = 600 if case["mode"] == "fp32" else 10000
        case.update(B=_log_int(rng, 1, max(1, min(32, rows // tok))), feat=rng.random() < 0.3)
        return case
    case["cfg_scale"] = rng.choice([1.5, 4.0]) if guided else 1.0
    dup = 2 if guided else 1
    if op == "draft":
        case["K"] = rng.randint(1, 8)
    elif op == "round":
        case.update(K=_log_int(rng, 1, max(1, min(16, 10000 // (dup * tok)))), relaxed=rng.random() < 0.5)
    else:
        # guidance on: the drafts of random networks are then far from acceptance, so that no rounding
        # difference can change which ones are accepted
        case.update(lat_h=2 * rng.randint(9, 15), lat_w=2 * rng.randint(9, 15), S=rng.randint(6, 9), L=rng.randint(2, 4),
                    cfg_scale=4.0)
    return case


# ---- sizes ---------------------------------------------------------------------------------------------------
def _cfg(case):
    depth, heads = WIDTHS[case["hidden"]]
    return synth.dit_config("xl2_256", lat_h=case["lat_h"], lat_w=case["lat_w"], hidden=case["hidden"], depth=depth,
                            heads=heads, mlp_hidden=4 * case["hidden"])


DRAFTER_DEPTH = {"draft": 1, "sample": 2}


def _dup(case):
    return 2 if case["cfg_scale"] > 1.0 else 1


# ---- what a program holds before the call --------------------------------------------------------------------
def _weights(spec, rng):
    """Every tensor ~ N(0, 0.02^2): a window of one seeded pool each (hundreds of millions of fresh draws would take
    longer than everything else here)."""
    pool = rng.standard_normal(POOL, dtype=np.float32) * np.float32(0.02)
    w = {}
    for name, shape in spec:
        n = int(np.prod(shape))
        o = int(rng.integers(0, (POOL - n) // 4)) * 4
        w[name] = pool[o:o + n].reshape(shape)
    return w


def _randn(shape, g):
    return torch.randn(shape, generator=g, device="cuda:0", dtype=torch.float32)


def _rand(shape, g):
    return torch.rand(shape, generator=g, device="cuda:0", dtype=torch.float32)


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to("cuda:0")


def _steps(t):
    """Device arrays of the transition coefficients at the timesteps t."""
    cx, ce, sg = binding.free_ddpm_schedule()
    return dict(t=_dev(t, np.int32), coef_x=_dev(cx[t], np.float32), coef_eps=_dev(ce[t], np.float32),
                sigma=_dev(sg[t], np.float32))


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    op = case["op"]
    if op in ("verify", "verify_diag"):
        return _prepare_verify(case, rng, g)
    cfg = _cfg(case)
    model = binding.FreeDit(cfg, _weights(synth.weight_spec(cfg), rng), case["mode"])
    st = dict(op=op, model=model)
    shape = (cfg["in_ch"], cfg["lat_h"], cfg["lat_w"])
    d, y = synth.latent_dim(cfg), int(rng.integers(0, cfg["num_classes"]))
    if op == "forward":
        B = case["B"]
        st.update(x=_randn((B,) + shape, g), feat=case["feat"], t=_dev(rng.integers(0, 1000, B), np.int32),
                  y=_dev(rng.integers(0, cfg["num_classes"] + 1, B), np.int32))
        return st
    if op in DRAFTER_DEPTH:
        depth = DRAFTER_DEPTH[op]
        st["drafter"] = binding.FreeDrafter(model, _weights(synth.drafter_weight_spec(cfg, depth), rng), depth)
    if op == "sample":
        # respaced schedule; the last transition is noise-free and never speculated
        S = case["S"]
        t = np.linspace(999, 0, S).round().astype(np.int32)
        a = _steps(t)
        a["sigma"][-1] = 0.0
        st.update(y=y, scale=case["cfg_scale"], S=S, L=case["L"], x=_randn(shape, g), xi=_randn((S, d), g), u=_rand((S,), g),
                  lam=_dev(synth.relaxation_profile(t), np.float32), **a)
        return st
    K = case["K"]
    t = int(rng.integers(K - 1, 1000)) - np.arange(K)
    st.update(y=y, scale=case["cfg_scale"], **_steps(t))
    if op == "draft":
        dup, ntok = _dup(case), synth.n_tokens(cfg)
        st.update(x_a=_randn(shape, g), f_a=_randn((dup, ntok, cfg["hidden"]), g), xi=_randn((K, d), g))
        return st
    # a verification round: the state, K drafts around it, each a sample of its proposal
    x_in = _randn((1,) + shape, g)
    drafts = x_in + 0.1 * _randn((K,) + shape, g)
    st.update(x_states=torch.cat([x_in, drafts[:K - 1]]), x_last=drafts[K - 1].clone(), u=_rand((K,), g),
              m_draft=drafts.reshape(K, d) - st["sigma"][:, None] * _randn((K, d), g),
              lam=_dev(synth.relaxation_profile(t), np.float32) if case["relaxed"] else None)
    st["out"] = dict(m_target=torch.empty(K, d, device="cuda:0"), log_ratio=torch.empty(K, device="cuda:0"),
                     accept=torch.empty(K, dtype=torch.uint8, device="cuda:0"),
                     n_accept=torch.empty(1, dtype=torch.int32, device="cuda:0"), x_out=torch.zeros(d, device="cuda:0"))
    return st


def _prepare_verify(case, rng, g):
    """Draft means at the distance from the target means that gives about half of the drafts a chance."""
    n, K, d = case["n_traj"], case["K"], case["d"]
    t = rng.integers(0, 1000, size=(n, K))
    sigma = _steps(t.reshape(-1))["sigma"].reshape(n, K)
    s = sigma[..., None]
    st = dict(op=case["op"], u=_rand((n, K), g), m_target=_randn((n, K, d), g),
              lam=_dev(synth.relaxation_profile(t), np.float32) if case["relaxed"] else None)
    if case["op"] == "verify_diag":
        s = s * torch.exp(0.4 * _randn((n, K, d), g))
        st["sigma_elem"] = s
    else:
        st["sigma"] = sigma
    st["m_draft"] = st["m_target"] + (1.349 / math.sqrt(d)) * s * _randn((n, K, d), g)
    st["x_draft"] = st["m_draft"] + s * _randn((n, K, d), g)
    st["out"] = dict(log_ratio=torch.empty(n, K, device="cuda:0"), accept=torch.empty(n, K, dtype=torch.uint8, device="cuda:0"),
                     n_accept=torch.empty(n, dtype=torch.int32, device="cuda:0"), x_out=torch.zeros(n, d, device="cuda:0"))
    st["ws"] = torch.empty(max(256, binding.spec_verify_workspace_bytes(n, K, d)), dtype=torch.uint8, device="cuda:0")
    return st


# ---- one call ------------------------------------------------------------------------------------------------
def run(s):
    op = s["op"]
    if op == "verify":
        return binding.spec_verify(s["m_target"], s["m_draft"], s["x_draft"], s["sigma"], s["u"], s["lam"], out=s["out"],
                                   workspace=s["ws"])
    if op == "verify_diag":
        return binding.spec_verify_diag(s["m_target"], s["m_draft"], s["x_draft"], s["sigma_elem"], s["u"], s["lam"],
                                        out=s["out"], workspace=s["ws"])
    if op == "forward":
        return s["model"].dit_forward_packed(s["x"], s["t"], s["y"], want_feat=s["feat"])
    if op == "draft":
        return s["drafter"].draft_round(s["x_a"], s["f_a"], s["t"], s["y"], s["scale"], s["coef_x"], s["coef_eps"],
                                        s["sigma"], s["xi"], want_feat=True)
    if op == "round":
        return s["model"].spec_round(s["x_states"], s["x_last"], s["m_draft"], s["t"], s["y"], s["scale"], s["coef_x"],
                                     s["coef_eps"], s["sigma"], s["u"], s["lam"], out=s["out"])
    x, stats, log = binding.free_sample(s["drafter"], s["x"], s["y"], s["scale"], s["S"] - 1, s["L"], s["t"], s["coef_x"],
                                        s["coef_eps"], s["sigma"], s["xi"], s["u"], s["lam"])
    return dict(x=x, stats=stats, accepted=np.asarray(log, np.int32))


# ---- what a call cannot do without -----------------------------------------------------------------------------
def _blocks_flops(cfg, rows, samples, depth):
    """Linear layers and attention of `depth` blocks, the modulation vectors of each sample, the output layer."""
    D, F, tok = cfg["hidden"], cfg["mlp_hidden"], synth.n_tokens(cfg)
    c_out = cfg["in_ch"] * cfg["patch"] ** 2 * 2
    return depth * (2.0 * rows * D * (4 * D + 2 * F) + 4.0 * rows * tok * D) + 2.0 * samples * D * D * (6 * depth + 2) + \
        2.0 * rows * D * c_out


def _weight_bytes(spec, mode):
    """Every weight once; of the label table only the rows that are looked up count (none here)."""
    return sum(int(np.prod(sh)) * (2 if mode == "bf16" and synth.is_big_matrix(n) else 4) for n, sh in spec if n != "y_table")


def work(case):
    op = case["op"]
    if op in ("verify", "verify_diag"):
        n, K, d = case["n_traj"], case["K"], case["d"]
        arrays = 4 if op == "verify_diag" else 3
        # the arrays once, scalars in and out, one state out per trajectory
        return {"bytes": 4 * arrays * n * K * d + 17 * n * K + 4 * n * d, "flops": 6 * n * K * d}
    cfg = _cfg(case)
    tok, D, d, mode = synth.n_tokens(cfg), cfg["hidden"], synth.latent_dim(cfg), case["mode"]
    wb = _weight_bytes(synth.weight_spec(cfg), mode)
    depth = cfg["depth"]
    if op == "forward":
        B = case["B"]
        return {"bytes": wb + 4 * B * d * 3 + (4 * B * tok * D if case["feat"] else 0),
                "flops": _blocks_flops(cfg, B * tok, B, depth)}
    dup = _dup(case)
    if op == "round":
        K = case["K"]
        return {"bytes": wb + 4 * d * (3 * K + 2), "flops": _blocks_flops(cfg, dup * K * tok, dup * K, depth)}
    dd = DRAFTER_DEPTH[op]
    emb = _weight_bytes([e for e in synth.weight_spec(cfg) if e[0].startswith(("patch_", "t_"))], mode)
    wd = _weight_bytes(synth.drafter_weight_spec(cfg, dd), mode)
    step = _blocks_flops(cfg, dup * tok, dup, dd) + 4.0 * dup * tok * D * D
    if op == "draft":
        K = case["K"]
        return {"bytes": emb + wd + 4 * (d * (3 * K + 2) + 2 * dup * tok * D), "flops": K * step}
    # sample: the first and the last step are plain target steps; in between every transition is a round of its own,
    # since the drafts of random networks are rejected (the last rounds are shorter than L)
    S, L = case["S"], case["L"]
    ks = [min(L, S - 1 - i) for i in range(1, S - 1)]
    flops = sum(_blocks_flops(cfg, dup * k * tok, dup * k, depth) + k * step for k in ks) + 2 * _blocks_flops(cfg, dup * tok, dup, depth)
    return {"bytes": wb + wd + 4 * d * (S + 2), "flops": flops}


# ---- how far apart two correct results may be ------------------------------------------------------------------
def tolerance(case):
    """About four times what was seen between the bf16 path and fp32 activations on the same (bf16) matrices, and between
    the LayerNorms folded into the matrix products and computed separately; for fp32 and the verification sums between the
    path and the same in 64 bits."""
    op = case["op"]
    if op in ("verify", "verify_diag"):
        return {"rel": 2e-6}        # fp64 sums rounded to fp32; the reflected sample is a short fp32 expression
    if case["mode"] == "fp32":
        return {"rel": 2e-5}        # seen: 4e-6
    # seen: forward 9e-4; top feature at the end of a drafting chain 2.3e-3; means of a round and what is computed from
    # them 2.2e-5 (the noise estimate enters with a small coefficient); result of a sampler run 1.2e-4
    return {"rel": {"forward": 4e-3, "draft": 1e-2, "round": 2e-4, "sample": 5e-4}[op]}
