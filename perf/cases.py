"""Performance cases of the denoising rollout library: what its users run, call by call.

A program that rolls a video world model out with this library calls, per
denoising step, the surrogate candidate and the risk controller on the latent
and, on exact steps, the denoiser F_theta: conditioning vector, transformer
blocks over the joint video + text sequence, output head. The cases are those
calls over the range of the repository's workloads (256 tokens in float32 to
118,800 tokens in bfloat16), most of them a single layer or block so that a
change of rounding shows where it happens.

``exact`` recomputes every case in float64 with plain torch from the same
seeded inputs, without any code of the package.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

DEV = "cuda:0"

# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------


def _model(kind, dtype, hidden, head_dim, lat, text=0, blocks=1, block="seq", cond=0, cam=0, text_dim=256, batch=1):
    f, h, w = lat
    return {"kind": kind, "dtype": dtype, "hidden": hidden, "head_dim": head_dim, "f": f, "h": h, "w": w,
            "text": text, "text_dim": text_dim, "blocks": blocks, "block": block, "cond": cond, "cam": cam,
            "batch": batch}


def _latent(kind, lat, bank=4, steps=12, surrogate="lifted", observation="kernel", tau=0.5):
    f, h, w = lat
    return {"kind": kind, "f": f, "h": h, "w": w, "bank": bank, "steps": steps, "surrogate": surrogate,
            "observation": observation, "tau": tau}


def listed():
    return [
        # whole F_theta of the smallest workload (float32, 256 tokens): launches and latency count
        {"name": "forward_tiny_f32", **_model("forward", "f32", 256, 64, (4, 16, 16), blocks=2, cond=256)},
        # one block of an ordinary model run in float32 (reference-precision runs)
        {"name": "block_f32", **_model("block", "f32", 1024, 64, (7, 32, 48))},
        # whole F_theta of the mid-size workload, one sample: an interactive rollout's exact step
        {"name": "forward_mid", **_model("forward", "bf16", 1024, 64, (7, 32, 48), blocks=8, cond=1024)},
        # eight rollouts served together: embedding, one block and head of the mid-size model at batch 8
        {"name": "batch8_mid", **_model("batch", "bf16", 1024, 64, (7, 32, 48), cond=1024, batch=8)},
        # a block of the 5B-shaped model: joint sequence with 226 text tokens (17,776 in all), head size 64
        {"name": "block_seq_5b", **_model("block", "bf16", 3072, 64, (13, 60, 90), text=226)},
        # a dual-stream block of the 13B-shaped model: 67,320 video and 256 text tokens, head size 128
        {"name": "block_dual_13b", **_model("block", "bf16", 3072, 128, (33, 68, 120), text=256, block="dual")},
        # a single-stream block at the longest sequence of the workloads (118,800 tokens)
        {"name": "block_single_long", **_model("block", "bf16", 3072, 128, (33, 90, 160), block="single")},
        # the attention of a short clip at an odd length, 24 heads of 128
        {"name": "attention_ragged", "kind": "attention", "dtype": "bf16", "heads": 24, "head_dim": 128, "n": 9001},
        # the text projection of the 5B-shaped model: few rows, long K
        {"name": "linear_text", "kind": "linear", "dtype": "bf16", "m": 226, "n": 3072, "k": 4096},
        # the conditioning vector of the 5B-shaped model (timestep, condition, camera): the smallest call
        {"name": "cond_embed_5b", **_model("cond", "bf16", 3072, 64, (1, 8, 8), cond=4096, cam=3072)},
        # one candidate and decision on the mid-size latent, through the step calls
        {"name": "step_mid", **_latent("step", (7, 32, 48))},
        # the surrogate, risk and exact-step kernels on the largest latent: a rollout on recorded velocities
        {"name": "rollout_large", **_latent("rollout", (33, 90, 160), steps=12)},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi):
    """Latent (f, h, w) with h and w even whose (1, 2, 2) patches make about lo..hi tokens."""
    n = _logint(rng, lo, hi)
    f = min(33, max(1, _logint(rng, 1, 33)), max(1, n // 16))
    hw = max(4.0, n / f)
    gh = max(2, min(45, int(round(math.sqrt(hw * rng.uniform(0.4, 0.8))))))
    gw = max(2, min(80, int(round(hw / gh))))
    return f, 2 * gh, 2 * gw


def draw(rng):
    kind = rng.choice(["forward_f32", "block_f32", "forward", "batch", "block", "block", "attention", "linear",
                       "cond", "step", "rollout"])
    text = rng.choice([0, rng.randint(1, 300)])
    block = rng.choice(["seq", "dual", "single"])
    hd = rng.choice([64, 128])
    if block == "dual" and text == 0:
        text = 77
    if kind == "forward_f32":
        return _model("forward", "f32", rng.choice([256, 512]), hd, _grid(rng, 40, 800), text=text % 64 if block != "dual" else 33,
                      blocks=rng.randint(1, 3), block=block, cond=256)
    if kind == "block_f32":
        return _model("block", "f32", rng.choice([256, 512, 768, 1024]), hd, _grid(rng, 200, 3000), text=text, block=block)
    if kind == "forward":
        return _model("forward", "bf16", rng.choice([512, 768, 1024, 1536]), hd, _grid(rng, 256, 6000), text=text,
                      blocks=rng.randint(1, 8), block=block, cond=rng.choice([0, 1024]))
    if kind == "batch":
        return _model("batch", "bf16", rng.choice([512, 1024, 1536]), hd, _grid(rng, 256, 4000), text=text, block=block,
                      cond=1024, batch=rng.randint(2, 8))
    if kind == "block":
        return _model("block", "bf16", rng.choice([1024, 1536, 2048, 3072]), hd, _grid(rng, 700, 70000), text=text,
                      block=block)
    if kind == "attention":
        return {"kind": "attention", "dtype": "bf16", "heads": rng.choice([4, 8, 12, 16, 24, 48] + [6, 30] * (hd == 128)),
                "head_dim": hd, "n": _logint(rng, 100, 40000)}
    if kind == "linear":
        return {"kind": "linear", "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), "m": _logint(rng, 1, 9000),
                "n": 64 * _logint(rng, 4, 144), "k": 64 * _logint(rng, 4, 144)}
    if kind == "cond":
        return _model("cond", rng.choice(["bf16", "f32"]), rng.choice([256, 1024, 1536, 3072]), 64, (1, 8, 8),
                      cond=rng.choice([256, 1000, 4096]), cam=rng.choice([0, 96, 3072]))
    lat = (rng.randint(1, 33), _logint(rng, 8, 90), _logint(rng, 8, 160))
    surrogate = rng.choice(["lifted", "lifted", "secant"])
    observation = rng.choice(["kernel", "kernel", "linear"])
    return _latent("step" if kind == "step" else "rollout", lat, bank=rng.choice([2, 4, 4, 8]),
                   steps=rng.randint(6, 16), surrogate=surrogate, observation=observation)


# ---------------------------------------------------------------------------
# seeded inputs
# ---------------------------------------------------------------------------


def _td(case):
    return torch.bfloat16 if case.get("dtype") == "bf16" else torch.float32


def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + what * 7919 + 17) % (1 << 62))
    return g


def _randn(g, shape, dtype=torch.float32, std=1.0):
    return (torch.randn(shape, generator=g, device=DEV, dtype=torch.float32) * std).to(dtype)


def _config(case):
    """The workload fields of a model, as the library's Context takes them."""
    hd, nb = case["head_dim"], case["blocks"]
    gf, gh, gw = case["f"], case["h"] // 2, case["w"] // 2
    return SimpleNamespace(
        name="case", dtype=case["dtype"], hidden=case["hidden"], heads=case["hidden"] // hd, head_dim=hd, mlp_ratio=4,
        n_seq=nb if case["block"] == "seq" else 0, n_dual=nb if case["block"] == "dual" else 0,
        n_single=nb if case["block"] == "single" else 0, cond_dim=case["cond"], cam_dim=case["cam"],
        text_tokens=case["text"], text_dim=case["text_dim"], latent=(16, case["f"], case["h"], case["w"]),
        patch=(1, 2, 2), rope=(16, 24, 24) if hd == 64 else (16, 56, 56), qk_norm=True, n_video=gf * gh * gw)


def _specs(case):
    """Names and shapes of the model's weights (Linear weights [out, in], biases [out])."""
    d, f = case["hidden"], 4 * case["hidden"]
    out = []

    def lin(name, n, k):
        out.append((name + ".w", (n, k)))
        out.append((name + ".b", (n,)))

    lin("t_embed.fc1", d, 256)
    lin("t_embed.fc2", d, d)
    if case["cond"]:
        lin("cond_embed", d, case["cond"])
    if case["cam"]:
        lin("cam_embed", d, case["cam"])
    if case["text"]:
        lin("text_proj", d, case["text_dim"])
    lin("patch_embed", d, 64)
    for i in range(case["blocks"]):
        if case["block"] == "single":
            lin(f"single.{i}.ada", 3 * d, d)
            lin(f"single.{i}.lin1", 3 * d + f, d)
            lin(f"single.{i}.lin2", d, d + f)
            continue
        for pre in ([f"seq.{i}"] if case["block"] == "seq" else [f"dual.{i}.vid", f"dual.{i}.txt"]):
            lin(pre + ".ada", 6 * d, d)
            lin(pre + ".qkv", 3 * d, d)
            lin(pre + ".out", d, d)
            lin(pre + ".fc1", f, d)
            lin(pre + ".fc2", d, f)
    lin("final.ada", 2 * d, d)
    lin("final.lin", 64, d)
    return out


def _weights(case, seed):
    """(name, values) of every weight, N(0, 0.02^2) rounded to the model type, one at a time."""
    g = _gen(seed, 1)
    for name, shape in _specs(case):
        yield name, _randn(g, shape, _td(case), 0.02)


def _model_inputs(case, seed):
    g, td, b = _gen(seed, 2), _td(case), case["batch"]
    lat = (16, case["f"], case["h"], case["w"])
    inp = {"z": [_randn(g, lat) for _ in range(b)]}
    for key, shape in (("cond", (case["cond"],)), ("cam", (case["cam"],)), ("text", (case["text"], case["text_dim"]))):
        inp[key] = [_randn(g, shape, td) if case[key] else None for _ in range(b)]
    return inp


def _block_inputs(case, seed):
    g = _gen(seed, 3)
    n = case["f"] * (case["h"] // 2) * (case["w"] // 2) + case["text"]
    return _randn(g, (n, case["hidden"])), _randn(g, (case["hidden"],))


def _attention_inputs(case, seed):
    g = _gen(seed, 4)
    shape = (case["heads"], case["n"], case["head_dim"])
    return [_randn(g, shape, _td(case)) for _ in range(3)]


def _linear_inputs(case, seed):
    g, td = _gen(seed, 5), _td(case)
    return (_randn(g, (case["m"], case["k"]), td), _randn(g, (case["n"], case["k"]), td, 0.02),
            _randn(g, (case["n"],), td, 0.02))


def _trajectory(case, seed, count):
    """z_T and ``count`` velocities: a shared direction plus per-step noise, as along a denoising trajectory."""
    g = _gen(seed, 6)
    lat = (16, case["f"], case["h"], case["w"])
    z, base = _randn(g, lat), _randn(g, lat)
    v = torch.empty((count,) + lat, device=DEV)
    for k in range(count):
        v[k] = base + 0.3 * _randn(g, lat)
    return z, v


def _step_inputs(case, seed):
    """Latents z_0..z_m of m exact steps that fill the bank (m = its capacity), inside a 50-step rollout."""
    z, v = _trajectory(case, seed, case["bank"])
    zs = [z]
    for k in range(case["bank"]):
        zs.append(zs[-1] - v[k] / 50)
    return zs


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------


def _context(case, seed):
    import paper_2608_01845_amd as wdc
    ctx = wdc.Context(_config(case), max_batch=case["batch"], allocate_weights=True)
    table = {name: (shape, off) for name, shape, off in ctx.weight_table()}
    for name, w in _weights(case, seed):
        shape, off = table.pop(name)
        assert tuple(shape) == tuple(w.shape), name
        flat = w.reshape(-1).view(torch.uint8)
        ctx.weights[off:off + flat.numel()].copy_(flat)
    assert not table
    return ctx


def _latent_context(case):
    import paper_2608_01845_amd as wdc
    # no blocks (surrogate-only use): one patch, so that the workspace holds no token buffers
    cfg = SimpleNamespace(
        name="latent", dtype="f32", hidden=256, heads=4, head_dim=64, mlp_ratio=4, n_seq=0, n_dual=0, n_single=0,
        cond_dim=0, cam_dim=0, text_tokens=0, text_dim=0, latent=(16, case["f"], case["h"], case["w"]),
        patch=(case["f"], case["h"], case["w"]), rope=(0, 0, 0), qk_norm=False, n_video=1)
    params = wdc.default_params(
        bank_capacity=case["bank"], tau_risk=case["tau"],
        surrogate=wdc.SURROGATE_SECANT if case["surrogate"] == "secant" else wdc.SURROGATE_LIFTED,
        observation=wdc.OBS_LINEAR if case["observation"] == "linear" else wdc.OBS_KERNEL)
    return wdc.Context(cfg, params=params, allocate_weights=False)


def prepare(case, seed):
    import paper_2608_01845_amd as wdc
    kind = case["kind"]
    s = SimpleNamespace(case=case, kind=kind)
    if kind in ("forward", "batch", "cond"):
        s.ctx, s.inp = _context(case, seed), _model_inputs(case, seed)
        s.out = [torch.empty_like(z) for z in s.inp["z"]]
        s.cemb = torch.empty(case["hidden"], device=DEV)
    elif kind == "block":
        s.ctx = _context(case, seed)
        s.x0, s.cemb = _block_inputs(case, seed)
        s.x = torch.empty_like(s.x0)
    elif kind in ("attention", "linear"):
        cfg = {"hidden": 256, "head_dim": 64, **case, "f": 1, "h": 8, "w": 8, "text": 0, "text_dim": 0, "blocks": 1,
               "block": "seq", "cond": 0, "cam": 0, "batch": 1}
        if kind == "attention":
            cfg["hidden"] = case["heads"] * case["head_dim"]
            # a model whose sequence has the case's length, so that its workspace is the one a program would hold
            cfg["w"] = 8 * ((case["n"] + 15) // 16)
        cfg["hidden"] = (cfg["hidden"] + 255) // 256 * 256 if kind == "linear" else cfg["hidden"]
        s.ctx = wdc.Context(_config(cfg), allocate_weights=False)
        if kind == "linear":
            s.a, s.w, s.b = _linear_inputs(case, seed)
            s.c = torch.empty((case["m"], case["n"]), dtype=_td(case), device=DEV)
        else:
            q, k, v = _attention_inputs(case, seed)
            n, npad = case["n"], s.ctx.attn_pad(case["n"])
            h, hd = case["heads"], case["head_dim"]
            pad = torch.nn.functional.pad
            s.q, s.k = (pad(t, (0, 0, 0, npad - n)).contiguous() for t in (q, k))
            pos = torch.arange(npad, device=DEV)
            col = (pos & ~12) | ((pos & 4) << 1) | ((pos & 8) >> 1)   # key j at column j with bits 2 and 3 swapped
            s.vt = pad(v, (0, 0, 0, npad - n)).transpose(1, 2)[:, :, col].contiguous()
            s.o = torch.empty((n, h * hd), dtype=_td(case), device=DEV)
    elif kind == "rollout":
        s.ctx = _latent_context(case)
        s.state = s.ctx.new_state()
        s.z0, s.v = _trajectory(case, seed, case["steps"])
        s.z = torch.empty_like(s.z0)
    else:
        s.ctx = _latent_context(case)
        s.state = s.ctx.new_state()
        s.state.reset()
        s.zs = _step_inputs(case, seed)
        s.zhat = torch.empty_like(s.zs[0])
        for k in range(case["bank"]):
            s.ctx.surrogate_step(s.state, s.zs[k], k, 50, s.zhat)
            s.ctx.risk_update(s.state, wdc.POST_EXACT, k, 50, s.zs[k], s.zs[k + 1])
    return s


def run(s):
    case, ctx, kind = s.case, s.ctx, s.kind
    if kind == "forward":
        i = s.inp
        return ctx.forward(i["z"][0], 0.6, i["cond"][0], i["text"][0], i["cam"][0], out=s.out[0])
    if kind == "batch":
        i = s.inp
        some = {k: i[k] if case[k] else None for k in ("cond", "text", "cam")}
        return ctx.forward_batch(i["z"], 0.6, some["cond"], some["text"], some["cam"], outs=s.out)
    if kind == "cond":
        return ctx.cond_embed(0.6, s.inp["cond"][0], s.inp["cam"][0], out=s.cemb)
    if kind == "block":
        s.x.copy_(s.x0)                       # the block updates the residual stream in place
        return ctx.block_forward(0, s.x, s.cemb)
    if kind == "attention":
        return ctx.attention(s.q, s.k, s.vt, case["n"], s.o, s.o.shape[1])
    if kind == "linear":
        return ctx.linear(s.a, s.w, s.b, s.c, case["m"], case["n"], case["k"])
    if kind == "rollout":
        s.z.copy_(s.z0)                       # the rollout updates the latent in place
        sched, logs = ctx.rollout(s.state, s.z, case["steps"], replay_v=s.v)
        return {"z": s.z, "schedule": np.array(sched, dtype=np.int64),
                "log": np.array([[lg["d_z"], lg["r_cand"], lg["eta"], lg["R"]] for lg in logs])}
    k = case["bank"]
    log = ctx.surrogate_step(s.state, s.zs[k], k, 50, s.zhat)
    dec = ctx.risk_update(s.state, 0, k, 50)  # 0: the decision
    return {"zhat": s.zhat, "exact": int(dec["exact"]), "log": np.array([log["d_z"], log["alpha"], dec["r_cand"]])}


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------


def _block_work(case):
    n = case["f"] * (case["h"] // 2) * (case["w"] // 2) + case["text"]
    d = case["hidden"]
    return n, 24.0 * n * d * d + 4.0 * n * n * d


def _param_count(case, pre=None):
    return sum(math.prod(shape) for name, shape in _specs(case) if pre is None or name.startswith(pre))


def work(case):
    kind = case["kind"]
    e = 2 if case.get("dtype") == "bf16" else 4
    if kind in ("forward", "batch"):
        n, fl = _block_work(case)
        b, d, nv = case["batch"], case["hidden"], n - case["text"]
        one = case["blocks"] * fl + 4.0 * nv * 64 * d + 2.0 * case["text"] * case["text_dim"] * d
        return {"bytes": e * _param_count(case) + b * (8.0 * nv * 64 + e * (case["text"] * case["text_dim"] + case["cond"])),
                "flops": b * one}
    if kind == "block":
        n, fl = _block_work(case)
        return {"bytes": e * _param_count(case, case["block"] + ".0") + 8.0 * n * case["hidden"], "flops": fl}
    if kind == "cond":
        p = sum(_param_count(case, pre) for pre in ("t_embed", "cond_embed", "cam_embed"))
        return {"bytes": e * p + 4.0 * case["hidden"], "flops": 2.0 * p}
    if kind == "attention":
        h, n, hd = case["heads"], case["n"], case["head_dim"]
        return {"bytes": 4.0 * e * h * n * hd, "flops": 4.0 * h * n * n * hd}
    if kind == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": float(e) * (m * k + n * k + m * n), "flops": 2.0 * m * n * k}
    elems = 16.0 * case["f"] * case["h"] * case["w"]
    if case["surrogate"] == "secant":
        m = 3
    else:
        m = case["bank"] if case["observation"] == "kernel" else 2 * case["bank"] + 1
    if kind == "step":   # z and the anchor, the combined latents, the candidate
        return {"bytes": elems * 4 * (2 + m + 1), "flops": elems * (2 * m + 8)}
    # every step builds its candidate; about one in four is exact (z, v, z_a, candidate read; z', bank, anchor written)
    return {"bytes": elems * 4 * case["steps"] * (m + 2 + 7 / 4), "flops": elems * case["steps"] * (2 * m + 12)}


def tolerance(case):
    # about four times the error against the float64 results: bf16 products and attention carry their
    # operands' and outputs' rounding, float32 paths only the order of their sums
    kind, bf16 = case["kind"], case.get("dtype") == "bf16"
    if kind in ("step", "rollout"):
        return {"rel": 2e-6, "max": 2e-5}
    if kind == "cond" or not bf16:
        return {"rel": 4e-6, "max": 4e-5}
    return {"forward": {"rel": 1.4e-2, "max": 0.1}, "batch": {"rel": 1.1e-2, "max": 0.1},
            "block": {"rel": 8e-3, "max": 0.15}, "attention": {"rel": 1.2e-2, "max": 0.1},
            "linear": {"rel": 7e-3, "max": 0.02}}[kind]


# ---------------------------------------------------------------------------
# float64 results
# ---------------------------------------------------------------------------


def _ln(x):
    x = x - x.mean(-1, keepdim=True)
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6)


def _softmax_attention(q, k, v):
    """[n, hd] float64 of one head, queries in slices."""
    out = torch.empty_like(q)
    step = max(256, (1 << 27) // k.shape[0])
    kt = k.t().contiguous() / math.sqrt(q.shape[1])
    for i in range(0, q.shape[0], step):
        p = q[i:i + step] @ kt
        p -= p.amax(-1, keepdim=True)
        p.exp_()
        out[i:i + step] = (p @ v) / p.sum(-1, keepdim=True)
    return out


def _rope_table(case):
    hd = case["head_dim"]
    dims = (16, 24, 24) if hd == 64 else (16, 56, 56)
    f, h, w = case["f"], case["h"] // 2, case["w"] // 2
    n = torch.arange(f * h * w, device=DEV)
    pos = (n // (h * w), (n // w) % h, n % w)
    ang = []
    for d, p in zip(dims, pos):
        fr = 10000.0 ** (-2.0 * torch.arange(d // 2, device=DEV, dtype=torch.float64) / d)
        ang.append(p.double()[:, None] * fr[None, :])
    a = torch.cat(ang, 1)
    return torch.cos(a), torch.sin(a)


class _Exact:
    """F_theta's parts in float64."""

    def __init__(self, case, seed):
        self.case = case
        self.W = dict(_weights(case, seed))

    def lin(self, name, x, rows=None):
        w, b = self.W[name + ".w"], self.W[name + ".b"]
        if rows is not None:
            w, b = w[rows[0]:rows[1]], b[rows[0]:rows[1]]
        return x @ w.double().t() + b.double()

    def cemb(self, t, cond, cam):
        fr = torch.exp(-math.log(10000.0) * torch.arange(128, device=DEV, dtype=torch.float64) / 128)
        arg = 1000.0 * t * fr
        x = torch.nn.functional.silu(self.lin("t_embed.fc1", torch.cat([torch.cos(arg), torch.sin(arg)])))
        y = self.lin("t_embed.fc2", x)
        if cond is not None:
            y = y + self.lin("cond_embed", cond.double())
        if cam is not None:
            y = y + self.lin("cam_embed", cam.double())
        return y

    def qkv(self, name, x, row0):
        """q, k, v [rows, D] of joint rows row0.. with QK-RMSNorm and rotary embedding of the video rows."""
        case, d, hd = self.case, self.case["hidden"], self.case["head_dim"]
        out = []
        for part in range(3):
            y = self.lin(name, x, (part * d, part * d + d))
            if part < 2:
                y = y.view(-1, d // hd, hd)
                y = y / torch.sqrt((y * y).mean(-1, keepdim=True) + 1e-6)
                nv = case["f"] * (case["h"] // 2) * (case["w"] // 2) - row0
                if nv > 0:
                    co, si = (c[row0:row0 + nv, None, :] for c in _rope_table(case))
                    a, b = y[:nv, :, 0::2].clone(), y[:nv, :, 1::2].clone()
                    y[:nv, :, 0::2] = a * co - b * si
                    y[:nv, :, 1::2] = a * si + b * co
                y = y.reshape(-1, d)
            out.append(y)
        return out

    def attn(self, q, k, v):
        hd = self.case["head_dim"]
        out = torch.empty_like(q)
        for i in range(0, q.shape[1], hd):
            out[:, i:i + hd] = _softmax_attention(*(t[:, i:i + hd].contiguous() for t in (q, k, v)))
        return out

    def mlp(self, name, x):
        return torch.nn.functional.gelu(self.lin(name, x), approximate="tanh")

    def block(self, i, x, cemb):
        case, d = self.case, self.case["hidden"]
        act = torch.nn.functional.silu(cemb)
        if case["block"] == "single":
            pre = f"single.{i}"
            sh, sc, g = self.lin(pre + ".ada", act).chunk(3)
            h = _ln(x) * (1 + sc) + sh
            a = self.attn(*self.qkv(pre + ".lin1", h, 0))
            m = torch.nn.functional.gelu(self.lin(pre + ".lin1", h, (3 * d, 7 * d)), approximate="tanh")
            w = self.W[pre + ".lin2.w"]
            y = a @ w[:, :d].double().t() + m @ w[:, d:].double().t() + self.W[pre + ".lin2.b"].double()
            return x + g * y
        nv = case["f"] * (case["h"] // 2) * (case["w"] // 2)
        if case["block"] == "seq":
            parts = [(f"seq.{i}", 0, x.shape[0])]
        else:
            parts = [(f"dual.{i}.vid", 0, nv), (f"dual.{i}.txt", nv, x.shape[0])]
        mods = [self.lin(pre + ".ada", act).chunk(6) for pre, _, _ in parts]
        qkv = [self.qkv(pre + ".qkv", _ln(x[a:b]) * (1 + m[1]) + m[0], a) for (pre, a, b), m in zip(parts, mods)]
        att = self.attn(*(torch.cat([p[j] for p in qkv]) for j in range(3)))
        del qkv
        out = []
        for (pre, a, b), m in zip(parts, mods):
            y = x[a:b] + m[2] * self.lin(pre + ".out", att[a:b])
            h = self.mlp(pre + ".fc1", _ln(y) * (1 + m[4]) + m[3])
            out.append(y + m[5] * self.lin(pre + ".fc2", h))
        return torch.cat(out)

    def forward(self, z, t, cond, text, cam):
        case, d = self.case, self.case["hidden"]
        f, h, w = case["f"], case["h"] // 2, case["w"] // 2
        c = self.cemb(t, cond, cam)
        tok = z.double().view(16, f, h, 2, w, 2).permute(1, 2, 4, 0, 3, 5).reshape(f * h * w, 64)
        x = self.lin("patch_embed", tok)
        if text is not None:
            x = torch.cat([x, self.lin("text_proj", text.double())])
        for i in range(case["blocks"]):
            x = self.block(i, x, c)
        sh, sc = self.lin("final.ada", torch.nn.functional.silu(c)).chunk(2)
        y = self.lin("final.lin", _ln(x[:f * h * w]) * (1 + sc) + sh)
        return y.view(f, h, w, 16, 2, 2).permute(3, 0, 1, 4, 2, 5).reshape(16, f, 2 * h, 2 * w)


class _ExactRollout:
    """Surrogate and risk controller in float64 (lifted summaries, retrieval, evolution, observation, risk)."""

    def __init__(self, case):
        self.c = case
        self.bank, self.inserts = [None] * case["bank"], 0
        self.za = self.h = None
        self.qa = self.qam1 = 0.0
        self.R, self.eta, self.ns = 0.0, 1.0, 0

    @staticmethod
    def pool(x, g):
        x = x.reshape(x.shape[0], -1)
        idx = (torch.arange(x.shape[1], device=DEV) * g) // x.shape[1]
        cnt = torch.bincount(idx, minlength=g).double()
        return (torch.zeros(x.shape[0], g, device=DEV, dtype=torch.float64).index_add_(1, idx, x) / cnt.sqrt()).reshape(-1)

    @staticmethod
    def rho(x):
        return torch.sqrt((x * x).mean() + 1e-6)

    def summary(self, z):
        zero = lambda n: torch.zeros(n, device=DEV, dtype=torch.float64)  # noqa: E731
        d = zero(64) if self.za is None else self.pool((z - self.za) / self.rho(z - self.za), 4)
        return torch.cat([self.pool(z / self.rho(z), 8), d, zero(32) if self.h is None else self.h, zero(32)])

    @staticmethod
    def sim(a, b):
        den = float(a.norm() * b.norm())
        return float(a @ b) / den if den >= 1e-30 else 0.0

    def candidate(self, z, k, steps):
        t, tn = (steps - k) / steps, (steps - k - 1) / steps
        self.s = self.summary(z)
        dz = dph = 0.0
        if self.za is not None:
            dz = float((z - self.za).abs().sum() / (self.za.abs().sum() + 1e-8))
            dph = abs(t - self.qa)
        self.p = dz + 0.05 * (self.ns + 1) / 7 + 0.5 * dph
        self.zhat, self.support, alpha = None, 0, 0.0
        recs = [r for r in self.bank if r is not None]
        if recs:
            if self.c["surrogate"] == "secant":
                r = self.bank[(self.inserts - 1) % self.c["bank"]]
                alpha = (tn - t) / (self.qam1 - self.qa)
                self.zhat, self.support = z + alpha * (r["z"] - self.za), 1
            else:
                sims = [self.sim(self.s, r["s_in"]) for r in recs]
                sup = [j for j, r in enumerate(recs) if sims[j] >= 0.25 and abs(t - r["q"]) <= 0.43]
                lo = [(sims[j] - 10 * (t - recs[j]["q"]) ** 2) / 0.05 for j in sup]
                pi = [math.exp(x - max(lo)) for x in lo]
                pi = [x / sum(pi) for x in pi]
                self.support = len(sup)
                alpha = min(max(abs(tn - t) / (abs(self.qam1 - self.qa) + 1e-8), 0.5), 2.0)
                if self.c["observation"] == "linear":
                    rc = self.rho(z)
                    self.zhat = z.clone()
                    for w, j in zip(pi, sup):
                        r = recs[j]
                        self.zhat += alpha * w * rc * (r["z"] / self.rho(r["z"]) - r["z_in"] / self.rho(r["z_in"]))
                else:
                    sh = self.s.clone()
                    for w, j in zip(pi, sup):
                        sh += alpha * w * (recs[j]["s_out"] - recs[j]["s_in"])
                    ks = [self.sim(sh, r["s_out"]) / 0.02 for r in recs]
                    ka = [math.exp(x - max(ks)) for x in ks]
                    self.zhat = sum(x / sum(ka) * r["z"] for x, r in zip(ka, recs))
        self.avail = bool(recs) and self.ns <= 6 and self.support >= 1 and 1 <= k <= steps - 1
        self.rcand = 0.8 * self.R + min(2.0, 1 + 0.5 * t) * self.eta * self.p
        return dz, alpha

    def exact(self, z, zn, k, steps):
        t, tn = (steps - k) / steps, (steps - k - 1) / steps
        if self.zhat is not None and self.support >= 1:
            dcf = float((zn - self.zhat).abs().mean() / (zn.abs().mean() + 1e-8))
            self.eta = min(max(0.8 * self.eta + 0.2 * dcf / (self.p + 1e-8), 0.05), 20.0)
        self.R *= 0.8
        self.bank[self.inserts % self.c["bank"]] = {"z": zn, "z_in": z, "s_in": self.s, "s_out": self.summary(zn), "q": t}
        self.inserts += 1
        self.h = self.pool((zn - z) / self.rho(zn - z), 2)
        self.za, self.qa, self.qam1, self.ns = z, t, tn, 0

    def run(self, z, v, steps, tau):
        z = z.double()
        sched, log = [], []
        for k in range(steps):
            dz, _ = self.candidate(z, k, steps)
            take = self.avail and self.rcand <= tau
            sched.append(int(take))
            rc = self.rcand
            if take:
                z, self.R, self.ns = self.zhat, rc, self.ns + 1
            else:
                zn = z - v[k].double() / steps
                self.exact(z, zn, k, steps)
                z = zn
            log.append([dz, rc, self.eta, self.R])
        return {"z": z, "schedule": np.array(sched, dtype=np.int64), "log": np.array(log)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("forward", "batch", "block"):
        n, fl = _block_work(case)
        if fl * case["blocks"] * case["batch"] > 1e14:    # over about 20 seconds in float64
            return None
    with torch.no_grad():
        if kind in ("forward", "batch"):
            m, i = _Exact(case, seed), _model_inputs(case, seed)
            out = [m.forward(i["z"][b], 0.6, i["cond"][b], i["text"][b], i["cam"][b]) for b in range(case["batch"])]
            return out if kind == "batch" else out[0]
        if kind == "cond":
            i = _model_inputs(case, seed)
            return _Exact(case, seed).cemb(0.6, i["cond"][0], i["cam"][0])
        if kind == "block":
            x, c = _block_inputs(case, seed)
            return _Exact(case, seed).block(0, x.double(), c.double())
        if kind == "attention":
            q, k, v = (t.double() for t in _attention_inputs(case, seed))
            return torch.cat([_softmax_attention(q[h], k[h], v[h]) for h in range(q.shape[0])], 1)
        if kind == "linear":
            a, w, b = (t.double() for t in _linear_inputs(case, seed))
            return a @ w.t() + b
        m = _ExactRollout(case)
        if kind == "rollout":
            z, v = _trajectory(case, seed, case["steps"])
            return m.run(z, v, case["steps"], case["tau"])
        zs = [z.double() for z in _step_inputs(case, seed)]
        for k in range(case["bank"]):
            m.candidate(zs[k], k, 50)
            m.exact(zs[k], zs[k + 1], k, 50)
        dz, alpha = m.candidate(zs[-1], case["bank"], 50)
        return {"zhat": m.zhat, "exact": int(not (m.avail and m.rcand <= case["tau"])),
                "log": np.array([dz, alpha, m.rcand])}
