"""The workloads this library is timed on: calls that a GRPO training program
makes through the public binding, from the smallest to the largest.

A case is a dict of plain values.  ``kind`` names the calls:

  step       forward of the endpoint pair with saved activations, then the JAGG
             group backward (Phases 1, 3 and 4 of a window)
  window     the JAGG group backward alone, the pair's forward being done
  perstep    the per-step baseline backward of a window (W accumulated VJPs)
  forward    the endpoint pair's forward alone
  linear     the backward of one linear layer: GELU' input gradient and weight
             gradient
  grpo       Phase 2 and 3 fused: composites of the GRPO upstream gradients
  aggregate  Phase 3 alone: composites of W given upstream gradients
  score      routing score of W per-step vectors

Model cases give the network's sizes as ``Config`` names them; ``batch`` is the
rollouts of a window, so the endpoint pair runs as a batch of twice that.
"""
from __future__ import annotations

import math

import torch

import paper_2607_17572_amd as pk

MODEL = ("step", "window", "perstep", "forward")
DT = {"bf16": torch.bfloat16, "fp32": torch.float32}


def _model(name, kind, n_double, n_single, heads, head_dim, n_txt, lat_h, lat_w, batch, W, act="bf16", grad="fp32",
           in_ch=16, patch=2, txt_dim=0, mlp=0, block_only=1, checkpoint=0):
    hidden = heads * head_dim
    return dict(name=name, kind=kind, n_double=n_double, n_single=n_single, heads=heads, head_dim=head_dim,
                mlp=mlp or 4 * hidden, n_txt=n_txt, lat_h=lat_h, lat_w=lat_w, in_ch=in_ch, patch=patch,
                txt_dim=txt_dim or hidden, block_only=block_only, checkpoint=checkpoint, act=act, grad=grad,
                batch=batch, W=W)


def listed():
    return [
        # the smallest network (two double blocks, hidden 64, 24 tokens, fp32): launches and latency decide
        _model("tiny_step_fp32", "step", 2, 0, 4, 16, 8, 4, 4, 1, 4, act="fp32", in_ch=4, patch=1, txt_dim=64,
               block_only=0),
        # a small fp32 block, as parity and debugging runs use: 256 image + 77 text tokens, hidden 512
        _model("block512_step_fp32", "step", 1, 0, 8, 64, 77, 32, 32, 2, 4, act="fp32"),
        # a small bf16 network with 64-wide heads: 256 image + 77 text tokens, hidden 768, four rollouts
        _model("block768_step_h64", "step", 1, 0, 12, 64, 77, 32, 32, 4, 4),
        # odd image and text lengths at middle width: 21 x 17 image + 77 text tokens, hidden 1536, three rollouts
        _model("block1536_step_ragged", "step", 1, 0, 12, 128, 77, 42, 34, 3, 4),
        # one double block of the 1024 x 1024 image (4096 + 512 tokens, hidden 3072): the pair's forward ...
        _model("block4608_forward", "forward", 1, 0, 24, 128, 512, 128, 128, 1, 4),
        # ... its JAGG group backward, the product of this library ...
        _model("block4608_window", "window", 1, 0, 24, 128, 512, 128, 128, 1, 4),
        # ... and the per-step backward that windows routed away from JAGG take
        _model("block4608_perstep", "perstep", 1, 0, 24, 128, 512, 128, 128, 1, 4),
        # a whole network of one double and one single block with embeddings and final layer, 512 x 512 image
        # (1024 + 512 tokens), activation checkpointing, bf16 gradients: a training step's forward and backward
        _model("model1536_step_checkpoint", "step", 1, 1, 24, 128, 512, 64, 64, 1, 8, grad="bf16", txt_dim=4096,
               block_only=0, checkpoint=1),
        # the second MLP layer's backward for a ragged row count (three samples of 363 tokens)
        dict(name="linear_rows1089", kind="linear", rows=1089, n_out=3072, n_in=12288, grad="fp32"),
        # GRPO composites over the block network's outputs, one rollout
        dict(name="grpo_w4", kind="grpo", n_txt=512, n_img=4096, hidden=3072, batch=1, W=4, act="bf16"),
        # composites over latents (16 x 128 x 128, four rollouts): a call of a few microseconds
        dict(name="aggregate_latents_w8", kind="aggregate", n=4 * 16 * 128 * 128, W=8, act="bf16"),
        # routing score of the hidden states of eight steps (4608 x 3072 each)
        dict(name="score_hidden_w8", kind="score", n=4608 * 3072, W=8, act="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "window", "window", "perstep", "forward", "linear", "grpo", "aggregate", "score"])
    if kind == "linear":
        rows = _log_int(rng, 60, 9216)
        return dict(kind=kind, rows=rows, n_out=8 * _log_int(rng, 32, 1152), n_in=8 * _log_int(rng, 32, 1536),
                    grad=rng.choice(["fp32", "bf16"]))
    if kind == "grpo":
        return dict(kind=kind, n_txt=_log_int(rng, 20, 512), n_img=_log_int(rng, 60, 2048),
                    hidden=128 * rng.randint(2, 24), batch=rng.randint(1, 3), W=rng.choice([2, 4, 8]),
                    act=rng.choice(["bf16", "fp32"]))
    if kind in ("aggregate", "score"):
        return dict(kind=kind, n=_log_int(rng, 1 << 14, 1 << 24), W=rng.randint(2, 8),
                    act=rng.choice(["bf16", "bf16", "fp32"]))
    for _ in range(1000):
        act = rng.choice(["bf16", "bf16", "bf16", "fp32"])
        head_dim = rng.choice([128, 128, 128, 64]) if act == "bf16" else rng.choice([16, 32, 64, 128])
        block_only = rng.choice([0, 1])
        c = _model("", kind, rng.randint(1, 2), 0 if block_only else rng.randint(0, 2), rng.randint(2, 24), head_dim,
                   _log_int(rng, 20, 512), 2 * rng.randint(6, 64), 2 * rng.randint(6, 64), rng.randint(1, 4),
                   rng.randint(2, 8), act=act, grad=rng.choice(["fp32", "bf16"]), txt_dim=64 * rng.randint(4, 64),
                   block_only=block_only, checkpoint=rng.choice([0, 0, 1]))
        del c["name"]
        # below the listed cases' cost: the 4608-token backward for 128-wide bf16 heads, the small ones otherwise
        most = 5e12 if act == "bf16" and head_dim == 128 else 1.2e11
        if c["heads"] * head_dim <= 3072 and work(c)["flops"] < most:
            return c
    raise AssertionError("no case of the range fits")


# ------------------------------------------------------------------ sizes
def _cfg(c):
    return pk.Config(n_double=c["n_double"], n_single=c["n_single"], hidden=c["heads"] * c["head_dim"],
                     heads=c["heads"], head_dim=c["head_dim"], mlp_hidden=c["mlp"], in_ch=c["in_ch"],
                     patch=c["patch"], lat_h=c["lat_h"], lat_w=c["lat_w"], n_txt=c["n_txt"], txt_dim=c["txt_dim"],
                     t_freq_dim=256, block_only=c["block_only"], act_dtype=pk.BF16 if c["act"] == "bf16" else pk.F32,
                     grad_dtype=pk.BF16 if c["grad"] == "bf16" else pk.F32, checkpoint=c["checkpoint"])


def _shapes(c):
    """[(name, shape)] of the parameters, in the flat buffer's order (each starts at a multiple of 128 elements)."""
    D, Dh, F, pd = c["heads"] * c["head_dim"], c["head_dim"], c["mlp"], c["in_ch"] * c["patch"] ** 2
    out = []

    def lin(name, o, i):
        out.append((name + ".w", (o, i)))
        out.append((name + ".b", (o,)))

    lin("t_in", D, 256)
    lin("t_out", D, D)
    if not c["block_only"]:
        lin("img_in", D, pd)
        lin("txt_in", D, c["txt_dim"])
    for i in range(c["n_double"]):
        for s in ("txt", "img"):
            p = f"double.{i}.{s}."
            lin(p + "mod", 6 * D, D)
            lin(p + "qkv", 3 * D, D)
            out += [(p + "q_gain", (Dh,)), (p + "k_gain", (Dh,))]
            lin(p + "o", D, D)
            lin(p + "fc1", F, D)
            lin(p + "fc2", D, F)
    for i in range(c["n_single"]):
        p = f"single.{i}."
        lin(p + "mod", 3 * D, D)
        lin(p + "in", 3 * D + F, D)
        out += [(p + "q_gain", (Dh,)), (p + "k_gain", (Dh,))]
        lin(p + "out", D, D + F)
    if not c["block_only"]:
        lin("final.mod", 2 * D, D)
        lin("final", pd, D)
    return out


def _n_img(c):
    return (c["lat_h"] // c["patch"]) * (c["lat_w"] // c["patch"])


def _t(c):
    """Timesteps of the window: t_k = 1 - k / T on a 16-step (or longer) grid."""
    T = max(16, c["W"] + 1)
    return [1.0 - k / T for k in range(c["W"] + (1 if c["kind"] == "grpo" else 0))]


def work(c):
    es = 2 if c.get("act") == "bf16" else 4
    if c["kind"] == "linear":
        r, o, i, gs = c["rows"], c["n_out"], c["n_in"], 4 if c["grad"] == "fp32" else 2
        return {"bytes": 2 * (r * o + o * i + 3 * r * i) + gs * o * i, "flops": 4 * r * o * i}
    if c["kind"] == "grpo":
        n = c["batch"] * (c["n_txt"] + c["n_img"]) * c["hidden"]
        return {"bytes": (2 * c["W"] + 3) * n * es, "flops": 0}
    if c["kind"] == "aggregate":
        return {"bytes": (c["W"] + 2) * c["n"] * es, "flops": 0}
    if c["kind"] == "score":
        return {"bytes": c["W"] * c["n"] * es, "flops": 0}
    D, F, N = c["heads"] * c["head_dim"], c["mlp"], c["n_txt"] + _n_img(c)
    par = sum(math.prod(s) for _, s in _shapes(c))
    nblk = c["n_double"] + c["n_single"]
    lin = 2 * N * nblk * (4 * D * D + 2 * D * F)          # a block's products, per sample
    if not c["block_only"]:
        lin += 2 * D * (c["n_txt"] * c["txt_dim"] + 2 * _n_img(c) * c["in_ch"] * c["patch"] ** 2)
    att = 4 * N * N * D * nblk
    fwd, bwd = lin + att, 2 * lin + 2 * att + (lin + att if c["checkpoint"] else 0)
    io = 2 * es * N * (D if c["block_only"] else 0)
    saved = es * N * ((13 * D + 2 * F) * nblk if not c["checkpoint"] else D * (nblk + 1))
    gs = 4 if c["grad"] == "fp32" else 2
    B2, B, W = 2 * c["batch"], c["batch"], c["W"]
    if c["kind"] == "forward":
        return {"bytes": par * es + B2 * (io + saved), "flops": B2 * fwd}
    if c["kind"] == "window":
        return {"bytes": par * (es + gs) + B2 * saved + W * B * io / 2, "flops": B2 * bwd}
    if c["kind"] == "perstep":
        return {"bytes": par * (es + gs) + W * B * (saved + io / 2), "flops": W * B * bwd}
    return {"bytes": par * (es + gs) + B2 * (io + 2 * saved) + W * B * io / 2, "flops": B2 * (fwd + bwd)}


# ----------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, dt, std=1.0):
    return torch.randn(shape, generator=g, device="cuda").mul_(std).to(dt)


def _model_inputs(c, seed):
    """theta (flat), per-step inputs z_j (and text), upstream gradients s_j."""
    dt, g = DT[c["act"]], _gen(seed)
    layout, total = pk.param_layout(_cfg(c))
    theta = _normal(g, (total,), dt, 0.02)
    for name, off, n, _, _ in layout:
        if name.endswith("_gain"):
            theta[off:off + n] = 1.0 + _normal(g, (n,), torch.float32, 0.02)
    B, W, D, nt, ni = c["batch"], c["W"], c["heads"] * c["head_dim"], c["n_txt"], _n_img(c)
    if c["block_only"]:
        shape, txt = (B * (nt + ni), D), None
    else:
        shape, txt = (B, c["in_ch"], c["lat_h"], c["lat_w"]), _normal(g, (B, nt, c["txt_dim"]), dt)
    z = [_normal(g, shape, dt) for _ in range(W if c["kind"] == "perstep" else 2)]
    adv = _normal(g, (B,), torch.float32)
    if c["block_only"]:
        scale = torch.cat([adv.repeat_interleave(nt), adv.repeat_interleave(ni)])[:, None]
    else:
        scale = adv[:, None, None, None]
    s = [(_normal(g, shape, torch.float32) * scale).to(dt) for _ in range(W)]
    return theta, z, txt, s


def _pair(c, z, txt):
    """The endpoint pair as one batch (endpoint 0 first; block-only rows are stream-major)."""
    if not c["block_only"]:
        return torch.cat([z[0], z[-1]]), torch.cat([txt, txt])
    k = c["batch"] * c["n_txt"]
    return torch.cat([z[0][:k], z[-1][:k], z[0][k:], z[-1][k:]]), None


def _grpo_inputs(c, seed):
    """Model outputs, latents, sigma, old log-probabilities and advantages of one window."""
    dt, g, W, B, D = DT[c["act"]], _gen(seed), c["W"], c["batch"], c["hidden"]
    shape = (B * (c["n_txt"] + c["n_img"]), D)
    v = [_normal(g, shape, dt) for _ in range(W)]
    z = [_normal(g, shape, dt) for _ in range(W + 1)]
    adv = _normal(g, (B,), torch.float32)
    t, sigma = _t(c), [0.3] * W
    t32 = torch.tensor(t, dtype=torch.float32).double().tolist()
    s32 = torch.tensor(sigma, dtype=torch.float32).double().tolist()
    logp = torch.stack([_log_prob(c, z[j], z[j + 1], v[j], t32[j + 1] - t32[j], s32[j])[0] for j in range(W)])
    old = logp - 0.1 * torch.randn((W, B), generator=g, device="cuda", dtype=torch.float64)
    return v, z, t, sigma, old.contiguous(), adv


def _per_sample(c, x):
    """Sum of the rows of each sample of a stream-major [rows] vector."""
    B, k = c["batch"], c["batch"] * c["n_txt"]
    return x[:k].reshape(B, -1).sum(1) + x[k:].reshape(B, -1).sum(1)


def _log_prob(c, z, zn, v, dt, sigma):
    d = zn.double() - z.double() - v.double() * dt
    n = (c["n_txt"] + c["n_img"]) * c["hidden"]
    sq = _per_sample(c, (d * d).sum(1))
    return -sq / (2 * sigma * sigma) - n * math.log(math.sqrt(2 * math.pi) * sigma), d


def prepare(c, seed):
    if c["kind"] == "linear":
        g = _gen(seed)
        r, o, i = c["rows"], c["n_out"], c["n_in"]
        ctx = pk.Context(_cfg(listed()[3]))  # any network: the call takes its sizes from the operands
        return dict(c=c, ctx=ctx, dY=_normal(g, (r, o), torch.bfloat16), X=_normal(g, (r, i), torch.bfloat16),
                    Wt=_normal(g, (o, i), torch.bfloat16, 0.02), pre=_normal(g, (r, i), torch.bfloat16),
                    dX=torch.empty((r, i), dtype=torch.bfloat16, device="cuda"),
                    dW=torch.empty((o, i), dtype=DT[c["grad"]], device="cuda"))
    if c["kind"] == "grpo":
        D = c["hidden"]
        cfg = pk.Config(n_double=1, n_single=0, hidden=D, heads=D // 128, head_dim=128, mlp_hidden=4 * D, in_ch=16,
                        patch=1, lat_h=c["n_img"], lat_w=1, n_txt=c["n_txt"], txt_dim=D, block_only=1,
                        act_dtype=pk.BF16 if c["act"] == "bf16" else pk.F32)
        v, z, t, sigma, old, adv = _grpo_inputs(c, seed)
        ctx = pk.Context(cfg)
        ctx.ensure_workspace(1)
        return dict(c=c, ctx=ctx, v=v, z=z, t=t, sigma=sigma, old=old, adv=adv, base=torch.empty_like(v[0]),
                    corr=torch.empty_like(v[0]), stats=torch.zeros((c["W"], c["batch"], 3), dtype=torch.float64,
                                                                  device="cuda"))
    if c["kind"] in ("aggregate", "score"):
        g = _gen(seed)
        # steps of one window share a direction: x_j = u + 0.7 e_j
        u = _normal(g, (c["n"],), torch.float32)
        x = [(u + _normal(g, (c["n"],), torch.float32, 0.7)).to(DT[c["act"]]) for _ in range(c["W"])]
        ctx = pk.Context(_cfg(listed()[3]))
        ctx.ensure_workspace(1)
        return dict(c=c, ctx=ctx, x=x, t=_t(c), base=torch.empty_like(x[0]), corr=torch.empty_like(x[0]))
    theta, z, txt, s = _model_inputs(c, seed)
    ctx = pk.Context(_cfg(c))
    B, t = c["batch"], _t(c)
    st = dict(c=c, ctx=ctx, theta=theta, s=s, t=t)
    if c["kind"] != "forward":
        st["dtheta"] = torch.zeros(ctx.n_params, dtype=ctx.grad_dtype, device="cuda")
    if c["kind"] == "perstep":
        ctx.ensure_workspace(B)
        st["saved"] = [ctx.new_saved(B) for _ in range(c["W"])]
        for j in range(c["W"]):
            ctx.forward_save(theta, z[j], [t[j]] * B, txt, saved=st["saved"][j])
        return st
    ctx.ensure_workspace(2 * B)
    st["z"], st["txt"] = _pair(c, z, txt)
    st["v"], st["saved"] = torch.empty_like(st["z"]), ctx.new_saved(2 * B)
    if c["kind"] == "window":
        ctx.forward_save(theta, st["z"], [t[0]] * B + [t[-1]] * B, st["txt"], saved=st["saved"], v_out=st["v"])
    return st


def run(st):
    c, ctx = st["c"], st["ctx"]
    kind, B = c["kind"], c.get("batch", 1)
    if kind == "linear":
        ctx.linear_grad(pk.DGRAD_GELU, st["dY"], st["Wt"], st["dX"], pre=st["pre"])
        ctx.linear_grad(pk.WGRAD, st["dY"], st["X"], st["dW"])
        return {"dX": st["dX"], "dW": st["dW"]}
    if kind == "grpo":
        ctx.grpo_composites(st["v"], st["z"], st["t"], st["sigma"], st["old"], st["adv"], st["base"], st["corr"],
                            stats=st["stats"])
        return {"base": st["base"], "corr": st["corr"], "stats": st["stats"]}
    if kind == "aggregate":
        ctx.aggregate(st["x"], st["t"], st["base"], st["corr"])
        return {"base": st["base"], "corr": st["corr"]}
    if kind == "score":
        return {"score": ctx.group_score(st["x"])}
    if kind == "perstep":
        return {"dtheta": ctx.perstep_group_backward(st["theta"], st["saved"], B, st["s"], st["dtheta"])}
    out = {}
    if kind in ("step", "forward"):
        tt = [st["t"][0]] * B + [st["t"][-1]] * B
        out["v"] = ctx.forward_save(st["theta"], st["z"], tt, st["txt"], saved=st["saved"], v_out=st["v"])
    if kind in ("step", "window"):
        out["dtheta"] = ctx.group_backward(st["theta"], st["saved"], B, st["s"], st["t"], st["dtheta"])
    return out


def tolerance(c):
    """About four times the distance from 64 bits that the ranges show (relative 2-norm; largest difference)."""
    if c["kind"] == "score":
        return {"rel": 1e-12}  # fp64 sums of exact products
    if c["kind"] in ("grpo", "aggregate"):  # fp32 sums, one rounding on store
        return {"rel": 1e-6, "max": 1e-5} if c["act"] == "fp32" else {"rel": 2e-3, "max": 1e-2}
    if c["kind"] == "linear":
        return {"rel": 7e-3, "max": 1.6e-2}
    if c["act"] == "fp32":
        return {"rel": 4e-6, "max": 4e-4}
    if c["kind"] == "forward":
        return {"rel": 1.6e-2, "max": 8e-2}
    return {"rel": 1.6e-2, "max": 0.99}  # a flat gradient: its tensors' scales differ by orders of magnitude


# ------------------------------------------- the same in 64 bits, plain torch
def _silu(x):
    return x * torch.sigmoid(x)


def _gelu(x):
    return 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))


def _ln(x):
    m = x.mean(-1, keepdim=True)
    return (x - m) * torch.rsqrt(((x - m) ** 2).mean(-1, keepdim=True) + 1e-6)


def _rms(x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-6) * gain


def _rotate(x, ang):
    a, b, co, si = x[..., 0::2], x[..., 1::2], torch.cos(ang), torch.sin(ang)
    return torch.stack([a * co - b * si, a * si + b * co], -1).flatten(-2)


def _angles(c):
    q = c["head_dim"] // 4
    f = 1e4 ** (-torch.arange(q, dtype=torch.float64, device="cuda") * 2 / (c["head_dim"] // 2))
    gw, n = c["lat_w"] // c["patch"], torch.arange(_n_img(c), device="cuda")
    zero = torch.zeros(c["n_txt"], dtype=torch.float64, device="cuda")
    r, col = torch.cat([zero, (n // gw).double()]), torch.cat([zero, (n % gw).double()])
    return torch.cat([r[:, None] * f, col[:, None] * f], 1)


def _attention(c, qkv, gains, ang):
    """qkv [N][3D] of one sample, gains: per token row; returns [N][D]."""
    D, Dh, out = c["heads"] * c["head_dim"], c["head_dim"], []
    for h in range(c["heads"]):
        q, k, v = (qkv[:, i * D + h * Dh:i * D + (h + 1) * Dh] for i in range(3))
        q, k = _rotate(_rms(q, gains[0]), ang), _rotate(_rms(k, gains[1]), ang)
        out.append(torch.softmax((q / math.sqrt(Dh)) @ k.t(), -1) @ v)
    return torch.cat(out, 1)


def _sample(c, P, z, txt, t, ang):
    """v of one sample; z: (text rows, image rows) or a latent."""
    D, nt, p = c["heads"] * c["head_dim"], c["n_txt"], c["patch"]

    def lin(name, x):
        return x @ P[name + ".w"].t() + P[name + ".b"]

    w = 1e4 ** (-torch.arange(128, dtype=torch.float64, device="cuda") / 128)
    temb = torch.cat([torch.cos(1000 * t * w), torch.sin(1000 * t * w)])
    vec = _silu(lin("t_out", _silu(lin("t_in", temb))))
    if c["block_only"]:
        x = list(z)
    else:
        gh, gw = c["lat_h"] // p, c["lat_w"] // p
        pt = z.reshape(c["in_ch"], gh, p, gw, p).permute(1, 3, 0, 2, 4).reshape(gh * gw, -1)
        x = [lin("txt_in", txt), lin("img_in", pt)]
    for i in range(c["n_double"]):
        pre = [f"double.{i}.{s}." for s in ("txt", "img")]
        mod = [lin(q + "mod", vec).chunk(6) for q in pre]
        qkv = torch.cat([lin(q + "qkv", _ln(x[s]) * (1 + mod[s][1]) + mod[s][0]) for s, q in enumerate(pre)])
        rows = [len(x[0]), len(x[1])]
        gains = [torch.cat([P[q + g].expand(n, -1) for q, n in zip(pre, rows)]) for g in ("q_gain", "k_gain")]
        o = _attention(c, qkv, gains, ang).split(rows)
        for s, q in enumerate(pre):
            xm = x[s] + mod[s][2] * lin(q + "o", o[s])
            x[s] = xm + mod[s][5] * lin(q + "fc2", _gelu(lin(q + "fc1", _ln(xm) * (1 + mod[s][4]) + mod[s][3])))
    if c["block_only"]:
        return x
    x = torch.cat(x)
    for i in range(c["n_single"]):
        q = f"single.{i}."
        mod = lin(q + "mod", vec).chunk(3)
        y = lin(q + "in", _ln(x) * (1 + mod[1]) + mod[0])
        o = _attention(c, y[:, :3 * D], (P[q + "q_gain"], P[q + "k_gain"]), ang)
        x = x + mod[2] * lin(q + "out", torch.cat([o, _gelu(y[:, 3 * D:])], 1))
    mod = lin("final.mod", vec).chunk(2)
    y = lin("final", _ln(x[nt:]) * (1 + mod[1]) + mod[0])
    return y.reshape(gh, gw, c["in_ch"], p, p).permute(2, 0, 3, 1, 4).reshape(c["in_ch"], c["lat_h"], c["lat_w"])


def _rows_of(c, x, b, B):
    nt, ni = c["n_txt"], _n_img(c)
    return x[b * nt:(b + 1) * nt], x[B * nt + b * ni:B * nt + (b + 1) * ni]


def _weights(t):
    t = torch.tensor(t, dtype=torch.float32).double()
    a = (t[0] - t) / (t[0] - t[-1])
    return (1 - a).tolist(), a.tolist()


def _exact_model(c, seed):
    theta, z, txt, s = _model_inputs(c, seed)
    B, t, off, P = c["batch"], _t(c), 0, {}
    flat = torch.zeros_like(theta, dtype=torch.float64)
    for name, shape in _shapes(c):
        n = math.prod(shape)
        P[name] = theta[off:off + n].double().reshape(shape).requires_grad_(c["kind"] != "forward")
        off += -(-n // 128) * 128
    ang = _angles(c)
    if c["kind"] == "perstep":
        points = [(j, t[j], s[j].double()) for j in range(c["W"])]
    else:
        wb, wc = _weights(t)
        points = [(0, t[0], sum(w * x.double() for w, x in zip(wb, s))),
                  (1, t[-1], sum(w * x.double() for w, x in zip(wc, s)))]
    vs = []
    for j, tj, cot in points:
        for b in range(B):
            if c["block_only"]:
                v = _sample(c, P, [x.double() for x in _rows_of(c, z[j], b, B)], None, tj, ang)
                u = _rows_of(c, cot, b, B)
            else:
                v, u = [_sample(c, P, z[j][b].double(), txt[b].double(), tj, ang)], [cot[b]]
            vs.append([x.detach() for x in v])
            if c["kind"] != "forward":
                torch.autograd.backward(v, u)  # adds into .grad: the sum over samples and points
    out = {}
    if c["kind"] in ("step", "forward"):
        if c["block_only"]:
            out["v"] = torch.cat([x[0] for x in vs] + [x[1] for x in vs])
        else:
            out["v"] = torch.stack([x[0] for x in vs])
    if c["kind"] != "forward":
        off = 0
        for name, shape in _shapes(c):
            n = math.prod(shape)
            if P[name].grad is not None:
                flat[off:off + n] = P[name].grad.reshape(-1)
            off += -(-n // 128) * 128
        out["dtheta"] = flat
    return out


def exact(c, seed):
    if c["kind"] in MODEL:
        return _exact_model(c, seed)
    if c["kind"] == "linear":
        g = _gen(seed)
        r, o, i = c["rows"], c["n_out"], c["n_in"]
        dY, X = _normal(g, (r, o), torch.bfloat16).double(), _normal(g, (r, i), torch.bfloat16).double()
        Wt, pre = _normal(g, (o, i), torch.bfloat16, 0.02).double(), _normal(g, (r, i), torch.bfloat16).double()
        pre.requires_grad_(True)
        d, = torch.autograd.grad(_gelu(pre).sum(), pre)
        return {"dX": (dY @ Wt) * d, "dW": dY.t().contiguous() @ X}
    if c["kind"] == "grpo":
        v, z, t, sigma, old, adv = _grpo_inputs(c, seed)
        W, B, k = c["W"], c["batch"], c["batch"] * c["n_txt"]
        wb, wc = _weights(t[:W])
        t = torch.tensor(t, dtype=torch.float32).double().tolist()
        sigma = torch.tensor(sigma, dtype=torch.float32).double().tolist()
        A = adv.double().clamp(-5.0, 5.0)
        base, corr, stats = 0, 0, []
        for j in range(W):
            dt = t[j + 1] - t[j]
            lp, d = _log_prob(c, z[j], z[j + 1], v[j], dt, sigma[j])
            rho = torch.exp(lp - old[j])
            eps = float(torch.tensor(0.1, dtype=torch.float32))
            plain, clipped = -A * rho, -A * rho.clamp(1 - eps, 1 + eps)
            stats.append(torch.stack([lp, rho, torch.maximum(plain, clipped) / W], 1))
            co = torch.where(clipped > plain, torch.zeros_like(A), -A / W) * rho * dt / sigma[j] ** 2
            row = torch.cat([co.repeat_interleave(c["n_txt"]), co.repeat_interleave(c["n_img"])])
            base, corr = base + wb[j] * row[:, None] * d, corr + wc[j] * row[:, None] * d
        return {"base": base, "corr": corr, "stats": torch.stack(stats)}
    st = prepare(c, seed)
    x = [v.double() for v in st["x"]]
    if c["kind"] == "aggregate":
        wb, wc = _weights(st["t"])
        return {"base": sum(w * v for w, v in zip(wb, x)), "corr": sum(w * v for w, v in zip(wc, x))}
    cos = [float((x[i] @ x[j]) / (x[i].norm() * x[j].norm())) for i in range(len(x)) for j in range(i)]
    return {"score": sum(cos) / len(cos)}
