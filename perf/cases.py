"""The workloads this library's speed is measured on.

Every case is one call (or the short sequence of calls) that a program using the
library makes through `paper_2607_06631_amd.binding`: whole denoise steps and
rollouts, single transformer blocks at the two model widths from a thumbnail to
the full 480x832, 81-frame latent, the switch to another step's structure, the
text cache of a prompt, the timestep embedding, and the two operators.

  listed()            the named cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) what a program holds before the call (inputs, weights, plans)
  run(state)          one pass; returns its outputs
  work(case)          bytes and flops one pass cannot do without
  tolerance(case)     how far another correct implementation may be off
  exact(case, seed)   what run() returns, in float64 by plain torch
"""
import math
import types

import numpy as np
import torch

from paper_2607_06631_amd import binding as B

# Model widths: the tiny float32 stack, the Wan-1.3B and the Wan-14B shapes.
WIDTHS = {
    "tiny": dict(dim=256, heads=4, head_dim=64, ffn=1024),
    "1.3b": dict(dim=1536, heads=12, head_dim=128, ffn=8960),
    "14b": dict(dim=5120, heads=40, head_dim=128, ffn=13824),
}
TIMESTEPS = (999, 750, 500, 250)
PATCH, FREQ, EPS, THETA = 64, 256, 1e-6, 10000.0


def _case(kind, width, grid, text, dtype="bf16", batch=1, layers=1, self_heads=None,
          cross_heads=None, ffn_keep=None, chunk=8, plan="compact", cached=False, step=1, name=None):
    w = WIDTHS[width]
    c = dict(kind=kind, width=width, frames=grid[0], rows=grid[1], cols=grid[2], text=text,
             dtype=dtype, batch=batch, layers=layers,
             self_heads=w["heads"] if self_heads is None else self_heads,
             cross_heads=w["heads"] if cross_heads is None else cross_heads,
             ffn_keep=w["ffn"] if ffn_keep is None else ffn_keep,
             chunk=chunk, plan=plan, cached=cached, step=step)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest whole call: one step of the tiny float32 two-layer stack
        # (128 tokens, 16 text tokens).  Launches and latency only.
        _case("step", "tiny", (2, 8, 8), 16, dtype="f32", layers=2, self_heads=3, cross_heads=3,
              ffn_keep=768, name="step_tiny_f32"),
        # Few-step generation of a still 480x832 picture (one latent frame): the
        # four-step re-noise rollout with the prompt's text cache, two layers.
        _case("rollout", "1.3b", (1, 30, 52), 512, layers=2, self_heads=9, cross_heads=9,
              ffn_keep=6720, cached=True, name="rollout_1.3b_still"),
        # One block of the 1.3B width on the full 480p, 81-frame latent.
        _case("block", "1.3b", (21, 30, 52), 512, self_heads=9, cross_heads=9, ffn_keep=6720,
              name="block_1.3b_480p"),
        # The same for the 14B width, the third step's structure, whose 9677
        # kept channels are not whole chunks: the largest case.
        _case("block", "14b", (21, 30, 52), 512, self_heads=28, cross_heads=28, ffn_keep=9677,
              chunk=1, step=2, name="block_14b_480p"),
        # One 14B block of a still picture, weights read in place through the
        # step's index tables (no gathered copy), odd head counts.
        _case("block", "14b", (1, 30, 52), 512, self_heads=27, cross_heads=31, ffn_keep=11712,
              plan="indexed", name="block_14b_still_indexed"),
        # A guidance pair (two samples) of a short clip, text from the cache.
        _case("block", "1.3b", (5, 30, 52), 512, batch=2, self_heads=10, cross_heads=11,
              ffn_keep=7616, cached=True, name="block_1.3b_pair_clip"),
        # The float32 path at the 1.3B width on a small clip with a short
        # prompt and per-channel FFN masks.
        _case("block", "1.3b", (3, 15, 26), 77, dtype="f32", self_heads=9, cross_heads=10,
              ffn_keep=6721, chunk=1, name="block_1.3b_small_f32"),
        # The engine moves on to another step on a memory budget: that step's
        # weights are gathered and the step is run, here on a thumbnail.
        _case("switch", "14b", (1, 15, 26), 512, self_heads=32, cross_heads=30, ffn_keep=11056,
              name="switch_14b_thumbnail"),
        # A new prompt arrives: the text keys and values of two 14B layers.
        _case("text", "14b", (1, 1, 1), 512, layers=2, name="text_cache_14b"),
        # The timestep embedding and modulation of a 14B step.
        _case("time", "14b", (1, 1, 1), 1, name="time_embed_14b"),
        # The attention operator as the blocks launch it, 720p still picture
        # (45 x 80 tokens), all 40 heads.
        dict(kind="attention", dtype="bf16", head_dim=128, heads=40, batch=1, lq=3600, lk=3600,
             prescaled=True, name="attention_720p_still"),
        # The matrix product operator: an FFN's first half over a ragged batch
        # of rows.
        dict(kind="gemm", dtype="bf16", out="bf16", m=1999, n=8960, k=1536, epilogue=1,
             name="gemm_ffn_ragged"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, most):
    while True:
        g = (rng.choice((1, 1, 2, 3, 5, 9, 13, 21)), _log_int(rng, 6, 45), _log_int(rng, 8, 80))
        if 48 <= g[0] * g[1] * g[2] <= most:
            return g


def draw(rng):
    pick = rng.random()
    if pick < 0.12:
        dtype = rng.choice(("bf16", "bf16", "f32"))
        hd = 128 if dtype == "bf16" else rng.choice((64, 128))
        lq = _log_int(rng, 60, 16000 if dtype == "bf16" else 3000)
        return dict(kind="attention", dtype=dtype, head_dim=hd, heads=rng.randint(4, 40),
                    batch=rng.choice((1, 1, 2)), lq=lq, lk=rng.choice((lq, _log_int(rng, 8, 512))),
                    prescaled=rng.random() < 0.7)
    if pick < 0.24:
        dtype = rng.choice(("bf16", "bf16", "f32"))
        return dict(kind="gemm", dtype=dtype, out=rng.choice((dtype, "f32")),
                    m=_log_int(rng, 60, 16000 if dtype == "bf16" else 4000), n=_log_int(rng, 60, 13824),
                    k=64 * rng.randint(1, 120), epilogue=rng.choice((0, 1, 2)))
    kind = rng.choice(("block", "block", "block", "block", "step", "rollout", "switch", "text", "time"))
    width = rng.choice(("tiny", "1.3b", "1.3b", "14b", "14b"))
    dtype = "f32" if width == "tiny" else "bf16"
    if width == "1.3b" and rng.random() < 0.25:
        dtype = "f32"
    most = {"tiny": 4000, "1.3b": 32760, "14b": 16000}[width]
    if dtype == "f32":
        most = min(most, 3000)
    if kind in ("rollout", "switch"):
        most = min(most, 3600)
    w = WIDTHS[width]
    chunk = rng.choice((8, 8, 1))
    ffn = rng.randint(int(0.4 * w["ffn"]), w["ffn"])
    if chunk == 8:
        ffn = max(8, ffn // 8 * 8)
    c = _case(kind, width, _grid(rng, most), _log_int(rng, 8, 512), dtype=dtype,
              batch=rng.choice((1, 1, 1, 2)), layers=rng.choice((1, 2)) if kind != "block" else 1,
              self_heads=rng.randint(max(1, int(0.4 * w["heads"])), w["heads"]),
              cross_heads=rng.randint(max(1, int(0.4 * w["heads"])), w["heads"]),
              ffn_keep=ffn, chunk=chunk, plan=rng.choice(("compact", "compact", "indexed")),
              cached=rng.random() < 0.4, step=rng.randint(0, 3))
    if kind in ("text", "time"):
        c.update(frames=1, rows=1, cols=1)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

class _Draws:
    """Seeded tensors on the GPU, each from a stream of its own."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.seed, self.n = seed, 0

    def __call__(self, shape, std=1.0, mean=0.0, dtype=torch.float32):
        self.gen.manual_seed(self.seed * 1000003 + self.n)
        self.n += 1
        t = torch.randn(shape, generator=self.gen, device="cuda")
        return t.mul_(std).add_(mean).to(dtype)


def _dtype(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _config(c):
    w = WIDTHS[c["width"]]
    return types.SimpleNamespace(
        dim=w["dim"], n_heads=w["heads"], head_dim=w["head_dim"], ffn_dim=w["ffn"],
        n_layers=c["layers"], patch_dim=PATCH, freq_dim=FREQ,
        grid=(c["frames"], c["rows"], c["cols"]), text_len=max(512, c["text"]), dtype=c["dtype"],
        eps=EPS, rope_theta=THETA)


def _weights(cfg, draws, gain):
    """Random weights of the architecture: matrices and biases N(0, 0.02), the
    patch embedding wider so the residual stream starts at unit scale.  `gain`
    is the mean of the query and key gains: 1.7 for single blocks, whose scores
    then spread as in a trained model (standard deviation about 3) and whose
    result depends on the attention; 1 for whole calls, where every layer after
    would otherwise amplify the 16-bit rounding of the ones before."""
    D, F, m = cfg.dim, cfg.ffn_dim, _dtype(cfg.dtype)
    mat = lambda *s: draws(s, 0.02, dtype=m)
    vec = lambda *s: draws(s, 0.02)
    w = {"patch_w": draws((D, PATCH), 0.125, dtype=m), "patch_b": vec(D), "t_w1": mat(D, FREQ), "t_b1": vec(D),
         "t_w2": mat(D, D), "t_b2": vec(D), "t_w3": mat(6 * D, D), "t_b3": vec(6 * D),
         "head_mod": vec(2, D), "head_w": mat(PATCH, D), "head_b": vec(PATCH), "layers": []}
    for _ in range(cfg.n_layers):
        lw = {"mod": draws((6, D), 0.1)}
        for pre in ("self", "cross"):
            for x in "qkvo":
                lw[pre + "_w" + x] = mat(D, D)
                lw[pre + "_b" + x] = vec(D)
            for x in "qk":
                lw[pre + "_g" + x] = draws((D,), 0.02, gain)
        lw["norm3_w"], lw["norm3_b"] = draws((D,), 0.02, 1.0), vec(D)
        lw["ffn_w1"], lw["ffn_b1"] = mat(F, D), vec(F)
        lw["ffn_w2"], lw["ffn_b2"] = mat(D, F), vec(D)
        w["layers"].append(lw)
    return w


def _masks(c, cfg, seed, step):
    """Keep masks with the case's counts; other steps of a rollout keep a little
    more or less (the outer steps more, as the method's structures do)."""
    g = np.random.Generator(np.random.PCG64([seed, step, 77]))
    N, H, F, chunk = cfg.n_layers, cfg.n_heads, cfg.ffn_dim, c["chunk"]
    more = 1.0 if c["kind"] != "rollout" else (1.2, 1.0, 0.95, 1.2)[step]

    def keep(n, k):
        m = np.zeros(n, np.uint8)
        m[g.permutation(n)[:max(1, min(n, int(round(k * more))))]] = 1
        return m

    return {"block_keep": np.ones(N, np.uint8),
            "self_head_keep": np.stack([keep(H, c["self_heads"]) for _ in range(N)]),
            "cross_head_keep": np.stack([keep(H, c["cross_heads"]) for _ in range(N)]),
            "ffn_keep": np.stack([np.repeat(keep(F // chunk, c["ffn_keep"] // chunk), chunk)
                                  for _ in range(N)])}


def _inputs(c, seed):
    draws = _Draws(seed)
    s = {"case": c}
    if c["kind"] == "gemm":
        d, o = _dtype(c["dtype"]), _dtype(c["out"])
        s["a"], s["b"] = draws((c["m"], c["k"]), dtype=d), draws((c["n"], c["k"]), 0.02, dtype=d)
        s["bias"] = draws((c["n"],), 0.02)
        s["c0"] = draws((c["m"], c["n"]), dtype=o)
        s["gate"] = draws((c["n"],), 0.5)
        return s
    if c["kind"] == "attention":
        d, w = _dtype(c["dtype"]), c["heads"] * c["head_dim"]
        # scores of standard deviation 2.5
        std = 2.5 * (math.log2(math.e) / math.sqrt(c["head_dim"]) if c["prescaled"] else 1.0)
        s["q"] = draws((c["batch"] * c["lq"], w), std, dtype=d)
        s["k"] = draws((c["batch"] * c["lk"], w), dtype=d)
        s["vt"] = draws((c["batch"] * w, -(-c["lk"] // 64) * 64), dtype=d)
        s["vt"][:, c["lk"]:] = 0
        return s
    cfg = _config(c)
    L, D = c["frames"] * c["rows"] * c["cols"], cfg.dim
    s["cfg"], s["weights"] = cfg, _weights(cfg, draws, 1.7 if c["kind"] == "block" else 1.0)
    s["ctx"] = draws((c["batch"], c["text"], D), dtype=_dtype(c["dtype"]))
    steps = range(4) if c["kind"] == "rollout" else (c["step"],)
    s["masks"] = {i: _masks(c, cfg, seed, i) for i in steps}
    if c["kind"] == "block":
        s["x0"] = draws((c["batch"], L, D), dtype=_dtype(c["dtype"]))
        s["e0"] = draws((6, D), 0.5)
    elif c["kind"] in ("step", "rollout", "switch"):
        s["z0"] = draws((c["batch"], L, PATCH))
        if c["kind"] == "rollout":
            s["eps"] = [draws((c["batch"], L, PATCH)) for _ in range(3)]
    return s


# ---------------------------------------------------------------------------
# the library's side
# ---------------------------------------------------------------------------

def prepare(c, seed):
    s = _inputs(c, seed)
    kind = c["kind"]
    if kind == "gemm":
        s["c"] = torch.empty_like(s["c0"])
        return s
    if kind == "attention":
        s["o"] = torch.empty_like(s["q"])
        s["split"] = torch.empty(B.dif_attention_split_bytes(c["head_dim"]), dtype=torch.uint8,
                                 device="cuda")
        return s
    cfg = s["cfg"]
    m = s["model"] = B.dif_model_create(cfg, s["weights"])
    L = c["frames"] * c["rows"] * c["cols"]
    s["ws"] = B.workspace(m, c["batch"], L, c["text"])
    if kind == "time":
        s["e"] = torch.empty(cfg.dim, device="cuda")
        s["e0"] = torch.empty(6, cfg.dim, device="cuda")
    if kind in ("block", "step", "rollout"):
        s["plans"] = [B.dif_plan_step(m, i, TIMESTEPS[i], s["masks"][i], kind=c["plan"])
                      for i in sorted(s["masks"])]
        if c["cached"]:
            s["cache"] = B.dif_text_cache_build(m, s["ctx"])
    if kind == "block":
        s["x"] = torch.empty_like(s["x0"])
    if kind in ("step", "rollout", "switch"):
        s["v"] = torch.empty_like(s["z0"])
    if kind == "rollout":
        s["z"] = torch.empty_like(s["z0"])
    return s


def run(s):
    c = s["case"]
    kind, cached = c["kind"], c.get("cached")
    if kind == "gemm":
        if c["epilogue"] == B.EPI_RESIDUAL:   # updates its output in place
            s["c"].copy_(s["c0"])
            B.dif_gemm(s["a"], s["b"], s["c"], c["epilogue"], s["bias"], s["gate"])
        else:
            B.dif_gemm(s["a"], s["b"], s["c"], c["epilogue"], s["bias"])
        return s["c"]
    if kind == "attention":
        w = c["heads"] * c["head_dim"]
        B.dif_attention_ex(s["q"], s["k"], s["vt"], s["o"], c["batch"], c["lq"], c["lk"], c["heads"],
                           c["head_dim"], w, w, s["vt"].shape[1], w,
                           B.DIF_ATTN_Q_PRESCALED if c["prescaled"] else 0, s["split"])
        return s["o"]
    if kind == "time":
        B.dif_time_embed(s["model"], TIMESTEPS[c["step"]], s["e"], s["e0"], s["ws"])
        return s["e"], s["e0"]
    if kind == "text":
        cache = B.dif_text_cache_build(s["model"], s["ctx"])
        return _text_views(c, s["cfg"], cache.mem)
    if kind == "block":
        s["x"].copy_(s["x0"])   # the block updates the residual stream in place
        if cached:
            B.dif_block_forward_cached(s["plans"][0], 0, s["x"], s["cache"], s["e0"], s["ws"])
        else:
            B.dif_block_forward(s["plans"][0], 0, s["x"], s["ctx"], s["e0"], s["ws"])
        return s["x"]
    if kind == "rollout":
        s["z"].copy_(s["z0"])
        if cached:
            B.dif_rollout_cached(s["plans"], TIMESTEPS, s["z"], s["cache"], s["v"], s["ws"], s["eps"])
        else:
            B.dif_rollout(s["plans"], TIMESTEPS, s["z"], s["ctx"], s["v"], s["ws"], s["eps"])
        return s["z"], s["v"]
    i = c["step"]
    if kind == "switch":
        plan = B.dif_plan_step(s["model"], i, TIMESTEPS[i], s["masks"][i], kind=c["plan"])
        s["plans"] = [plan]   # the previous structure's plan is released here
    plan = s["plans"][0]
    if cached and kind == "step":
        B.dif_step_forward_cached(plan, s["z0"], TIMESTEPS[i], s["cache"], s["v"], s["ws"])
    else:
        B.dif_step_forward(plan, s["z0"], TIMESTEPS[i], s["ctx"], s["v"], s["ws"])
    return s["v"]


def _text_views(c, cfg, mem):
    """Each layer's keys [B * Lc, D] and transposed values [B, D, Lc up to 64]."""
    es = 2 if c["dtype"] == "bf16" else 4
    rows, D, ld = c["batch"] * c["text"], cfg.dim, -(-c["text"] // 64) * 64
    nk, nv, at, out = rows * D * es, c["batch"] * D * ld * es, 0, []
    for _ in range(cfg.n_layers):   # (both sizes are multiples of 256 for these widths)
        out.append(mem[at:at + nk].view(_dtype(c["dtype"])).view(rows, D))
        out.append(mem[at + nk:at + nk + nv].view(_dtype(c["dtype"])).view(c["batch"], D, ld))
        at += nk + nv
    return out


# ---------------------------------------------------------------------------
# accounting
# ---------------------------------------------------------------------------

def _block_work(c, cfg, h, hc, f):
    es = 2 if c["dtype"] == "bf16" else 4
    D, dh = cfg.dim, cfg.head_dim
    L, Lc = c["frames"] * c["rows"] * c["cols"], c["text"]
    M, Mc, a, ac = c["batch"] * L, c["batch"] * Lc, h * dh, hc * dh
    kv = not (c["cached"] and c["kind"] != "switch")
    fl = 2.0 * M * D * (4 * a + 2 * ac + 2 * f) + 4.0 * M * (L * a + Lc * ac)
    by = es * (4.0 * a * D + (4.0 if kv else 2.0) * ac * D + 2.0 * f * D)
    if kv:
        fl += 4.0 * Mc * D * ac
        by += es * Mc * D
    else:
        by += es * Mc * 2.0 * ac
    return by, fl, es * 2.0 * M * D


def work(c):
    kind = c["kind"]
    if kind == "gemm":
        es, eo = (2 if c["dtype"] == "bf16" else 4), (2 if c["out"] == "bf16" else 4)
        m, n, k = c["m"], c["n"], c["k"]
        return {"bytes": es * (m + n) * k + eo * m * n * (2 if c["epilogue"] == 2 else 1),
                "flops": 2.0 * m * n * k}
    if kind == "attention":
        es, w = (2 if c["dtype"] == "bf16" else 4), c["heads"] * c["head_dim"]
        return {"bytes": es * c["batch"] * w * 2.0 * (c["lq"] + c["lk"]),
                "flops": 4.0 * c["batch"] * c["lq"] * c["lk"] * w}
    cfg = _config(c)
    es, D = (2 if c["dtype"] == "bf16" else 4), cfg.dim
    t_by, t_fl = es * D * (FREQ + 7.0 * D), 2.0 * D * (FREQ + 7.0 * D)
    if kind == "time":
        return {"bytes": t_by, "flops": t_fl}
    if kind == "text":
        Mc = c["batch"] * c["text"]
        return {"bytes": es * (c["layers"] * (2.0 * D * D + 2.0 * Mc * D) + Mc * D),
                "flops": 4.0 * c["layers"] * Mc * D * D}
    by, fl, xio = _block_work(c, cfg, c["self_heads"], c["cross_heads"], c["ffn_keep"])
    if kind == "block":
        return {"bytes": by + xio, "flops": fl}
    M = c["batch"] * c["frames"] * c["rows"] * c["cols"]
    by = c["layers"] * by + t_by + es * 2.0 * PATCH * D + 8.0 * M * PATCH
    fl = c["layers"] * fl + t_fl + 4.0 * M * PATCH * D
    if kind == "switch" and c["plan"] == "compact":   # the gathered copy is written as well
        by *= 2.0
    if kind == "rollout":
        by, fl = 4.0 * by, 4.0 * fl
    return {"bytes": by, "flops": fl}


def tolerance(c):
    # About four times what these paths are off from float64 (exact below):
    # float32 6e-7 to 1.1e-6; bfloat16 products 1.7e-3 (their last rounding),
    # attention 2.2e-3, blocks 4e-3 to 9e-3.
    f32, kind = c["dtype"] == "f32", c["kind"]
    if f32 or kind == "time" or (kind == "gemm" and c["out"] == "f32"):
        return {"rel": 1e-5}
    return {"rel": {"gemm": 8e-3, "text": 8e-3, "attention": 1e-2}.get(kind, 2e-2)}


# ---------------------------------------------------------------------------
# the same in float64
# ---------------------------------------------------------------------------

def _attend(q, k, v, scale):
    """softmax(q k^T scale) v for [heads, rows, dim] float64, in row chunks."""
    out = torch.empty_like(q)
    kt = k.transpose(1, 2).contiguous()
    rows = max(1, int(2e8 // (q.shape[0] * k.shape[1])))
    for r in range(0, q.shape[1], rows):
        p = torch.softmax(torch.bmm(q[:, r:r + rows].contiguous(), kt) * scale, dim=-1)
        out[:, r:r + rows] = torch.bmm(p, v)
    return out


def _heads(x, n):
    return x.view(x.shape[0], n, -1).transpose(0, 1).contiguous()


def _ln(x):
    mu = x.mean(-1, keepdim=True)
    return (x - mu) / ((x - mu).square().mean(-1, keepdim=True) + EPS).sqrt()


def _gelu(x):
    return 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))


def _rope(x, cfg, n):
    dh, (gf, gh, gw) = cfg.head_dim, cfg.grid
    dhw = 2 * (dh // 6)
    tok = torch.arange(gf * gh * gw, device=x.device)
    ang = []
    for pos, d in ((tok // (gh * gw), dh - 2 * dhw), (tok // gw % gh, dhw), (tok % gw, dhw)):
        om = THETA ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
        ang.append(pos.double()[:, None] * om)
    phi = torch.cat(ang, 1)[:, None, :]
    y = x.view(x.shape[0], n, dh // 2, 2)
    x0, x1, cs, sn = y[..., 0], y[..., 1], phi.cos(), phi.sin()
    return torch.stack((x0 * cs - x1 * sn, x0 * sn + x1 * cs), -1).reshape(x.shape)


def _block64(x, ctx, e0, w, masks, l, cfg):
    """One block on one sample [L, D] over the kept heads and channels."""
    D, dh = cfg.dim, cfg.head_dim
    g = lambda k: w[k].double()
    idx = lambda m: torch.from_numpy(np.flatnonzero(m)).cuda()
    rows = lambda m: idx(np.repeat(m, dh))
    sh1, sc1, g1, sh2, sc2, g2 = w["mod"].double() + e0.double()
    scale = 1.0 / math.sqrt(dh)

    def proj(a, k, r):
        return a @ w["%s_w%s" % k][r].double().T + w["%s_b%s" % k].double()[r]

    def rms(t, gain, r):
        return t / (t.square().sum(-1, keepdim=True) / D + EPS).sqrt() * gain.double()[r]

    r, n = rows(masks["self_head_keep"][l]), int(masks["self_head_keep"][l].sum())
    a = _ln(x) * (1 + sc1) + sh1
    q = _rope(rms(proj(a, ("self", "q"), r), w["self_gq"], r), cfg, n)
    k = _rope(rms(proj(a, ("self", "k"), r), w["self_gk"], r), cfg, n)
    o = _attend(_heads(q, n), _heads(k, n), _heads(proj(a, ("self", "v"), r), n), scale)
    o = o.transpose(0, 1).reshape(x.shape[0], -1)
    x = x + g1 * (o @ w["self_wo"][:, r].double().T + g("self_bo"))

    r, n = rows(masks["cross_head_keep"][l]), int(masks["cross_head_keep"][l].sum())
    a = _ln(x) * g("norm3_w") + g("norm3_b")
    q = rms(proj(a, ("cross", "q"), r), w["cross_gq"], r)
    k = rms(proj(ctx, ("cross", "k"), r), w["cross_gk"], r)
    o = _attend(_heads(q, n), _heads(k, n), _heads(proj(ctx, ("cross", "v"), r), n), scale)
    o = o.transpose(0, 1).reshape(x.shape[0], -1)
    x = x + (o @ w["cross_wo"][:, r].double().T + g("cross_bo"))

    r = idx(masks["ffn_keep"][l])
    a = _ln(x) * (1 + sc2) + sh2
    u = _gelu(a @ w["ffn_w1"][r].double().T + w["ffn_b1"].double()[r])
    return x + g2 * (u @ w["ffn_w2"][:, r].double().T + g("ffn_b2"))


def _time64(w, t):
    om = 10000.0 ** (-torch.arange(FREQ // 2, device="cuda", dtype=torch.float64) / (FREQ // 2))
    emb = torch.cat(((t * om).cos(), (t * om).sin()))
    silu = torch.nn.functional.silu
    g = lambda k: w[k].double()
    e = g("t_w2") @ silu(g("t_w1") @ emb + g("t_b1")) + g("t_b2")
    return e, (g("t_w3") @ silu(e) + g("t_b3")).view(6, -1)


def _step64(z, t, ctx, w, masks, cfg):
    e, e0 = _time64(w, t)
    sh, sc = w["head_mod"].double() + e
    out = []
    for b in range(z.shape[0]):
        x = z[b] @ w["patch_w"].double().T + w["patch_b"].double()
        for l in range(cfg.n_layers):
            x = _block64(x, ctx[b].double(), e0, w["layers"][l], masks, l, cfg)
        out.append((_ln(x) * (1 + sc) + sh) @ w["head_w"].double().T + w["head_b"].double())
    return torch.stack(out)


def exact(c, seed):
    s = _inputs(c, seed)
    kind = c["kind"]
    if kind == "gemm":
        y = s["a"].double() @ s["b"].double().T + s["bias"].double()
        if c["epilogue"] == 1:
            y = _gelu(y)
        return s["c0"].double() + s["gate"].double() * y if c["epilogue"] == 2 else y
    if kind == "attention":
        n, out = c["heads"], []
        scale = math.log(2.0) if c["prescaled"] else 1.0 / math.sqrt(c["head_dim"])
        vt = s["vt"].double().view(c["batch"], n, c["head_dim"], -1)[..., :c["lk"]]
        for b in range(c["batch"]):
            q = _heads(s["q"][b * c["lq"]:(b + 1) * c["lq"]].double(), n)
            k = _heads(s["k"][b * c["lk"]:(b + 1) * c["lk"]].double(), n)
            o = _attend(q, k, vt[b].transpose(1, 2).contiguous(), scale)
            out.append(o.transpose(0, 1).reshape(c["lq"], -1))
        return torch.cat(out)
    cfg, w = s["cfg"], s["weights"]
    if kind == "time":
        return _time64(w, TIMESTEPS[c["step"]])
    if kind == "text":
        out, rows, ld = [], c["batch"] * c["text"], -(-c["text"] // 64) * 64
        x = s["ctx"].double().view(rows, -1)
        for lw in w["layers"]:
            out.append(x @ lw["cross_wk"].double().T + lw["cross_bk"].double())
            v = (x @ lw["cross_wv"].double().T + lw["cross_bv"].double()).view(c["batch"], c["text"], -1)
            vt = torch.zeros(c["batch"], cfg.dim, ld, device="cuda", dtype=torch.float64)
            vt[:, :, :c["text"]] = v.transpose(1, 2)
            out.append(vt)
        return out
    if kind == "block":
        return torch.stack([_block64(s["x0"][b].double(), s["ctx"][b].double(), s["e0"],
                                     w["layers"][0], s["masks"][c["step"]], 0, cfg)
                            for b in range(c["batch"])])
    if kind == "rollout":
        z, v = s["z0"].double(), None
        for i, t in enumerate(TIMESTEPS):
            v = _step64(z, t, s["ctx"], w, s["masks"][i], cfg)
            z = z - t / 1000.0 * v
            if i < 3:
                st = TIMESTEPS[i + 1] / 1000.0
                z = (1 - st) * z + st * s["eps"][i].double()
        return z, v
    i = c["step"]
    return _step64(s["z0"].double(), TIMESTEPS[i], s["ctx"], w, s["masks"][i], cfg)
