"""The text projections' launch (keys and transposed values as two segments,
values written transposed with zeroed padding) and the norm that reads cached
keys through the head table, at text lengths around its cases: 1, not a
multiple of 4, a multiple of 4 but not of 64, whole tiles; one sample and two.

The cache is compared with the float64 projection of the same inputs, its
padding with zero; the cached block must equal the uncached one bit for bit.
"""
import numpy as np
import pytest

from paper_2607_06631_amd import binding as B
from tests.gpu_util import rel_err, say, to_np
from workloads import get_config, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", ["tiny", "bf16"])
@pytest.mark.parametrize("Lc,batch", [(1, 1), (5, 2), (63, 1), (64, 2), (68, 1), (77, 2), (130, 1)])
def test_text_cache_values_and_cached_block(width, Lc, batch):
    import torch
    cfg = get_config("tiny").with_(n_layers=2, text_len=Lc, batch=batch, grid=(1, 5, 7))
    if width == "bf16":
        cfg = cfg.with_(dtype="bf16", head_dim=128, n_heads=3, dim=384, ffn_dim=512,
                        keep_heads=(3, 2, 1, 2), keep_ffn=(512, 384, 320, 256))
    say(f"text values {width} Lc={Lc} batch={batch}")
    w = synth.make_weights(cfg, seed=0)
    ctx = synth.make_context(cfg)
    model = B.dif_model_create(cfg, B.upload_weights(w, cfg.dtype))
    tdt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    cd = torch.from_numpy(ctx).cuda().to(tdt)
    n = B.dif_text_cache_bytes(model, batch, Lc)
    mem = torch.full((n,), 0xAB, dtype=torch.uint8, device="cuda")
    B._check(B.lib().dif_text_cache_build(model.handle, cd.data_ptr(), batch, Lc, mem.data_ptr(), n, None))
    torch.cuda.synchronize()
    es, D, ld = (2 if cfg.dtype == "bf16" else 4), cfg.dim, -(-Lc // 64) * 64
    up = lambda b: -(-b // 256) * 256
    tol = 8e-3 if cfg.dtype == "bf16" else 1e-5
    at = 0
    for l in range(cfg.n_layers):
        lw = {k: v.astype(np.float64) for k, v in w["layers"][l].items()}
        x = ctx.astype(np.float64).reshape(-1, D)
        k = mem[at:at + batch * Lc * D * es].view(tdt).view(-1, D)
        at += up(batch * Lc * D * es)
        vt = mem[at:at + batch * D * ld * es].view(tdt).view(batch, D, ld)
        at += up(batch * D * ld * es)
        assert rel_err(to_np(k), x @ lw["cross_wk"].T + lw["cross_bk"]) <= tol
        v = (x @ lw["cross_wv"].T + lw["cross_bv"]).reshape(batch, Lc, D).transpose(0, 2, 1)
        assert rel_err(to_np(vt[:, :, :Lc]), v) <= tol
        assert bool((vt[:, :, Lc:] == 0).all())
    cache = B.TextCache(mem, batch, Lc)
    ws = B.workspace(model, batch, cfg.seq_len, Lc)
    e0 = torch.from_numpy(synth.make_e0(cfg)).cuda()
    x0 = torch.from_numpy(synth.make_block_input(cfg)).cuda().to(tdt)
    for kind in ("compact", "indexed"):
        for step in (1, 2):
            plan = B.dif_plan_step(model, step, cfg.timesteps[step], synth.make_masks(cfg, step), kind=kind)
            xa, xb = x0.clone(), x0.clone()
            B.dif_block_forward(plan, 0, xa, cd, e0, ws)
            B.dif_block_forward_cached(plan, 0, xb, cache, e0, ws)
            torch.cuda.synchronize()
            assert torch.equal(xa, xb)
