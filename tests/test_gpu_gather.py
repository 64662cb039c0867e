"""The plan's gather of kept rows and columns, checked exactly on the reordered
FFN weights (the same launches: rows of W1 and b1, columns of W2 by an arbitrary
permutation) at widths that take each path: whole 16-byte vectors, a width that
is none, source or destination addresses off a 16-byte boundary (each alone and
both), row counts that are not a multiple of a lane's rows.  Kept runs and dropped
entries are covered bit for bit by the compact / indexed plan tests, and here at
an FFN width that is no whole number of vectors, whose W2 rows start off a 16-byte
boundary and go to padded, aligned ones.
"""
import numpy as np
import pytest

from paper_2607_06631_amd import binding as B
from tests.gpu_util import rel_err, say, to_np
from workloads import get_config, synth

pytestmark = pytest.mark.gpu


def _at(t, shift):
    """A copy of t that starts `shift` elements past a 256-byte boundary."""
    import torch
    buf = torch.empty(t.numel() + 64, dtype=t.dtype, device="cuda")
    v = buf[shift:shift + t.numel()].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ffn", [1, 64, 203, 1030])
@pytest.mark.parametrize("shift,to", [(0, 0), (1, 1), (1, 0), (0, 1)])
def test_reordered_weights_are_the_permuted_ones(dtype, ffn, shift, to):
    import ctypes as C
    import torch
    cfg = get_config("tiny").with_(ffn_dim=ffn, n_layers=1, dtype=dtype, ffn_chunk=1,
                                   head_dim=64 if dtype == "f32" else 128, n_heads=4 if dtype == "f32" else 2)
    say(f"gather {dtype} ffn={ffn} shift={shift} to {to}")
    w = B.upload_weights(synth.make_weights(cfg, seed=3), dtype)
    lw = w["layers"][0]
    for k in ("ffn_w1", "ffn_w2", "ffn_b1"):
        lw[k] = _at(lw[k], shift)
    model = B.dif_model_create(cfg, w)
    w1, w2, b1 = (_at(torch.zeros_like(lw[k]), to) for k in ("ffn_w1", "ffn_w2", "ffn_b1"))
    scratch = torch.empty(ffn * 12 + 16, dtype=torch.uint8, device="cuda")
    perm = np.zeros(ffn, np.int32)
    B._check(B.lib().dif_ffn_reorder(model.handle, 0, w1.data_ptr(), b1.data_ptr(), w2.data_ptr(),
                                     perm.ctypes.data, scratch.data_ptr(), scratch.numel(), None))
    torch.cuda.synchronize()
    p = torch.from_numpy(perm.astype(np.int64)).cuda()
    assert sorted(perm.tolist()) == list(range(ffn))
    assert torch.equal(w1, lw["ffn_w1"][p])
    assert torch.equal(w2, lw["ffn_w2"][:, p])
    assert torch.equal(b1, lw["ffn_b1"][p])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ffn,kept", [(1030, 1030), (1030, 701), (203, 90)])
def test_compact_plan_of_a_ragged_ffn(dtype, ffn, kept):
    import oracle as O
    import torch
    cfg = get_config("tiny").with_(ffn_dim=ffn, n_layers=1, dtype=dtype, ffn_chunk=1, keep_ffn=(kept,),
                                   keep_heads=(2,), head_dim=64 if dtype == "f32" else 128,
                                   n_heads=4 if dtype == "f32" else 2)
    say(f"gather compact plan {dtype} ffn={kept}/{ffn}")
    w = synth.make_weights(cfg, seed=3)
    masks = synth.make_masks(cfg, 0)
    assert int(masks["ffn_keep"].sum()) == kept
    x0, ctx, e0 = synth.make_block_input(cfg), synth.make_context(cfg), synth.make_e0(cfg)
    model = B.dif_model_create(cfg, B.upload_weights(w, cfg.dtype))
    plan = B.dif_plan_step(model, 0, cfg.timesteps[0], masks)
    ws = B.workspace(model, 1, cfg.seq_len, cfg.text_len)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.from_numpy(x0).cuda().to(tdt)
    B.dif_block_forward(plan, 0, x, torch.from_numpy(ctx).cuda().to(tdt), torch.from_numpy(e0).cuda(), ws)
    torch.cuda.synchronize()
    wz = O.apply_keep(w["layers"][0], masks["self_head_keep"][0], masks["cross_head_keep"][0],
                      masks["ffn_keep"][0], cfg.head_dim)
    ref = O.block(x0[0], ctx[0], e0, wz, True, cfg.n_heads, cfg.head_dim, cfg.grid)
    assert rel_err(to_np(x)[0], ref) <= (1e-4 if dtype == "f32" else 2e-2)
