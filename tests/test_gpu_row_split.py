"""Row kernels (LayerNorm + modulation, q / k RMSNorm) over row counts that
change their split into workgroups: one row, fewer rows than waves, each step
of waves per workgroup and rows per wave, remainders.

Run through one block on token grids of those sizes (L = 1 .. 4500, B 1 and 2)
in float32 against the oracle, with the modulation vectors at an address that
allows 16-byte loads and at one that does not (both paths, same bits).
"""
import numpy as np
import pytest

import oracle as O
from paper_2607_06631_amd import binding as B
from tests.gpu_util import rel_err, say, to_np
from workloads import get_config, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,batch", [((1, 1, 1), 1), ((1, 1, 3), 1), ((2, 8, 8), 2), ((1, 19, 27), 1),
                                        ((1, 25, 41), 1), ((1, 40, 52), 1), ((1, 45, 50), 2)])
def test_block_over_row_counts(grid, batch):
    import torch
    cfg = get_config("tiny").with_(grid=grid, n_layers=1, batch=batch)
    say(f"row split grid={grid} batch={batch}")
    w = synth.make_weights(cfg, seed=0)
    masks = synth.make_masks(cfg, 1)
    x0, ctx, e0 = synth.make_block_input(cfg), synth.make_context(cfg), synth.make_e0(cfg)
    model = B.dif_model_create(cfg, B.upload_weights(w, cfg.dtype))
    plan = B.dif_plan_step(model, 1, cfg.timesteps[1], masks)
    ws = B.workspace(model, batch, cfg.seq_len, cfg.text_len)
    outs = []
    for shift in (0, 1):
        e = torch.zeros(6 * cfg.dim + 4, device="cuda")[shift:shift + 6 * cfg.dim].view(6, cfg.dim)
        e.copy_(torch.from_numpy(e0))
        x = torch.from_numpy(x0).cuda()
        B.dif_block_forward(plan, 0, x, torch.from_numpy(ctx).cuda(), e, ws)
        torch.cuda.synchronize()
        outs.append(to_np(x))
    wz = O.apply_keep(w["layers"][0], masks["self_head_keep"][0], masks["cross_head_keep"][0],
                      masks["ffn_keep"][0], cfg.head_dim)
    for b in range(batch):
        ref = O.block(x0[b], ctx[b], e0, wz, True, cfg.n_heads, cfg.head_dim, cfg.grid)
        assert rel_err(outs[0][b], ref) <= 1e-4
    assert np.array_equal(outs[0], outs[1])
