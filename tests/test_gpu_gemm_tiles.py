"""The GEMM operator over its tile shapes, ragged in every dimension.

The sizes are such that the choice of the tile (least estimated time) takes
most shapes in turn, with plain operands of the output's type; the first group
walks the k-loop's edges (fewer k-tiles than ring slots, one more, a whole number
of turns, one less) on the smallest.
Reference: the float64 product of the same inputs on sampled rows.
"""
import numpy as np
import pytest

import oracle as O
from paper_2607_06631_amd import binding as B
from tests.gpu_util import rel_err, say, to_np
from workloads.synth import bf16_round

pytestmark = pytest.mark.gpu

K_EDGES = [(70, 101, 64 * n) for n in (1, 2, 3, 5, 6, 7, 11, 12, 13, 17)]
SHAPES = [(200, 100, 256), (1001, 3002, 320), (1037, 2001, 512), (1101, 5203, 448), (390, 7681, 5120),
          (1501, 5001, 576), (4101, 4099, 512), (2001, 5201, 512), (2301, 5401, 512), (8199, 8190, 192)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", K_EDGES + SHAPES)
def test_gemm_tile_shapes(dtype, M, N, K):
    import torch
    say(f"gemm tiles {dtype} M={M} N={N} K={K}")
    g = np.random.default_rng(M * 7 + N + K)
    bf = dtype == "bf16"
    tdt = torch.bfloat16 if bf else torch.float32

    def rand(shape, scale=1.0):
        a = g.standard_normal(shape, dtype=np.float32) * np.float32(scale)
        return bf16_round(a) if bf else a

    a, b = rand((M, K), 0.5), rand((N, K), 0.5)
    bias, gate = g.standard_normal(N).astype(np.float32), g.standard_normal(N).astype(np.float32)
    A, Bm = torch.from_numpy(a).cuda().to(tdt), torch.from_numpy(b).cuda().to(tdt)
    tb, tg = torch.from_numpy(bias).cuda(), torch.from_numpy(gate).cuda()
    rows = np.unique(np.concatenate([np.arange(min(M, 40)), g.choice(M, min(M, 120), replace=False),
                                     np.arange(max(0, M - 40), M)]))
    acc = a[rows].astype(np.float64) @ b.astype(np.float64).T + bias
    # float32 sums of K products: K * 2^-24 of the largest at worst; bf16
    # output adds one rounding, 2^-9 of the element
    tol = 8e-3 if bf else 1e-5
    for epi, ref in ((B.EPI_STORE, acc), (B.EPI_GELU, O.gelu_tanh(acc)), (B.EPI_RESIDUAL, None)):
        x = torch.empty((M + 1, N), device="cuda", dtype=tdt).fill_(7.0)
        if epi == B.EPI_RESIDUAL:
            x0 = rand((M, N))
            x[:M] = torch.from_numpy(x0).cuda().to(tdt)
            ref = x0[rows] + gate * acc
        B.dif_gemm(A, Bm, x[:M], epi, bias=tb, gate0=tg if epi == B.EPI_RESIDUAL else None)
        torch.cuda.synchronize()
        assert rel_err(to_np(x[torch.from_numpy(rows).cuda()]), ref) <= tol
        assert bool((x[M] == 7.0).all())
