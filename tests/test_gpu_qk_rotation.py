"""The q / k rotation's rounding, bit for bit, over every instance of its kernel.

A rotated pair is (x0 cos - x1 sin, x0 sin + x1 cos) with one product rounded and
the other inside a fused multiply-add.  Which one is part of the result: it must
not change with the rows per wave or from build to build.  The launcher is called
with rows of +-1 (their RMS is exactly 1, so the normalised value is the gain,
exactly) and the output compared with the products summed in extended precision.
Widths: 4, 8, 12 and 16 vectors per lane, one segment and two; row counts for one
row per wave, four and sixteen.
"""
import ctypes as C

import numpy as np
import pytest

from paper_2607_06631_amd import binding as B
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


class _Rope(C.Structure):
    _fields_ = ([("table", C.c_void_p)]
                + [(k, C.c_int) for k in ("L", "gf", "gh", "gw", "jt", "jh", "jw", "head_dim", "rows1")]
                + [("src1", C.c_void_p), ("dst1", C.c_void_p), ("lds1", C.c_int64), ("ldd1", C.c_int64),
                   ("src_idx1", C.c_void_p), ("gain1", C.c_void_p)])


def _fma(a, b, c):
    ld = np.longdouble
    return (a.astype(ld) * b.astype(ld) + c.astype(ld)).astype(np.float32)


@pytest.mark.parametrize("rows", [37, 9000, 33000])
@pytest.mark.parametrize("nseg", [1, 2])
@pytest.mark.parametrize("vectors", [4, 8, 12, 16])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rotation_rounds_the_same_product(dtype, vectors, nseg, rows):
    import torch
    bf = dtype == "bf16"
    tdt = torch.bfloat16 if bf else torch.float32
    a, dh = vectors * 64 * (8 if bf else 4), 128
    say(f"qk rotation {dtype} width={a} segments={nseg} rows={rows}")
    gen = torch.Generator(device="cuda").manual_seed(a + rows)
    x = torch.randint(0, 2, (rows, nseg * a), generator=gen, device="cuda").mul_(2).sub_(1).to(tdt)
    gains = [torch.randn(a, generator=gen, device="cuda") for _ in range(2)]
    ang = torch.randn(rows * 22 + 42, generator=gen, device="cuda")
    tab = torch.stack((ang.cos(), ang.sin()), -1).contiguous()
    rope = _Rope(table=tab.data_ptr(), L=rows, gf=rows, gh=1, gw=1, jt=22, jh=21, jw=21, head_dim=dh)
    f = getattr(B.lib(), "_ZN3dif14launch_qk_normI%sEE10hipError_tPT_liiiiiPKfS5_ffPKNS_8RopeDescEP12"
                         "ihipStream_tPKif" % ("DF16b" if bf else "f"))
    f.restype = C.c_int
    f.argtypes = ([C.c_void_p, C.c_int64] + [C.c_int] * 5 + [C.c_void_p] * 2 + [C.c_float] * 2
                  + [C.c_void_p] * 3 + [C.c_float])
    keep = torch.arange(0, rows, max(1, rows // 500), device="cuda")
    sign = x[keep].float().cpu().numpy()
    assert f(x.data_ptr(), nseg * a, rows, a, nseg, 0, a, gains[0].data_ptr(), gains[1].data_ptr(), 1.0 / a,
             1e-30, C.byref(rope), torch.cuda.current_stream().cuda_stream, None, 1.0) == 0
    torch.cuda.synchronize()
    z = x[keep].float().cpu().numpy()

    y = sign * np.concatenate([g.cpu().numpy() for g in gains[:nseg]])
    n, k = keep.cpu().numpy()[:, None], np.arange(0, nseg * a, 2) // 2 % (dh // 2)
    t = tab.cpu().numpy()[np.where(k < 22, n * 22 + k, rows * 22 + k - 22)]
    cs, sn, y0, y1 = t[..., 0], t[..., 1], y[:, ::2], y[:, 1::2]
    out = (lambda v: torch.from_numpy(v).to(tdt).float().numpy())
    assert np.array_equal(z[:, ::2], out(_fma(y0, cs, -(y1 * sn))))
    rounds_x0 = vectors == 16 or (vectors == 12 and bf) or (vectors == 8 and nseg == 2)
    want, other = _fma(y1, cs, y0 * sn), _fma(y0, sn, y1 * cs)
    if not rounds_x0:
        want, other = other, want
    assert np.array_equal(z[:, 1::2], out(want))
    # (the test can tell them apart; bf16 rounds most differences away)
    assert rows < 500 or not np.array_equal(z[:, 1::2], out(other))
