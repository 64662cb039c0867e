"""Attention over the sizes where its choice of kernel and its key groups can go
wrong: fewer keys than a group's first tile, one more, ranges that leave the
second key group nothing or one key, query counts around a workgroup's; and the
two-group kernel below its long-key threshold, whole and with its last round
split.  Reference: the oracle's two-pass softmax in float64.
"""
import numpy as np
import pytest

import oracle as O
from paper_2607_06631_amd import binding as B
from tests.gpu_util import rel_err, say, to_np
from workloads.synth import bf16_round

pytestmark = pytest.mark.gpu


def _case(dtype, dh, H, Lq, Lk, Bn, heads, qscale, split=False):
    import torch
    g = np.random.default_rng(Lq * 131 + Lk)
    bf = dtype == "bf16"
    tdt = torch.bfloat16 if bf else torch.float32
    W = H * dh

    def rand(shape, scale=1.0):
        a = g.standard_normal(shape, dtype=np.float32) * np.float32(scale)
        return bf16_round(a) if bf else a

    q, k, v = rand((Bn, Lq, W), qscale), rand((Bn, Lk, W)), rand((Bn, Lk, W))
    ldvt = -(-Lk // 64) * 64 + 64       # padded, garbage in the pad
    vt = np.full((Bn, W, ldvt), np.nan, np.float32)
    vt[:, :, :Lk] = v.transpose(0, 2, 1)
    Q, K, Vt = (torch.from_numpy(a).cuda().to(tdt) for a in (q, k, vt))
    Ot = torch.full((Bn, Lq + 1, W), float("nan"), device="cuda", dtype=tdt)
    out = Ot.view(-1, W)[:Bn * Lq]
    ws = None
    if split:
        ws = torch.empty(B.dif_attention_split_bytes(dh), dtype=torch.uint8, device="cuda")
    B.dif_attention_ex(Q, K, Vt, out, Bn, Lq, Lk, H, dh, W, W, ldvt, W, 0, ws)
    torch.cuda.synchronize()
    assert bool(torch.isnan(Ot.view(-1, W)[Bn * Lq:]).all())
    got = to_np(out).reshape(Bn, Lq, W)
    errs = []
    for h in heads:
        c = slice(h * dh, (h + 1) * dh)
        ref = np.stack([O.attention(q[b][:, c].astype(np.float64), k[b][:, c].astype(np.float64),
                                    v[b][:, c].astype(np.float64), 1, dh) for b in range(Bn)])
        errs.append(rel_err(got[:, :, c], ref))
    return max(errs)


@pytest.mark.parametrize("dtype,dh", [("bf16", 128), ("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("Lq,Lk", [(1, 1), (31, 31), (32, 32), (33, 33), (64, 63), (65, 64), (66, 65),
                                   (127, 96), (128, 97), (129, 128), (63, 129), (200, 511)])
def test_key_groups(dtype, dh, Lq, Lk):
    say(f"attention groups {dtype} dh={dh} Lq={Lq} Lk={Lk}")
    err = _case(dtype, dh, 3, Lq, Lk, 2, range(3), 3.0)
    assert err <= (2e-2 if dtype == "bf16" else 1e-5)


@pytest.mark.parametrize("H,Lq,Lk,split", [(42, 1290, 2049, False), (42, 1290, 2049, True),
                                           (29, 2600, 2100, False), (29, 2600, 2100, True),
                                           (30, 256, 1024, False), (12, 1000, 4095, True)])
def test_below_the_long_key_threshold(H, Lq, Lk, split):
    say(f"attention bf16 H={H} Lq={Lq} Lk={Lk} split={split}")
    assert _case("bf16", 128, H, Lq, Lk, 1, (0, H - 1), 3.0, split) <= 2e-2


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("lo,hi,Lk", [(128, 160, 256), (96, 193, 193), (40, 256, 256), (64, 65, 65)])
def test_keys_whose_scores_overflow_downwards(dh, lo, hi, Lk):
    """Keys [lo, hi), which begin the second key group's range or are all of it,
    score -inf for every query: they weigh nothing, and the result is the
    attention over the others (1e25 * -1e25 overflows float32; the other keys
    meet that channel of the queries with zero)."""
    import torch
    say(f"attention -inf scores dh={dh} keys {lo}..{hi} of {Lk}")
    g = np.random.default_rng(lo + Lk)
    H, Lq = 3, 130
    W = H * dh
    q, k, v = (g.standard_normal((n, W), dtype=np.float32) for n in (Lq, Lk, Lk))
    q[:, ::dh], k[:, ::dh] = 1e25, 0
    k[lo:hi, ::dh] = -1e25
    ldvt = -(-Lk // 64) * 64
    vt = np.zeros((W, ldvt), np.float32)
    vt[:, :Lk] = v.T
    Q, K, Vt = (torch.from_numpy(a).cuda() for a in (q, k, vt))
    out = torch.empty_like(Q)
    B.dif_attention_ex(Q, K, Vt, out, 1, Lq, Lk, H, dh, W, W, ldvt, W, 0, None)
    torch.cuda.synchronize()
    keep = np.r_[0:lo, hi:Lk]
    q[:, ::dh] = 0
    for h in range(H):
        c = slice(h * dh, (h + 1) * dh)
        ref = O.attention(q[:, c].astype(np.float64), k[keep][:, c].astype(np.float64),
                          v[keep][:, c].astype(np.float64), 1, dh)
        assert rel_err(to_np(out)[:, c], ref) <= 1e-5


@pytest.mark.parametrize("cus", [32, 64, 128, 250])
@pytest.mark.parametrize("dtype,H,Lq,Lk", [("bf16", 9, 1300, 2100), ("bf16", 5, 700, 600), ("f32", 5, 700, 600),
                                           ("bf16", 3, 300, 4200)])
def test_choice_and_key_split_for_other_cu_counts(dtype, H, Lq, Lk, cus):
    """The launcher given another CU count than the whole chip's (a partition's):
    the choice of kernel and the key split are made for that count, with every
    query in exactly one workgroup or one split pair."""
    import ctypes as C
    import torch
    say(f"attention {dtype} H={H} Lq={Lq} Lk={Lk} for {cus} CUs")
    g = np.random.default_rng(Lq + Lk)
    bf, dh = dtype == "bf16", 128
    tdt, W, ldvt = (torch.bfloat16 if bf else torch.float32), H * dh, -(-Lk // 64) * 64
    q, k, v = (g.standard_normal((n, W), dtype=np.float32) for n in (Lq, Lk, Lk))
    if bf:
        q, k, v = (bf16_round(a) for a in (q, k, v))
    vt = np.zeros((W, ldvt), np.float32)
    vt[:, :Lk] = v.T
    Q, K, Vt = (torch.from_numpy(a).cuda().to(tdt) for a in (q, k, vt))
    out = torch.full_like(Q, float("nan"))
    ws = torch.empty(B.dif_attention_split_bytes(dh), dtype=torch.uint8, device="cuda")
    f = getattr(B.lib(), "_ZN3dif16launch_attentionI%sEE10hipError_tiPKT_lS4_lS4_lPS2_liiiiP12ihipStream_tbPfi"
                         % ("DF16b" if bf else "f"))
    f.restype = C.c_int
    f.argtypes = ([C.c_int] + [C.c_void_p, C.c_int64] * 4 + [C.c_int] * 4
                  + [C.c_void_p, C.c_bool, C.c_void_p, C.c_int])
    assert f(dh, Q.data_ptr(), W, K.data_ptr(), W, Vt.data_ptr(), ldvt, out.data_ptr(), W, 1, Lq, Lk, H,
             torch.cuda.current_stream().cuda_stream, False, ws.data_ptr(), cus) == 0
    torch.cuda.synchronize()
    for h in range(H):
        c = slice(h * dh, (h + 1) * dh)
        ref = O.attention(q[:, c].astype(np.float64), k[:, c].astype(np.float64), v[:, c].astype(np.float64), 1, dh)
        assert rel_err(to_np(out)[:, c], ref) <= (2e-2 if bf else 1e-5)
