"""Every instance of the ring GEMM, tile shape by tile shape, through its launcher.

The choice of the tile decides which instance a public call runs, so a shape's
gathered forms, segments, transposed columns and float32 output are reached only
at sizes that happen to choose it.  Here each shape is asked for: plain operands
with the three epilogues, rows of B through a table (dropped rows, two segments,
transposed columns), K chunks through a table (dropped chunks), for k-tile counts
below, at and past the ring's slots, ragged in every dimension, output rows that
allow vector accesses and rows that do not.  Reference: float64 products; and the
shapes must agree bit for bit, since the choice may not change a result.
"""
import ctypes as C

import pytest

from paper_2607_06631_amd import binding as B
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

# (rows, columns, k-tiles in flight) of the shapes by their number
BF16 = {0: (256, 256, 2), 1: (224, 256, 2), 2: (192, 256, 2), 3: (160, 256, 3), 4: (128, 256, 3), 5: (96, 256, 3),
        6: (128, 128, 4), 7: (96, 128, 5), 8: (64, 128, 3), 9: (64, 64, 4), 10: (32, 32, 6), 12: (128, 128, 2)}
F32 = {7: (96, 128, 2), 8: (64, 128, 3), 9: (64, 64, 4), 10: (32, 32, 6)}
SMALLEST = 10
NONE, ROWS, KCH = 0, 1, 2
STORE, GELU, RESIDUAL = 0, 1, 2


class _Params(C.Structure):
    _fields_ = [("A", C.c_void_p), ("Bs", C.c_void_p * 3), ("C", C.c_void_p), ("lda", C.c_int64), ("ldb", C.c_int64),
                ("ldc", C.c_int64), ("M", C.c_int), ("N", C.c_int), ("K", C.c_int), ("biases", C.c_void_p * 3),
                ("nseg", C.c_int), ("gate0", C.c_void_p), ("gate1", C.c_void_p), ("rows", C.c_void_p),
                ("kch", C.c_void_p), ("b_rows", C.c_int), ("vec4", C.c_int), ("vt", C.c_void_p), ("ldvt", C.c_int64),
                ("vt_col0", C.c_int), ("vt_dims", C.c_int), ("vt_L", C.c_int), ("vt_vec4", C.c_int),
                ("vt_pad", C.c_int)]


def _launch(types, shape, p, epi, ga):
    import torch
    t = {"bf16": "DF16bDF16b", "bf16_f32": "DF16bf", "f32": "ff"}[types]
    f = getattr(B.lib(), f"_ZN3dif16launch_gemm_ringI{t}EE10hipError_tiRKNS_10GemmParamsIT_T0_EEiiP12ihipStream_t")
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_void_p, C.c_int, C.c_int, C.c_void_p]
    assert f(shape, C.addressof(p), epi, ga, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


class _Problem:
    """Operands of one M x N x K problem with every table; N columns per segment."""

    def __init__(self, types, M, N, K, ldc_pad, seed):
        import torch
        self.types, self.M, self.N, self.K = types, M, N, K
        self.tdt = torch.float32 if types == "f32" else torch.bfloat16
        self.odt = torch.bfloat16 if types == "bf16" else torch.float32
        vec = 4 if types == "f32" else 8
        gen = torch.Generator(device="cuda").manual_seed(seed)
        rand = lambda *s: torch.randn(s, generator=gen, device="cuda")
        perm = lambda n: torch.randperm(n, generator=gen, device="cuda").int()
        self.A = rand(M, K).mul_(0.5).to(self.tdt)
        self.union, self.width = N + 9, K + 5 * vec      # rows of B, columns of B
        self.B = [rand(self.union, self.width).mul_(0.5).to(self.tdt) for _ in range(2)]
        self.bias = [rand(self.union) for _ in range(2)]
        self.gate = [rand(N) for _ in range(2)]
        self.rows = perm(self.union)[:N].contiguous()
        self.rows[::7] = -1
        self.kch = perm(self.width // vec)[:K // vec].contiguous()
        self.kch[3::5] = -1
        self.vec, self.ldc = vec, 2 * N + ldc_pad
        self.x0 = rand(M, self.ldc).to(self.odt)

    def params(self, c, ga, nseg=1):
        p = _Params(A=self.A.data_ptr(), C=c.data_ptr(), lda=self.K, ldb=self.width, ldc=self.ldc, M=self.M, N=self.N,
                    K=self.K, nseg=nseg, gate0=self.gate[0].data_ptr(), gate1=self.gate[1].data_ptr())
        for i in range(2):
            p.Bs[i], p.biases[i] = self.B[i].data_ptr(), self.bias[i].data_ptr()
        # (a second segment's columns start N elements in)
        p.vec4 = int(self.ldc % 4 == 0 and (nseg == 1 or self.N % 4 == 0))
        if ga == ROWS:
            p.rows, p.b_rows = self.rows.data_ptr(), self.union
        if ga == KCH:
            p.kch = self.kch.data_ptr()
        return p

    def ref(self, ga, seg=0):
        b, bias = self.B[seg].double(), self.bias[seg].double()
        if ga == ROWS:
            r = self.rows.long()
            b, bias = b[r.clamp_min(0)], bias[r.clamp_min(0)]
            b[r < 0], bias[r < 0] = 0, 0
        else:
            b, bias = b[:self.N], bias[:self.N]
        if ga == KCH:
            k = self.kch.long()
            b = b.view(self.N, -1, self.vec)[:, k.clamp_min(0)].clone()
            b[:, k < 0] = 0
            b = b.reshape(self.N, -1)
        return self.A.double() @ b[:, :self.K].t() + bias

    def run(self, shape, epi, ga, nseg=1, vt_L=0):
        import torch
        c, vt = self.x0.clone(), None
        p = self.params(c, ga, nseg)
        if vt_L:
            ldvt = vt_L + (4 if vt_L % 4 == 0 else 5)
            vt = torch.full((self.M // vt_L * self.N, ldvt), 7.0, device="cuda", dtype=self.odt)
            p.vt, p.ldvt, p.vt_col0, p.vt_dims, p.vt_L, p.vt_pad = vt.data_ptr(), ldvt, self.N, self.N, vt_L, 1
            p.vt_vec4 = int(vt_L % 4 == 0)
        _launch(self.types, shape, p, epi, ga)
        return c, vt


def _close(got, ref, tol):
    got = got.double()
    assert bool(got.isfinite().all())
    assert float((got - ref).abs().max()) <= tol * float(ref.abs().max())


def _gelu(x):
    import torch
    return torch.nn.functional.gelu(x, approximate="tanh")


CASES = ([("bf16", s) for s in BF16] + [("bf16_f32", s) for s in BF16 if s] + [("f32", s) for s in F32])


@pytest.mark.parametrize("types,shape", CASES)
def test_instances(types, shape):
    import torch
    bm, bn, nst = (F32 if types == "f32" else BF16)[shape]
    kt = 32 if types == "f32" else 64
    # float32 sums: K * 2^-24 of the largest at worst; bf16 output adds 2^-9 of the element
    tol = 8e-3 if types == "bf16" else 1e-5
    for n, (nk, ldc_pad) in enumerate(((1, 0), (nst, 3), (nst + 1, 0), (2 * nst - 1, 0), (2 * nst, 1), (3 * nst + 2, 0))):
        M, N, K = 2 * bm + (5 if n % 2 else 8), bn + (37 if n % 2 else 36), nk * kt
        say(f"gemm instance {types} shape={shape} M={M} N={N} K={K} ldc+{ldc_pad}")
        q = _Problem(types, M, N, K, ldc_pad, 17 * shape + n)
        forms = []
        if shape:   # (the largest plain problems run another kernel)
            forms += [(STORE, NONE), (GELU, NONE), (RESIDUAL, NONE)]
        if types != "bf16_f32":
            forms += [(STORE, ROWS), (GELU, ROWS), (RESIDUAL, KCH)]
        for epi, ga in forms:
            if shape == 12 and epi != STORE:
                continue
            c, _ = q.run(shape, epi, ga)
            y = q.ref(ga)
            if epi == GELU:
                y = _gelu(y)
            if epi == RESIDUAL:
                y = q.x0[:, :N].double() + (q.gate[0].double() + q.gate[1].double()) * y
            _close(c[:, :N], y, tol)
            assert torch.equal(c[:, N:], q.x0[:, N:])
            assert torch.equal(c, q.run(SMALLEST, epi, ga)[0])
            if epi == STORE:   # two segments, and the second one transposed
                c2, _ = q.run(shape, epi, ga, nseg=2)
                y1 = q.ref(ga, 1)
                _close(c2[:, N:2 * N], y1, tol)
                assert torch.equal(c2[:, :N], c[:, :N]) and torch.equal(c2[:, 2 * N:], q.x0[:, 2 * N:])
                for vt_L in (M, M // 2) if M % 2 == 0 else (M,):
                    c3, vt = q.run(shape, epi, ga, nseg=2, vt_L=vt_L)
                    t = vt.view(M // vt_L, N, -1)
                    assert torch.equal(t[:, :, :vt_L].transpose(1, 2).reshape(M, N), c2[:, N:2 * N])
                    assert bool((t[:, :, vt_L:] == 0).all())
                    assert torch.equal(c3[:, :N], c[:, :N]) and torch.equal(c3[:, N:], q.x0[:, N:])


@pytest.mark.parametrize("shape", [3, 4, 0])
@pytest.mark.parametrize("chunks", [2048, 2056, 8192])
def test_chunk_tables_up_to_the_longest(shape, chunks):
    """160 x 256 keeps room for 2048 chunk numbers beside its three slots; longer
    tables go to 128 x 256, whose room the longest (8192) fills."""
    say(f"gemm chunk table {chunks} shape={shape}")
    q = _Problem("bf16", 170, 292, chunks * 8, 0, chunks)
    c, _ = q.run(shape, RESIDUAL, KCH)
    y = q.x0[:, :q.N].double() + (q.gate[0].double() + q.gate[1].double()) * q.ref(KCH)
    _close(c[:, :q.N], y, 8e-3)


@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("ldc_pad", [0, 1, 5])
@pytest.mark.parametrize("k", [64, 192, 320, 1088])
def test_the_kernel_of_the_largest_problems(k, ldc_pad, out):
    """Plain bf16 operands at sizes whose choice is 256 x 256 (4001 x 8003 and 4001 x
    8004), through the operator: odd and even k-tile counts, rows that allow vector
    accesses (8004 + 0) and rows that do not, both output types."""
    import torch
    M, N = 4001, 8003 + (ldc_pad == 0)
    say(f"gemm 256x256 M={M} N={N} K={k} ldc+{ldc_pad} out={out}")
    gen = torch.Generator(device="cuda").manual_seed(k + ldc_pad)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda")
    a, b = rand(M, k).mul_(0.5).bfloat16(), rand(N, k).mul_(0.5).bfloat16()
    bias, gate = rand(N), rand(N)
    odt, tol = (torch.bfloat16, 8e-3) if out == "bf16" else (torch.float32, 1e-5)
    x0 = rand(M + 1, N + ldc_pad).to(odt)
    y = a.double() @ b.double().t() + bias
    for epi in (STORE, GELU, RESIDUAL):
        c = x0.clone()
        B.dif_gemm(a, b, c[:M, :N], epi, bias=bias, gate0=gate if epi == RESIDUAL else None)
        torch.cuda.synchronize()
        ref = y if epi == STORE else _gelu(y) if epi == GELU else x0[:M, :N].double() + gate * y
        _close(c[:M, :N], ref, tol)
        assert torch.equal(c[M], x0[M]) and torch.equal(c[:, N:], x0[:, N:])
