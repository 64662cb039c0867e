"""The row kernels are bound by memory and keep a row in registers: none may spill
to scratch memory.  Compiles ``rowops.hip`` and reads the compiler's resource
remarks; the one exception is the widest bf16 LayerNorm (16 chunks per lane under
the 128 registers of a sixteen-wave workgroup)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2607_06631_amd", "csrc", "rowops.hip")
KNOWN = {"norm_kernelIDF16bLi16E": 11}   # registers it may spill


def test_row_kernels_do_not_spill(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    from paper_2607_06631_amd import build
    cmd = [hipcc, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c", SRC,
           "-o", str(tmp_path / "rowops.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    spills, name = {}, None
    for line in r.stderr.split("\n"):
        if m := re.search(r"Function Name: (\S+)", line):
            name = m.group(1)
        elif m := re.search(r"VGPRs Spill: (\d+)", line):
            spills[name] = int(m.group(1))
    assert sum("norm_kernel" in k for k in spills) >= 8
    for k, n in spills.items():
        assert n <= next((v for s, v in KNOWN.items() if "3dif11" + s in k), 0), (k, n)
