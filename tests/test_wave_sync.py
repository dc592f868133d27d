"""The kernels whose lanes read LDS records that other lanes of their wave
stored, without a workgroup barrier: in the device code as the front end hands
it to the optimiser, every wave barrier stands between a release and an acquire
fence of wavefront scope, so that neither the stores nor the reads may be moved
across it. No GPU needed."""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_18889_amd", "csrc")


@pytest.mark.parametrize("src", ("force_sym.hip", "adjoint_sym.hip", "adjoint_sym_group.hip"))
def test_wave_barriers_are_fenced(src, tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = str(tmp_path / "device.ll")
    r = subprocess.run([hipcc, "-O3", "-std=c++17", "--offload-arch=gfx950", "--cuda-device-only",
                        "-Xclang", "-disable-llvm-passes", "-S", "-emit-llvm",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(CSRC, src), "-o", out],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    with open(out) as fh:
        code = [l.strip() for l in fh if l.strip()]
    at = [i for i, l in enumerate(code) if re.match(r"(tail )?call void @llvm\.amdgcn\.wave\.barrier", l)]
    assert at
    for i in at:
        assert code[i - 1].startswith('fence syncscope("wavefront") release')
        assert code[i + 1].startswith('fence syncscope("wavefront") acquire')
