"""The bound of the one-sided force partials over all set sizes, checked on the
host against the shapes the library chooses
(tests/c/partials_bound_check.cpp). No GPU needed."""

import os
import shutil
import subprocess

import pytest

from paper_2411_18889_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_partials_bound(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    _lib.lib()  # built
    libdir = os.path.dirname(_lib.LIB_PATH)
    exe = str(tmp_path / "partials_bound_check")
    r = subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(libdir, "csrc"),
                        os.path.join(ROOT, "tests", "c", "partials_bound_check.cpp"),
                        "-L", libdir, "-lnbody", "-Wl,-rpath," + libdir, "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.stdout, r.stderr)
