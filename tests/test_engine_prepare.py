"""The pass kernels' dynamic-LDS limit only grows, also when two threads raise it at once (tests/engine_emu/prepare.cpp,
run against the built library with the HIP call replaced; no GPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2508_13615_amd")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_limit_grows_under_two_threads(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "libsv.so")):
        pytest.skip("libsv.so not built")
    out = str(tmp_path / "prepare")
    cmd = [HIPCC, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
           os.path.join(HERE, "engine_emu", "prepare.cpp"), "-o", out, "-L", PKG, "-lsv", f"-Wl,-rpath,{PKG}",
           "-rdynamic", "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]
