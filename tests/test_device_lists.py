"""The lists the kernels read (thread-bit lanes, phase tables, byte offsets, supports, gradient groups) against the
planner's own, over many circuits and tile shapes: tests/engine_emu/device_lists.cpp, compiled from the library's host
source.  Needs hipcc (host compilation only) and the built library; no GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2508_13615_amd")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_device_lists_say_what_the_planner_says(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "libsv.so")):
        pytest.skip("libsv.so not built")
    out = str(tmp_path / "device_lists")
    cmd = [HIPCC, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
           os.path.join(HERE, "engine_emu", "device_lists.cpp"), "-o", out, "-L", PKG, "-lsv", f"-Wl,-rpath,{PKG}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([out], capture_output=True, text=True, timeout=600)
    print(r.stdout[-4000:])
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-2000:]
    assert "all ok (0 errors)" in r.stdout
