"""Workspace slices against the kernels that index them, on the CPU (ws_slices_check.cpp)."""
import os
import shutil
import subprocess

import pytest

from paper_2204_04898_amd import build, pm4g

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build(tmp_path):
    if not os.path.exists(build.HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc is not installed")
    pm4g.load()   # the library must be built
    exe = str(tmp_path / "ws_slices_check")
    r = subprocess.run([build.HIPCC, *[f for f in build.FLAGS if f != "-O3"], "-O1", "-I", build.CSRC,
                        os.path.join(ROOT, "tests", "ws_slices_check.cpp"), "-L", build.HERE, "-lpm4g",
                        "-Wl,-rpath," + build.HERE, "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


def test_every_slice_holds_what_its_kernels_index(tmp_path):
    r = subprocess.run([_build(tmp_path)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-3000:]
    assert "0 failures" in r.stdout and "FAIL" not in r.stdout
