"""The pinned slots through which raw-log calls get their few words, on the CPU:
hostback_check.cpp runs them over stand-ins for the HIP calls they make."""
import os
import shutil
import subprocess

import pytest

from paper_2204_04898_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_slots(tmp_path):
    if not os.path.exists(build.HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc is not installed")
    exe = str(tmp_path / "hostback_check")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-x", "hip", "-I", build.CSRC,
                        os.path.join(ROOT, "tests", "hostback_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "0 failures" in r.stdout
