"""The order of the batched views' walks over tiles, on the CPU (walk_items_check.cpp)."""
import os
import shutil
import subprocess

import pytest

from paper_2204_04898_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_item_once_and_no_block_idle(tmp_path):
    if not os.path.exists(build.HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc is not installed")
    exe = str(tmp_path / "walk_items_check")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-x", "hip", "-I", build.CSRC,
                        os.path.join(ROOT, "tests", "walk_items_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-2000:]
    assert "0 failures" in r.stdout
