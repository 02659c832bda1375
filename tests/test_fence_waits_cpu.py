"""What a block announces to others while they run (grid barriers of the
persistent launch, tables of shared segments) must have left its L2: in the
compiled code each write-back of the L2 is waited for before the next store or
atomic.  Compiles the batched views' kernels to assembly; nothing runs."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2204_04898_amd import build

STORE = re.compile(r"(global|flat|buffer)_(store|atomic)")
WAIT = re.compile(r"s_waitcnt (0$|.*vmcnt\(0\))")


def unwaited(lines):
    """(line, store) of every write-back followed by a store before a wait."""
    bad = []
    for i, line in enumerate(lines):
        if not line.startswith("buffer_wbl2"):
            continue
        for nxt in lines[i + 1:]:
            if WAIT.match(nxt) or nxt.startswith(("s_endpgm", "s_setpc")):
                break
            if STORE.match(nxt):
                bad.append((i, nxt))
                break
    return bad


def test_the_check_itself():
    assert unwaited(["buffer_wbl2 sc1", "buffer_inv sc1", "flat_store_dword v[0:1], v2"])
    assert not unwaited(["buffer_wbl2 sc1", "s_waitcnt vmcnt(0) lgkmcnt(0)", "flat_store_dword v[0:1], v2"])


def test_write_backs_are_waited_for(tmp_path):
    if not os.path.exists(build.HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc is not installed")
    asm = str(tmp_path / "views.s")
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall")]
    r = subprocess.run([build.HIPCC, *flags, "-S", "--cuda-device-only", os.path.join(build.CSRC, "views.hip"), "-o", asm],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(asm) as f:
        lines = [l.strip() for l in f]
    assert sum(l.startswith("buffer_wbl2") for l in lines) >= 4   # the barriers' and the shared segments'
    assert not unwaited(lines), unwaited(lines)[:5]
