"""Raw logs with a case beyond the per-case sort's window: the DFG that is
queued before this is known reads no event, so the call's DFG stages take as
long as those of a log without such a case, not twice as long."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import check_dfg, cols, note

pytestmark = pytest.mark.gpu


def _dfg_stages_ms(call):
    L = pm4g.load()
    k = L.pm4g_profile_stage_count()
    ms = (ctypes.c_double * k)()
    best = float("inf")
    for _ in range(8):
        L.pm4g_profile_enable(1)
        try:
            call()
            torch.cuda.synchronize()
            assert L.pm4g_profile_read(ms, None, k) == pm4g.PM4G_OK
        finally:
            L.pm4g_profile_enable(0)
        best = min(best, sum(ms[i] for i in range(k) if L.pm4g_profile_stage_name(i).decode().startswith("dfg_")))
    return best


@pytest.mark.parametrize("A", [50, 100])
def test_work_queued_for_a_long_case(A):
    n = 20_000_000
    rng = np.random.default_rng(A)
    case = rng.integers(0, n // 10, n).astype(np.int32)
    act, ts = rng.integers(0, A, n).astype(np.int32), rng.integers(0, 10**12, n)
    c, a, t = cols(case, act, ts)
    even = _dfg_stages_ms(lambda: pm4g.pm4g_dfg(c, a, t, A))
    c[:5000] = 7
    long = _dfg_stages_ms(lambda: pm4g.pm4g_dfg(c, a, t, A))
    note(f"raw fallback A={A}: DFG stages {even:.3f} ms, with a long case {long:.3f} ms")
    assert long <= 1.5 * even


@pytest.mark.parametrize("A", [20, 80, 1000])
@pytest.mark.parametrize("n", [3073, 16_384, 16_385, 300_000])
def test_one_case(n, A):
    rng = np.random.default_rng(n)
    note(f"raw fallback one case n={n} A={A}")
    check_dfg(np.full(n, -9, np.int32), rng.integers(0, A, n).astype(np.int32), rng.integers(0, n, n), A)
