"""The fold of the DFG's partial tables around its split by buckets of cells (32
and 256 buckets): values, and that just below 256 buckets a call takes no
longer than just above, where it folds more cells."""
import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, check_dfg, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A", [362, 363, 1024, 1025])
def test_fold_at_the_bounds(A):
    rng = np.random.default_rng(A)
    n = 60_000
    case = rng.integers(0, n // 12, n).astype(np.int32)
    act = (rng.random(n) ** 4 * A).astype(np.int32)
    note(f"fold: A={A}")
    check_dfg(case, act, rng.integers(0, 10**12, n).astype(np.int64), A)


def _time_us(A, n):
    g = torch.Generator(device=DEV)
    g.manual_seed(A)
    case = torch.arange(n, device=DEV, dtype=torch.int32) // 10
    act = torch.randint(0, A, (n,), generator=g, device=DEV, dtype=torch.int32)
    prep = pm4g.pm4g_prepare(case, act, torch.arange(n, device=DEV), A, presorted=True)
    out = pm4g.pm4g_dfg_prepared(prep)
    best = float("inf")
    for _ in range(15):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        pm4g.pm4g_dfg_prepared(prep, out=out)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("n", [20_000, 700_000])
def test_fewer_cells_take_no_longer(n):
    below, above = _time_us(1000, n), _time_us(1100, n)
    note(f"fold: n={n}: 1000 activities {below:.0f} us, 1100 activities {above:.0f} us")
    assert below <= 1.25 * above
