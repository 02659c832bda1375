"""The DFG of a few thousand events of many activities when pairs and starts are
far from even: values, and that a log of one pair takes no more than twice the
time of one whose pairs all differ (its lanes add up before they touch memory)."""
import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, check_dfg, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("A", [65, 300])
@pytest.mark.parametrize("n", [1, 255, 257, 16_384])
@pytest.mark.parametrize("kind", ["one", "two", "most", "four", "starts", "bad"])
def test_uneven_pairs(n, A, kind):
    rng = np.random.default_rng(n + A)
    case = np.sort(rng.integers(0, n // 9 + 1, n)).astype(np.int32)
    act = {"one": np.zeros(n), "two": np.arange(n) % 2, "most": np.where(rng.random(n) < 0.8, 3, rng.integers(0, A, n)),
           "four": np.arange(n) // 3 % 17, "starts": np.zeros(n), "bad": np.zeros(n)}[kind].astype(np.int32)
    if kind == "starts":
        case = np.arange(n, dtype=np.int32)
    ts = np.cumsum(rng.integers(0, 1 << 55, n)) if n < 100 else rng.integers(-(1 << 62), 1 << 62, n)
    note(f"few events: n={n} A={A} {kind}")
    if kind == "bad":
        act[n // 2] = A
        c, a, t = (torch.from_numpy(x).to(DEV) for x in (case, act, np.sort(ts)))
        with pytest.raises(pm4g.Pm4gError) as e:
            pm4g.pm4g_dfg(c, a, t, A)
        assert e.value.code == pm4g.PM4G_E_RANGE
        return
    check_dfg(case, act, ts, A)


def _time_us(act, A):
    n = len(act)
    case = torch.arange(n, device=DEV, dtype=torch.int32) // 8
    prep = pm4g.pm4g_prepare(case, act, torch.arange(n, device=DEV), A, presorted=True)
    out = pm4g.pm4g_dfg_prepared(prep)
    best = float("inf")
    for _ in range(30):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        pm4g.pm4g_dfg_prepared(prep, out=out)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("A", [65, 1000])
def test_one_pair_takes_no_longer(A):
    n = 16_384
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    even = _time_us(torch.randint(0, A, (n,), generator=g, device=DEV, dtype=torch.int32), A)
    one = _time_us(torch.zeros(n, dtype=torch.int32, device=DEV), A)
    note(f"few events: A={A}: even pairs {even:.0f} us, one pair {one:.0f} us")
    assert one <= 2 * even
