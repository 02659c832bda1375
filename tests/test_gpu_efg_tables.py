"""The eventually-follows sums on both sides of the narrow table's gap bound
(2^44 time units per case), with gaps at the bound in every word, sources
whose pairs end inside a lane group's steps, and several passes per entry."""
import numpy as np
import pytest

from paper_2204_04898_amd import pm4g
from tests.gpu_util import note
from tests.test_gpu_efg import _check

pytestmark = pytest.mark.gpu

B = 2**44


@pytest.mark.parametrize("top", [B - 1, B, B + 1, 2**24 - 1, 2**24, 2**22, 1, 0])
@pytest.mark.parametrize("A", [1, 3, 70])
def test_gap_bounds(top, A):
    rng = np.random.default_rng(top % 1000 + A)
    case = np.repeat(np.arange(40), 50)
    ts = rng.choice(np.array([0, top, top // 2, max(top - 1, 0)]), case.size)
    ts[::50], ts[1::50] = 0, top
    note(f"efg gaps up to {top}, A={A}")
    _check(case, rng.integers(0, A, case.size), ts, A)


@pytest.mark.parametrize("lengths", [[2] * 500, [1, 2, 3, 4, 5, 6, 7, 8, 9, 10] * 30, [63, 64, 65, 66] * 5, [700], [1] * 200 + [300]])
@pytest.mark.parametrize("A", [5, 90])
def test_source_ends(lengths, A):
    rng = np.random.default_rng(len(lengths) + A)
    case = np.repeat(np.arange(len(lengths)), lengths)
    note(f"efg case lengths {lengths[:4]}..., A={A}")
    act, ts = rng.integers(0, A, case.size), rng.integers(0, 10**7, case.size)
    _check(case, act, ts, A)
    for wide in (False, True):
        old = pm4g.load().pm4g_debug_efg_pass_pairs(37)
        try:
            _check(case, act, ts * (B if wide else 1), A)
        finally:
            pm4g.load().pm4g_debug_efg_pass_pairs(old)
