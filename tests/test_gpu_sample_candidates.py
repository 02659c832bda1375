"""Sampling's last steps with many candidates: lists of dozens to thousands that
one block ranks, and candidates beyond the list, selected among digit by digit
(fewer digit passes and shorter lists, by the test hooks; three passes leave two
or three candidates on such logs)."""
import contextlib

import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, note

pytestmark = pytest.mark.gpu


def _keys(seed, x):
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (x + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


@contextlib.contextmanager
def _hooks(passes, entries):
    L = pm4g.load()
    old = L.pm4g_debug_sample_passes(passes), L.pm4g_debug_sample_list(entries)
    try:
        yield
    finally:
        L.pm4g_debug_sample_passes(old[0])
        L.pm4g_debug_sample_list(old[1])


@pytest.mark.parametrize("by_events", [False, True])
@pytest.mark.parametrize("units,passes,entries", [
    (20_000, 1, -1),        # lists of about 78
    (900_000, 1, -1),       # of about 3500: every thread of the block ranks several
    (900_000, 2, -1),       # of about 14
    (1_500_000, 1, -1),     # about 5900: beyond the list
    (20_000, 1, 40), (20_000, 2, 0), (20_000, 3, 0), (20_000, 3, 1), (700, 1, 2), (900_000, 3, 0),
])
def test_candidates(units, passes, entries, by_events):
    seed = 4242
    rng = np.random.default_rng(units)
    if by_events:
        n, x = units, np.arange(units, dtype=np.uint64)
        case = np.sort(rng.integers(0, units // 4 + 1, n)).astype(np.int32)
    else:
        ids = np.unique(rng.integers(-(1 << 31), 1 << 31, units + units // 8))
        ids = np.sort(rng.choice(ids, units, replace=False)).astype(np.int32)
        x = ids.view(np.uint32).astype(np.uint64)
        case = np.repeat(ids, 1 + (np.arange(units) % 3 == 0))
        n = len(case)
    act, ts = np.zeros(n, np.int32), np.arange(n, dtype=np.int64)
    p = pm4g.pm4g_prepare(*(torch.from_numpy(c).to(DEV) for c in (case, act, ts)), 1, presorted=True)
    order = np.argsort(_keys(seed, x))
    note(f"sample candidates: units={units} by_events={by_events} passes={passes} list={entries}")
    for k in (1, 2, units // 3, units // 2 + 1, units - 1):
        with _hooks(passes, entries):
            q = pm4g.pm4g_sample(p, k, seed, by_events)
        m = int(q.case_off[int(q.n_cases.item())].item())
        if by_events:
            want = np.sort(order[:k])
        else:
            kept = np.zeros(units, bool)
            kept[order[:k]] = True
            want = np.flatnonzero(kept[np.searchsorted(ids, case)])
        assert int(q.status.item()) == 0 and m == len(want), k
        assert np.array_equal(q.ts_s[:m].cpu().numpy(), ts[want]), k
        assert np.array_equal(q.case_s[:m].cpu().numpy(), case[want]), k
