"""Variant grouping when nearly all cases share a sequence: the answer, and that
such a log takes no longer than one whose cases all differ (the members of a
variant meet in one block's memory first; a global atomic per case would queue
on one address)."""
import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, check_variants, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,L", [(64, 3), (65, 7), (700, 8), (5000, 9), (40, 3000)])
@pytest.mark.parametrize("seed", [0, 1])
def test_nearly_one_variant(C, L, seed):
    rng = np.random.default_rng(C + L + seed)
    seqs = np.tile(rng.integers(0, 6, L), (C, 1))
    odd = rng.integers(0, C, 3)
    seqs[odd, rng.integers(0, L, 3)] ^= 1                     # alike but for one event
    lens = np.full(C, L)
    lens[rng.integers(0, C)] -= 1                             # and but for the last
    if seed:
        lens[rng.integers(0, C, C // 3)] = 1
    keep = np.arange(L)[None, :] < lens[:, None]
    case = np.repeat(rng.permutation(C), lens).astype(np.int32)
    act, ts = seqs[keep].astype(np.int32), np.tile(np.arange(L), (C, 1))[keep].astype(np.int64)
    rows = rng.permutation(len(case))
    note(f"one variant: C={C} L={L} seed={seed}")
    check_variants(case[rows], act[rows], ts[rows], 8)


def _time_us(prep):
    o = pm4g.pm4g_variants_prepared(prep)
    best = float("inf")
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        pm4g.pm4g_variants_prepared(prep, out=o)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best, int(o["n_variants"].item())


@pytest.mark.parametrize("C,L", [(20_000, 500), (50_000, 60), (200_000, 50), (1_000_000, 12)])
def test_one_variant_takes_no_longer_than_many(C, L):
    g = torch.Generator(device=DEV)
    g.manual_seed(C)
    case = torch.arange(C, device=DEV, dtype=torch.int32).repeat_interleave(L)
    ts = torch.arange(C * L, device=DEV, dtype=torch.int64)
    times = []
    for rows in (1, C):
        act = torch.randint(0, 100, (rows, L), generator=g, device=DEV, dtype=torch.int32)
        act[:, 0] = 5
        prep = pm4g.pm4g_prepare(case, act.repeat(C // rows, 1).reshape(-1), ts, 100, presorted=True)
        us, variants = _time_us(prep)
        times.append(us)
        note(f"variants: C={C} L={L}, {variants} variants: {us:.0f} us")
        assert variants == (1 if rows == 1 else C)
    assert times[0] <= 1.15 * times[1], times
