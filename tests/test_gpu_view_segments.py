"""Segments of a view's records that several blocks share, and their limits:
one record below and at the count from which a segment is split, a segment of
many parts, one whose cells are all start cells, and the record layout of logs
with very long cases, next to views whose segments are not split."""
import numpy as np
import pytest

from paper_2204_04898_amd import pm4g, synth
from tests.gpu_util import note
from tests.test_gpu_views import INT64_MAX, INT64_MIN, check_views

pytestmark = pytest.mark.gpu


def log_of(n, A, mean, seed, span=0):
    rng = np.random.default_rng(seed)
    lens = []
    while sum(lens) < n:
        lens.append(int(rng.geometric(1.0 / mean)))
    lens[-1] -= sum(lens) - n
    case = np.repeat(np.arange(len(lens), dtype=np.int32), lens)
    act = (rng.random(n) ** 3 * A).astype(np.int32)          # a few activities hold most events
    ts = rng.integers(-(1 << 40), 1 << 40, n, dtype=np.int64)
    if span:
        first = int(np.flatnonzero(np.asarray(lens) > 1)[0])
        at = int(np.flatnonzero(case == first)[0])
        ts[at], ts[at + 1] = -span // 2, span - span // 2
    perm = rng.permutation(n)
    return synth.Log(case=case[perm], act=act[perm], ts=ts[perm], n_activities=A, presorted=False,
                     lengths_by_code=np.asarray(lens, np.int64))


@pytest.mark.parametrize("launch", [0, 1])
@pytest.mark.parametrize("n,A,mean,span", [
    (65_535, 3, 8, 0), (65_536, 3, 8, 0), (65_537, 5, 8, 0),     # one bucket: not split, two parts
    (400_000, 40, 10, 0),                                        # one bucket, six parts
    (150_000, 64, 2, 0),                                         # the start cells alone: a second bucket, split
    (300_000, 90, 6, 1 << 53),                                   # two buckets, cells kept apart from the gaps
])
def test_split_segments(n, A, mean, span, launch):
    log = log_of(n, A, mean, n + A, span)
    C = int(log.case.max()) + 1
    rng = np.random.default_rng(5)
    V = 6
    lo = np.array([0, 0, C // 3, C - 2, 0, C // 2], np.int32)
    hi = np.array([C, C, C // 2, C, C // 100 + 1, C], np.int32)
    tl, th = np.full(V, INT64_MIN, np.int64), np.full(V, INT64_MAX, np.int64)
    tl[1], th[1] = -(1 << 38), 1 << 39
    masks = np.full((V, (A + 63) // 64), np.uint64(0xFFFFFFFFFFFFFFFF))
    masks[5] = rng.integers(0, 1 << 63, masks.shape[1]).astype(np.uint64)
    views = synth.Views(case_lo=lo, case_hi=hi, t_lo=tl, t_hi=th, masks=masks)
    note(f"split segments: N={n} A={A} launch={launch}")
    res = check_views(log, views, tuning=pm4g.BatchedTuning(launch=launch))
    assert res[0]["n_events"] == n


@pytest.mark.parametrize("launch", [0, 1])
@pytest.mark.parametrize("n,A,V,tile,widest", [
    (30_000, 90, 1501, 4096, 900),       # the segments' counters over several blocks, a last one cut short
    (2_300_000, 20, 5, 2048, 200_000),   # more tiles than the tile scan has threads
])
def test_places_over_blocks(n, A, V, tile, widest, launch):
    log = log_of(n, A, 12, n + V)
    C = int(log.case.max()) + 1
    rng = np.random.default_rng(8)
    lo = rng.integers(0, C, V).astype(np.int32)
    hi = (lo + rng.integers(0, widest, V)).astype(np.int32)
    tl = rng.integers(-(1 << 40), 1 << 39, V)
    th = tl + rng.integers(1, 1 << 41, V)
    masks = rng.integers(0, 1 << 63, (V, (A + 63) // 64)).astype(np.uint64)
    views = synth.Views(case_lo=lo, case_hi=hi, t_lo=tl, t_hi=th, masks=masks)
    note(f"view places: N={n} A={A} V={V} launch={launch}")
    sample = sorted({0, V - 1, *rng.integers(0, V, 40).tolist()})
    check_views(log, views, tuning=pm4g.BatchedTuning(launch=launch, tile_events=tile), sample=sample)
