"""The walks' ways through a tile: a view per wave and views shared by waves
(many and few views on a tile), cases that go on across slices and tiles, one
bucket of cells and several, and both classes of activity counts."""
import numpy as np
import pytest

from paper_2204_04898_amd import pm4g, synth
from tests.gpu_util import note
from tests.test_gpu_views import INT64_MAX, INT64_MIN, check_views

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,launch", [(4096, 1), (2048, 1), (4096, 0)])
@pytest.mark.parametrize("V", [3, 45])
@pytest.mark.parametrize("A", [16, 63, 64, 512, 513])
def test_walks(A, V, tile, launch):
    rng = np.random.default_rng(A * 100 + V)
    lens = [700, 1, 511, 513, 1025, 5, 3000, 64, 63, 2] + list(rng.integers(1, 60, 300)) + [1500]
    case = np.repeat(np.arange(len(lens), dtype=np.int32) * 3, lens)
    n = case.size
    act = (rng.random(n) ** 2 * A).astype(np.int32)
    act[rng.integers(0, n, 5)] = A - 1
    ts = rng.integers(0, 10**7, n, dtype=np.int64)
    perm = rng.permutation(n)
    log = synth.Log(case=case[perm], act=act[perm], ts=ts[perm], n_activities=A, presorted=False,
                    lengths_by_code=np.asarray(lens, np.int64))
    top = int(case.max()) + 1
    lo = rng.integers(0, 12, V).astype(np.int32)
    hi = (lo + rng.integers(1, top, V)).astype(np.int32)
    tl = rng.integers(0, 9 * 10**6, V)
    th = tl + rng.integers(10**4, 10**7, V)            # down to a few kept events per slice
    lo[0], hi[0], tl[0], th[0] = 0, top, INT64_MIN, INT64_MAX
    masks = rng.integers(0, 1 << 63, (V, (A + 63) // 64)).astype(np.uint64)
    masks[0] = np.uint64(0xFFFFFFFFFFFFFFFF)
    masks[1] &= np.uint64(0x0101010101010101)
    views = synth.Views(case_lo=lo, case_hi=hi, t_lo=tl, t_hi=th, masks=masks)
    note(f"view walks: A={A} V={V} tile={tile} launch={launch}")
    res = check_views(log, views, tuning=pm4g.BatchedTuning(tile_events=tile, launch=launch))
    assert res[0]["n_events"] == n


@pytest.mark.parametrize("launch", [0, 1])
@pytest.mark.parametrize("n,V", [(5000, 31), (5000, 32), (5000, 700), (200_000, 300), (1_050_000, 40)])
def test_tiles_shared_by_blocks(n, V, launch):
    """Few tiles under many views: several blocks per tile (2 to 257 tiles, below
    and at the limits, a share cut short)."""
    rng = np.random.default_rng(n + V)
    A = 30
    case = np.sort(rng.integers(0, n // 9 + 1, n)).astype(np.int32)
    act = rng.integers(0, A, n).astype(np.int32)
    ts = rng.integers(0, 10**6, n, dtype=np.int64)
    log = synth.Log(case=case, act=act, ts=ts, n_activities=A, presorted=False,
                    lengths_by_code=np.bincount(case))
    top = int(case.max()) + 1
    lo = rng.integers(0, max(1, top // 2), V).astype(np.int32)
    hi = (lo + rng.integers(1, top, V)).astype(np.int32)
    tl = rng.integers(0, 9 * 10**5, V)
    th = tl + rng.integers(10**3, 10**5, V)
    masks = rng.integers(0, 1 << 30, (V, 1)).astype(np.uint64)
    views = synth.Views(case_lo=lo, case_hi=hi, t_lo=tl, t_hi=th, masks=masks)
    note(f"shared tiles: N={n} V={V} launch={launch}")
    sample = sorted({0, V - 1, *rng.integers(0, V, 25).tolist()})
    check_views(log, views, tuning=pm4g.BatchedTuning(launch=launch), sample=sample)
