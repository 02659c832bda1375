"""The directly-follows event filter and the containment tests of the case
filter: pair sets held in LDS and in memory (the limit lies between 572 and
573 activities), cases across lanes, waves and steps, and an activity column
that is not 16-byte aligned."""
import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, cols, note

pytestmark = pytest.mark.gpu


def words_of(bits):
    m = np.zeros((bits.size + 63) // 64 * 64, bool)
    m[:bits.size] = bits
    return torch.from_numpy(np.packbits(m, bitorder="little").view(np.int64).copy()).to(DEV)


def events_of(q):
    C = int(q.n_cases.item())
    k = int(q.case_off[C].item())
    assert int(q.status.item()) == 0
    return q.ts_s[:k].cpu().numpy()


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("A", [3, 64, 512, 572, 573, 700])
def test_pair_sets(A, shift):
    rng = np.random.default_rng(A)
    lens = np.concatenate([[1, 2, 63, 64, 65, 255, 257, 300], rng.integers(1, 30, 2500)])
    case = np.repeat(np.arange(lens.size, dtype=np.int32), lens)
    n = case.size
    act, ts = rng.integers(0, A, n).astype(np.int32), np.arange(n, dtype=np.int64)   # a timestamp names its event
    p = pm4g.pm4g_prepare(*cols(case, act, ts), A, presorted=True)
    room = torch.zeros(n + 4, dtype=torch.int32, device=DEV)
    room[shift:shift + n] = p.act_s
    p.act_s = room[shift:shift + n]
    bits = rng.random(A * A) < 3.0 / 20
    path, mask = words_of(bits), rng.random(A) < 2.0 / A
    mask[act[-1]] = True
    note(f"pair sets A={A} shift={shift}")
    same = case[1:] == case[:-1]
    hit = np.zeros(n + 1, bool)                              # hit[i]: the pair (i - 1, i)
    hit[1:n] = same & bits[act[:-1].astype(np.int64) * A + act[1:]]
    for side in (0, 1):
        pair = hit[:n] if side == 0 else hit[1:]
        for keep in (True, False):
            assert np.array_equal(events_of(pm4g.pm4g_filter_df_events(p, path, side, keep)), ts[pair == keep])
    has_path = np.zeros(lens.size, bool)
    has_path[case[hit[:n]]] = True
    has_act = np.zeros(lens.size, bool)
    has_act[case[mask[act]]] = True
    am = words_of(mask)
    for got, want in ((pm4g.pm4g_filter_cases(p, path_mask=path), has_path),
                      (pm4g.pm4g_filter_cases(p, path_mask=path, path_keep=False), ~has_path),
                      (pm4g.pm4g_filter_cases(p, act_mask=am), has_act),
                      (pm4g.pm4g_filter_cases(p, act_mask=am, path_mask=path), has_act & has_path)):
        assert np.array_equal(events_of(got), ts[want[case]])
