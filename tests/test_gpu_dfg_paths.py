"""The DFG's paths at the sizes where one takes over from the next, against the
oracle: one LDS block (two tiles of 4096 events), several blocks, blocks with
several tiles and cell copies (few activities), the global-atomics path for few
events of more than 64 activities (up to 16384), the bucketed path above it."""
import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import check_dfg, cols, note

pytestmark = pytest.mark.gpu


def _log(n, A, seed, mean=6):
    rng = np.random.default_rng(seed)
    case = rng.integers(0, max(1, n // mean), n).astype(np.int32) - 3
    act = np.minimum(rng.zipf(1.3, n) - 1, A - 1).astype(np.int32)
    ts = rng.integers(0, 50 * max(n, 1), n).astype(np.int64)
    return case, act, ts


@pytest.mark.parametrize("A", [1, 16, 45, 64, 65, 300])
@pytest.mark.parametrize("n", [0, 1, 3, 4096, 8192, 8193, 16384, 16385, 70001])
def test_path_edges(n, A):
    note(f"dfg paths n={n} A={A}")
    check_dfg(*_log(n, A, 100 * n + A), A)


@pytest.mark.parametrize("A", [2, 16, 33])
def test_many_tiles_per_block(A):
    n = 9_000_001                       # 2198 tiles on 256 blocks: copies of each cell
    note(f"dfg paths n={n} A={A}")
    check_dfg(*_log(n, A, 7 + A, mean=9), A)


@pytest.mark.parametrize("n,A", [(4096, 20), (30000, 20), (9000, 90), (40000, 90)])
@pytest.mark.parametrize("shift", [1, 3])
def test_columns_off_16_byte_alignment(n, A, shift):
    case, act, ts = _log(n, A, 11)
    order = np.lexsort((np.arange(n), ts, case))
    note(f"dfg paths unaligned n={n} A={A} shift={shift}")
    c, a, t = cols(*(np.concatenate([np.zeros(shift, x.dtype), x[order]]) for x in (case, act, ts)))
    c, a, t = c[shift:], a[shift:], t[shift:]
    prep = pm4g.pm4g_prepare(c.clone(), a.clone(), t.clone(), A, presorted=True)
    want = pm4g.dfg_to_host(pm4g.pm4g_dfg_prepared(prep), A)
    prep.case_s, prep.act_s, prep.ts_s = c, a, t
    got = pm4g.dfg_to_host(pm4g.pm4g_dfg_prepared(prep), A)
    for k in want:
        assert np.array_equal(np.asarray(got[k]), np.asarray(want[k]), equal_nan=k == "dt_mean"), k


@pytest.mark.parametrize("n,A", [(5000, 30), (50000, 30), (5000, 200), (50000, 200)])
def test_invalid_activity_in_a_prepared_log(n, A):
    case, act, ts = _log(n, A, 5)
    note(f"dfg paths invalid activity n={n} A={A}")
    prep = pm4g.pm4g_prepare(*cols(case, act, ts), A)
    prep.act_s[n - 2] = A
    o = pm4g.pm4g_dfg_prepared(prep)
    torch.cuda.synchronize()
    assert int(o["status"].item()) == pm4g.PM4G_E_RANGE
