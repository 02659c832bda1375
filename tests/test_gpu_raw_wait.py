"""Raw-log calls whose later work is queued before the host knows how the sort
went: a case beyond the sort's window among short ones (the work runs again
after the fallback), logs around the window size, ordered logs used in place,
false claims and invalid activities reported all the same, several threads."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2204_04898_amd import pm4g
from tests.gpu_util import (assert_dfg_equal, assert_variants_equal, check_dfg, check_prepare, check_variants, cols,
                            note)

pytestmark = pytest.mark.gpu


def _log(n, A, seed, long=0):
    rng = np.random.default_rng(seed)
    case = rng.integers(0, max(1, n // 7), n).astype(np.int32)
    if long:
        case[rng.permutation(n)[:long]] = n // 20
    return case, rng.integers(0, A, n).astype(np.int32), rng.integers(0, 3 * n, n).astype(np.int64)


@pytest.mark.parametrize("A", [12, 90])
@pytest.mark.parametrize("n,long", [(40_000, 2100), (40_000, 5000), (3072, 3000), (3073, 3073), (3072, 0), (3073, 0)])
def test_long_case_after_queued_work(n, long, A):
    note(f"raw wait n={n} long={long} A={A}")
    log = _log(n, A, n + long + A, long)
    check_dfg(*log, A)
    check_variants(*log, A)
    check_prepare(*log, A)


@pytest.mark.parametrize("n,A", [(1, 5), (9_000, 5), (9_000, 80), (60_000, 80)])
def test_ordered_log_in_place(n, A):
    case, act, ts = _log(n, A, n)
    order = np.lexsort((np.arange(n), ts, case))
    note(f"raw wait ordered n={n} A={A}")
    log = case[order], act[order], ts[order]
    check_dfg(*log, A, presorted=True)
    check_variants(*log, A, presorted=True)
    c, a, t = cols(*log)
    if n > 1:
        for bad, code in (((c.flip(0), a, t.flip(0)), pm4g.PM4G_E_NOT_SORTED),
                          ((c, torch.where(torch.arange(n, device=c.device) == n - 2, A, a).int(), t), pm4g.PM4G_E_RANGE)):
            for call in (pm4g.pm4g_dfg, pm4g.pm4g_variants, pm4g.pm4g_prepare):
                with pytest.raises(pm4g.Pm4gError) as e:
                    call(*bad, A, presorted=True)
                assert e.value.code == code
    check_dfg(*log, A, presorted=True)


def test_threads_with_their_own_streams():
    A = 20
    logs = [_log(3_000 * (k + 1), A, k, 2500 if k % 3 == 2 else 0) for k in range(6)]
    want = [(oracle.dfg(*l, A), oracle.variants(*l, A)) for l in logs]
    errors = []

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                c = cols(*logs[k])
                for _ in range(5):
                    d = pm4g.pm4g_dfg(*c, A, stream=s)
                    v = pm4g.pm4g_variants(*c, A, stream=s)
                    s.synchronize()
                    assert_dfg_equal(pm4g.dfg_to_host(d, A), want[k][0], A)
                    assert_variants_equal(pm4g.variants_to_host(v, want[k][1]["n_cases"]), want[k][1])
        except Exception as e:   # reported by the test, not by the thread
            errors.append((k, repr(e)))

    note("raw wait threads")
    ts = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
