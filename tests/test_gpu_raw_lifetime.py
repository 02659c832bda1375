"""A raw log's columns on a stream of their own: when a call on another stream
has returned, its kernels may still read them, so memory that the caller drops
right after the call must not be handed to new tensors before that stream has
passed."""
import numpy as np
import pytest
import torch

import oracle
from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, assert_dfg_equal, note

pytestmark = pytest.mark.gpu


def _busy(stream):
    """Some tens of milliseconds of work queued on the stream."""
    with torch.cuda.stream(stream):
        x = torch.zeros(1 << 27, dtype=torch.float32, device=DEV)
        for _ in range(100):
            x.add_(1.0)
        done = torch.cuda.Event()
        done.record()
    return done


@pytest.mark.parametrize("n", [1500, 40_000])
@pytest.mark.parametrize("presorted", [False, True])
@pytest.mark.parametrize("call", ["pm4g_prepare", "pm4g_dfg", "pm4g_variants"])
def test_columns_dropped_after_the_call(call, presorted, n):
    A = 9
    rng = np.random.default_rng(n)
    case = rng.integers(0, n // 5, n).astype(np.int32)
    act, ts = rng.integers(0, A, n).astype(np.int32), rng.integers(0, 10**6, n)
    if presorted:
        rows = np.lexsort((np.arange(n), ts, case))
        case, act, ts = case[rows], act[rows], ts[rows]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    cols = [torch.from_numpy(x).to(DEV) for x in (case, act, ts)]
    where = {t.data_ptr() for t in cols}
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    out = getattr(pm4g, call)(*cols, A, presorted=presorted, stream=s)
    done = _busy(s)
    del cols
    fresh = [torch.zeros(n, dtype=d, device=DEV) for d in (torch.int32, torch.int32, torch.int64)]
    note(f"raw lifetime {call} n={n} presorted={presorted}")
    assert not done.query(), "the stream had passed already: nothing was tested"
    assert not where & {t.data_ptr() for t in fresh}
    s.synchronize()
    if call == "pm4g_dfg":
        assert_dfg_equal(pm4g.dfg_to_host(out, A), oracle.dfg(case, act, ts, A), A)
