"""The case passes' digits and rows: one tile (no histograms), few tiles (rows
added up by the scatter) and many, ranges around 8, 9, 10, 17, 18, 19 and 25
bits, raw rows turned by a case minimum, packed and separate (12 + 21 bits)
activities, with and without the row order; against a stable sort."""
import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import cols, note

pytestmark = pytest.mark.gpu
TILE, FEW = 4096, 64


@pytest.mark.parametrize("A,rows", [(30, False), (30, True), (4096, False)])
@pytest.mark.parametrize("n,span", [
    (1, 1), (TILE, 1), (TILE, 256), (TILE, 257), (TILE - 3, 1 << 10), (TILE, (1 << 10) + 1),
    (TILE + 1, 256), (TILE + 1, 512), (3 * TILE, 1 << 10), (FEW * TILE, 1 << 16), (FEW * TILE, (1 << 20) - 7),
    (FEW * TILE + 1, 1 << 16), (FEW * TILE + 1, 1 << 17), (300_000, 1 << 18), (300_000, (1 << 18) + 1),
    (300_000, 1 << 25), (TILE, 1 << 21), (100_000, 1 << 21), (4 * TILE, 700), (4 * TILE + 1, 700),
])
def test_case_digits(n, span, A, rows):
    rng = np.random.default_rng(n + span + A)
    first = -12_345
    case = (first + rng.integers(0, span, n)).astype(np.int32)
    case[:2] = [first, first + span - 1][:n]
    act = rng.integers(0, A, n).astype(np.int32)
    ts = rng.integers(0, 1000, n, dtype=np.int64)         # many ties: the row order decides
    note(f"case digits: n={n} span={span} A={A} rows={rows}")
    p = pm4g.pm4g_prepare(*cols(case, act, ts), A, rows=rows)
    order = np.lexsort((np.arange(n), ts, case))
    C = int(p.n_cases.item())
    assert C == np.unique(case).size
    for got, want in ((p.case_s, case), (p.act_s, act), (p.ts_s, ts)):
        assert np.array_equal(got.cpu().numpy(), want[order])
    if rows:
        assert np.array_equal(p.row.cpu().numpy(), order)
    assert torch.equal(p.case_code[:C].cpu(), torch.from_numpy(np.unique(case)))
