"""CSV code assignment around its row tiles (2048 rows; several tiles per block
above 1024 tiles), values first seen late, and the newline count that bounds
the rows, at sizes around its 16-byte words and off their alignment."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, note
from tests.test_gpu_csv import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 255, 2047, 2048, 2049, 30_011])
def test_tiles(rows):
    rng = np.random.default_rng(rows)
    case = rng.integers(0, max(1, rows // 3), rows)
    act = np.minimum(rng.zipf(1.5, rows), 40)
    act[rows // 2:] += (np.arange(rows - rows // 2) % 50 == 0)   # values that first occur in later tiles
    note(f"csv codes rows={rows}")
    _check(b"c,a,t\n" + b"".join(b"%d,act %d,%d\n" % x for x in zip(case, act, range(rows))))


def test_many_tiles_per_block():
    rows = 2048 * 1024 * 2 + 77
    rng = np.random.default_rng(3)
    case = rng.integers(0, 700_000, rows).astype(np.int64)
    act = rng.integers(0, 9, rows).astype(np.int64)
    act[-5:] = 9
    d = np.empty((rows, 12), np.uint8)
    d[:, 7], d[:, 9], d[:, 10], d[:, 11] = ord(","), ord(","), ord("5"), ord("\n")
    for k in range(7):
        d[:, k] = case // 10 ** (6 - k) % 10 + 48
    d[:, 8] = act + 48
    note(f"csv codes rows={rows}")
    g = pm4g.pm4g_ingest_csv(torch.from_numpy(d.reshape(-1)).to(DEV), 0, 1, 2, has_header=False)
    for got, values in ((g["case_code"], case), (g["act_code"], act)):
        u, first, inv = np.unique(values, return_index=True, return_inverse=True)
        rank = np.empty(len(u), np.int64)
        rank[np.argsort(first)] = np.arange(len(u))
        assert np.array_equal(got.cpu().numpy(), rank[inv])
    assert (g["n_rows"], g["n_acts"]) == (rows, 10)


@pytest.mark.parametrize("shift", [0, 1, 7])
@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 4096, 1_000_003, 9_000_001])
def test_newlines(n, shift):
    rng = np.random.default_rng(n + shift)
    x = torch.from_numpy(rng.choice(np.array([10, 11, 9, 138, 65, 0], np.uint8), n + shift)).to(DEV)[shift:]
    out = ctypes.c_int64(-1)
    ws = torch.empty(pm4g.load().pm4g_csv_newlines_workspace_bytes(), dtype=torch.uint8, device=DEV)
    rc = pm4g.load().pm4g_csv_newlines(ctypes.c_void_p(x.data_ptr()), n, ctypes.byref(out),
                                       ctypes.c_void_p(ws.data_ptr()), ws.numel(),
                                       ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0 and out.value == int((x == 10).sum())
