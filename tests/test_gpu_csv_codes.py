"""CSV code assignment around its row tiles (2048 rows; several tiles per block
above 1024 tiles), values first seen late, and the newline count that bounds
the rows, at sizes around its 16-byte words and off their alignment."""
import ctypes

import numpy as np
import pytest
import torch

import oracle

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


FORMS = ["2021-02-03T04:05:06", "2021-02-03 04:05:06", "2021-02-03T04:05:06Z", "2021-02-03T04:05:06.1", "2021-02-03T04:05",
         "2021-02-03T04:05:06,12Z", "2021-02-03T04:05:06.123456789", "2021-02-03T04:05:06.123456789Z", "2021-02-03",
         "2021-02-03T04:05:06.12345678Z", "2021-02-03T04:05:06.123+01:30", "2021-02-03T04:05:06-02", "2000-02-29T23:59:59.9Z",
         "1969-12-31T23:59:59.999Z", "1800-01-01T00:00:00.000000001Z", "2021-02-03T04:05:06.12345Z", "\"2021-02-03T04:05:06.5\""]
BAD = ["2021-02-30T04:05:06Z", "2021-02-03T24:05:06Z", "2021-02-03T04:60:06.1", "2021-02-03T04:05:06.", "2021-02-03T04:05:06.Z",
       "2021-02-03T04:05:06.1234567890", "2021-02-03T04:05:06.12a", "2021-02-03T04:05:06ZZ", "2021-13-03T04:05:06", "202a-02-03T04:05:06",
       "2021-02-03T04:05:06.1234567890Z", "2021-02-03T0:05:06.00", "2021/02/03T04:05:06"]


@pytest.mark.parametrize("scale", [0, 3, 6, 9])
def test_date_time_forms(scale):
    rows = [b"%d,a%d,%s" % (k % 5, k % 3, f.encode()) for k, f in enumerate(FORMS * 20)]
    note(f"csv date-time forms, scale {scale}")
    _check(b"c,a,t\n" + b"\n".join(rows) + b"\n", ts_iso=True, ts_scale=scale)


@pytest.mark.parametrize("bad", BAD)
def test_bad_date_times(bad):
    text = b"c,a,t\n" + b"".join(b"%d,x,2021-02-03T04:05:06.5Z\n" % k for k in range(70)) + b"7,y," + bad.encode() + b"\n1,x,2021-01-01\n"
    with pytest.raises(oracle.CsvParseError) as e:
        oracle.ingest_csv(text, 0, 1, 2, ts_iso=True)
    assert e.value.row == 70
    with pytest.raises(pm4g.Pm4gError) as g:
        pm4g.pm4g_ingest_csv(torch.frombuffer(bytearray(text), dtype=torch.uint8).to(DEV), 0, 1, 2, ts_iso=True)
    assert g.value.code == pm4g.PM4G_E_PARSE and "row 70" in str(g.value)


@pytest.mark.parametrize("width", [20, 70, 75, 150, 310, 620, 800, 30_000])
def test_row_lengths_around_the_stage(width):
    rng = np.random.default_rng(width)
    rows = 700 if width < 10_000 else 40
    note(f"csv rows of about {width} bytes")
    text = b"x,c,a,t\n" + b"".join(b"%s,%d,a%d,%d\n" % (b"p" * int(rng.integers(0, 2 * width - 20)), k % 90, k % 7, k)
                                   for k in range(rows))
    _check(text, cols=(1, 2, 3))
