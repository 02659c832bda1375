"""Workspace sizes never shrink with the log: a buffer sized for a caller's
largest log serves every smaller one (no GPU work)."""
import ctypes

import pytest

from paper_2204_04898_amd import pm4g

TILE = 4096


def _events():
    """Ascending event counts, dense around the bounds of tiles and of the rules
    that change with their number."""
    around = {1, 2, 3, 256, 1024, 3072, 16384, 10**6, 10**7, 98_969_504, 2**31 - 2}
    around |= {k * TILE for k in (1, 2, 3, 4, 8, 63, 64, 65, 66, 128, 255, 256, 257, 1024, 1025, 24163)}
    ns = {0, 2**31 - 1}
    for n in around:
        ns |= {m for m in range(n - 3, n + 4) if 0 <= m < 2**31}
    return sorted(ns)


@pytest.mark.parametrize("op", ["PREPARE", "DFG", "DFG_PREPARED", "VARIANTS", "VARIANTS_PREPARED"])
@pytest.mark.parametrize("A", [1, 16, 64, 65, 300, 512, 4096])
def test_log_operations(op, A):
    L = pm4g.load()
    sizes = [int(L.pm4g_workspace_bytes(getattr(pm4g, "OP_" + op), n, A, 0)) for n in _events()]
    assert sizes[0] > 0
    drops = [(n, a, b) for n, a, b in zip(_events()[1:], sizes, sizes[1:]) if b < a]
    assert not drops, drops[:5]


@pytest.mark.parametrize("name", ["filter", "filter_cases", "sample"])
def test_filters(name):
    f = getattr(pm4g.load(), f"pm4g_{name}_workspace_bytes")
    sizes = [int(f(n)) for n in _events()]
    assert sizes[0] > 0 and sizes == sorted(sizes)


@pytest.mark.parametrize("A,V", [(20, 1), (20, 31), (20, 32), (512, 48), (1024, 4096)])
@pytest.mark.parametrize("tile", [0, 2048])
def test_views(A, V, tile):
    L = pm4g.load()
    t = pm4g.BatchedTuning(tile_events=tile)
    sizes = [int(L.pm4g_batched_workspace_bytes(n, A, V, ctypes.byref(t))) for n in _events()]
    assert sizes[0] > 0 and sizes == sorted(sizes)


@pytest.mark.parametrize("A", [5, 64, 65, 1000])
def test_efg(A):
    sizes = [int(pm4g.load().pm4g_efg_workspace_bytes(n, A)) for n in _events()]
    assert sizes[0] > 0 and sizes == sorted(sizes)


def test_ingestion():
    L = pm4g.load()
    rows = [r for r in _events() if r <= 10**8]
    for size in (lambda r: L.pm4g_ingest_csv_workspace_bytes(10**9, r), lambda r: L.pm4g_ingest_csv_workspace_bytes(r, 1000),
                 lambda r: L.pm4g_ingest_parquet_workspace_bytes(10**9, r)):
        sizes = [int(size(r)) for r in rows]
        assert sizes[-1] > 0 and sizes == sorted(sizes)
