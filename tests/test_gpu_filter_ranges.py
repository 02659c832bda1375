"""Event and case filters and sampling around their block ranges (4096-event
tiles, 512-case steps), capacities of exactly the kept events and one less,
views at the ends of the case range, and case ids whose sampling keys share
their leading bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2204_04898_amd import pm4g
from tests.gpu_util import DEV, cols, note

pytestmark = pytest.mark.gpu

M64 = 2**64 - 1


def _log(n, A, seed, mean=5):
    rng = np.random.default_rng(seed)
    case = rng.integers(-3, max(1, n // mean), n).astype(np.int32)
    return case, rng.integers(0, A, n).astype(np.int32), rng.integers(0, 9 * max(n, 1), n).astype(np.int64)


def _host(q):
    C = int(q.n_cases.item())
    off = q.case_off[:C + 1].cpu().numpy()
    k = int(off[C])
    return (q.case_s[:k].cpu().numpy(), q.act_s[:k].cpu().numpy(), q.ts_s[:k].cpu().numpy(), off,
            q.case_code[:C].cpu().numpy(), int(q.status.item()))


def _expect(h, keep):
    """Kept positions of a formatted log as a formatted log."""
    c, a, t = h["case_s"][keep], h["act_s"][keep], h["ts_s"][keep]
    code, first = np.unique(c, return_index=True)
    return c, a, t, np.append(np.sort(first), len(c)), code, 0


def _same(got, want):
    for g, w in zip(got, want):
        assert np.array_equal(g, w), (g, w)


@pytest.mark.parametrize("n", [1, 4095, 4096, 4097, 8192, 70_001])
def test_event_filters(n):
    A = 9
    log = _log(n, A, n)
    h = oracle.prepare(*log, A)
    p = pm4g.pm4g_prepare(*cols(*log), A)
    rng = np.random.default_rng(n + 1)
    bits = rng.random(A * A) < 0.5
    words = torch.from_numpy(np.packbits(np.pad(bits, (0, 128 - A * A)), bitorder="little").view(np.int64).copy()).to(DEV)
    c, a = h["case_s"], h["act_s"]
    for side in (0, 1):
        pair = np.zeros(n, bool)
        same = c[1:] == c[:-1]
        hit = same & bits[a[:-1].astype(np.int64) * A + a[1:]]
        (pair[1:] if side == 0 else pair[:-1])[:] = hit
        for keep in (True, False):
            want = np.flatnonzero(pair == keep)
            note(f"filter ranges n={n} side={side} keep={keep}: {len(want)} kept")
            _same(_host(pm4g.pm4g_filter_df_events(p, words, side, keep)), _expect(h, want))
            if len(want) > 1:   # an output of capacity 0 has no arrays and is refused
                q = pm4g.pm4g_filter_df_events(p, words, side, keep, out=pm4g.Prepared.empty(len(want), A, DEV))
                _same(_host(q), _expect(h, want))
                q = pm4g.pm4g_filter_df_events(p, words, side, keep, out=pm4g.Prepared.empty(len(want) - 1, A, DEV))
                assert int(q.status.item()) == pm4g.PM4G_E_CAPACITY and int(q.n_cases.item()) == 0


@pytest.mark.parametrize("n", [1, 64, 4097, 300_000])
def test_views_at_the_ends(n):
    A = 5
    log = _log(n, A, n + 7)
    h = oracle.prepare(*log, A)
    p = pm4g.pm4g_prepare(*cols(*log), A)
    mask = torch.full((1,), -1, dtype=torch.int64, device=DEV)
    codes = h["case_code"]
    for lo, hi in ((-2**31, 2**31 - 1), (int(codes[0]), int(codes[0]) + 1), (int(codes[-1]), int(codes[-1]) + 1),
                   (int(codes[-1]) + 1, 2**31 - 1), (-2**31, int(codes[0])), (int(codes[len(codes) // 2]), int(codes[-1])), (5, 5)):
        rec = np.zeros(1, dtype=np.dtype([("lo", "<i4"), ("hi", "<i4"), ("t_lo", "<i8"), ("t_hi", "<i8")]))
        rec["lo"], rec["hi"], rec["t_lo"], rec["t_hi"] = lo, hi, n, 8 * n
        v = torch.from_numpy(rec.view(np.uint8).copy()).to(DEV)
        keep = np.flatnonzero((h["case_s"] >= lo) & (h["case_s"] < hi) & (h["ts_s"] >= n) & (h["ts_s"] <= 8 * n))
        note(f"filter ranges view n={n} [{lo}, {hi}): {len(keep)} kept")
        _same(_host(pm4g.pm4g_filter_view(p, v, mask)), _expect(h, keep))


@pytest.mark.parametrize("cases", [1, 511, 512, 513, 5000, 600_000])
def test_case_filter_ranges(cases):
    rng = np.random.default_rng(cases)
    L = rng.integers(1, 6, cases)
    L[cases // 2] = 300                     # longer than a wave's trip
    case = np.repeat(np.arange(cases), L).astype(np.int32)
    n = len(case)
    act, ts = rng.integers(0, 4, n).astype(np.int32), np.arange(n, dtype=np.int64)
    h = dict(case_s=case, act_s=act, ts_s=ts)
    p = pm4g.pm4g_prepare(*cols(case, act, ts), 4, presorted=True)
    for lo, hi in ((3, 4), (1, 1000), (300, 300), (1001, 2000)):
        keep = np.flatnonzero(np.repeat((L >= lo) & (L <= hi), L))
        note(f"case filter ranges cases={cases} events {lo}..{hi}")
        _same(_host(pm4g.pm4g_filter_cases(p, min_events=lo, max_events=hi)), _expect(h, keep))
        if len(keep) > 1:
            q = pm4g.pm4g_filter_cases(p, min_events=lo, max_events=hi, out=pm4g.Prepared.empty(len(keep) - 1, 4, DEV))
            assert int(q.status.item()) == pm4g.PM4G_E_CAPACITY and int(q.n_cases.item()) == 0


def _unmix(key, seed):
    """The x whose SplitMix64 output from `seed` is key (the steps inverted)."""
    def unshift(z, s):
        x = z
        for _ in range(64 // s + 1):
            x = z ^ (x >> s)
        return x
    z = unshift(key, 31) * pow(0x94D049BB133111EB, -1, 2**64) & M64
    z = unshift(z, 27) * pow(0xBF58476D1CE4E5B9, -1, 2**64) & M64
    z = unshift(z, 30)
    return ((z - seed) * pow(0x9E3779B97F4A7C15, -1, 2**64) - 1) & M64


def test_sampling_keys_with_equal_leading_bits():
    """The cases with the smallest keys of 2^24 ids: their leading bytes are equal,
    so the digit passes narrow nothing down before the last, and the candidates
    listed decide; the key's steps are inverted on the host as a check."""
    seed, want = 12345, 0x0123456789ABCDEF
    x = _unmix(want, seed)
    z = (seed + (x + 1) * 0x9E3779B97F4A7C15) & M64
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & M64
    assert z ^ (z >> 31) == want
    ids = np.arange(2**24, dtype=np.uint64) * 251          # distinct 32-bit ids
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (ids + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
    order = np.argsort(z)
    case = ids[order[:20_000]].astype(np.uint32).view(np.int32)   # the smallest keys: leading bits nearly equal
    rng = np.random.default_rng(1)
    case = rng.permutation(np.repeat(case, 2))
    act, ts = np.zeros(len(case), np.int32), np.arange(len(case), dtype=np.int64)
    h = oracle.prepare(case, act, ts, 1)
    p = pm4g.pm4g_prepare(*cols(case, act, ts), 1)
    for k in (1, 7, 10_000, 19_999, 20_000):
        note(f"sampling with equal leading bits k={k}")
        kept = ids[order[:k]].astype(np.uint32).view(np.int32)
        _same(_host(pm4g.pm4g_sample(p, k, seed, False)), _expect(h, np.flatnonzero(np.isin(h["case_s"], kept))))


@pytest.mark.parametrize("n,k", [(1, 1), (5000, 1), (5000, 4999), (5000, 5000), (2_000_003, 200_000)])
def test_event_sampling(n, k):
    A = 3
    log = _log(n, A, n + k)
    h = oracle.prepare(*log, A)
    p = pm4g.pm4g_prepare(*cols(*log), A)
    seed = 99
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (np.arange(n, dtype=np.uint64) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
    note(f"event sampling n={n} k={k}")
    _same(_host(pm4g.pm4g_sample(p, k, seed, True)), _expect(h, np.sort(np.argsort(z)[:k])))
