"""Timed workloads of the library: what a program using it does, at the sizes it
does it.

Every log is drawn on the GPU from a seed with the laws of `synth.py` (case
lengths, Markov activities, exponential gaps, shuffled or ordered rows).  A
case names the call sequence (`kind`) and the log it runs on:

  dfg       raw columns -> DFG (pm4g_dfg)
  discover  raw columns -> prepared log -> DFG and trace variants
  views     many drill-down views of a resident log in one batched call
  serve     the serving executor on a small batch of mixed requests
  drill     one drill-down view materialised, then its variants
  explore   cases dataframe, then three filters or samples of a resident log
  efg       eventually-follows graph and temporal profile of a resident log
  csv       CSV text -> columns
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2204_04898_amd import pm4g, serve

DEV = "cuda:0"
YEAR_MS = 365 * 86_400_000


def listed():
    return [
        # the textbook call: the DFG of a small ordered log (10k cases, 16 activities)
        {"name": "dfg_100k_ordered", "kind": "dfg", "events": 100_000, "mean": 10.0, "law": "geom", "A": 16,
         "acts": "dirichlet", "unit": "ms", "ordered": True},
        # an interactive look at a filtered-down log: a few thousand events, short cases
        {"name": "discover_4k", "kind": "discover", "events": 4_111, "mean": 3.7, "law": "geom", "A": 11,
         "acts": "dirichlet", "unit": "ms", "ordered": False},
        # a department's log: hundreds of activities, long-tailed case lengths
        {"name": "discover_700k", "kind": "discover", "events": 700_003, "mean": 19.8, "law": "lognorm", "A": 300,
         "acts": "zipf", "unit": "ns", "ordered": False},
        # performance DFG of a 10M-event log in arrival order
        {"name": "dfg_10M", "kind": "dfg", "events": 10_000_000, "mean": 10.0, "law": "geom", "A": 64,
         "acts": "zipf", "unit": "ms", "ordered": False},
        # the headline workload: 5M cases, 99M events, 512 activities, everything discovered
        {"name": "discover_99M", "kind": "discover", "events": 99_000_000, "mean": 19.8, "law": "lognorm", "A": 512,
         "acts": "zipf", "unit": "ns", "ordered": False},
        # thousands of drill-down views of the headline log in one call
        {"name": "views_4096_99M", "kind": "views", "events": 99_000_000, "mean": 19.8, "law": "lognorm", "A": 512,
         "acts": "zipf", "unit": "ns", "views": 4096, "slice": 20_000_000},
        # a dashboard's views of a mid-size log
        {"name": "views_48_3M", "kind": "views", "events": 3_000_000, "mean": 10.0, "law": "geom", "A": 100,
         "acts": "zipf", "unit": "ms", "views": 48, "slice": 3_000_000},
        # a server's small mixed batch over a resident 10M-event log
        {"name": "serve_mixed_10M", "kind": "serve", "events": 10_000_000, "mean": 10.0, "law": "geom", "A": 64,
         "acts": "zipf", "unit": "ms", "slice": 300_000},
        # the variants of one drill-down view
        {"name": "drill_10M", "kind": "drill", "events": 10_000_000, "mean": 10.0, "law": "geom", "A": 64,
         "acts": "zipf", "unit": "ms", "slice": 4_000_000},
        # an analyst's filters, one after the other, on a resident log
        {"name": "explore_20M", "kind": "explore", "events": 20_000_000, "mean": 19.8, "law": "lognorm", "A": 512,
         "acts": "zipf", "unit": "ns", "steps": "cases,paths,df"},
        # the temporal profile of a log with many activities (several tables of cells)
        {"name": "efg_4M", "kind": "efg", "events": 4_000_000, "mean": 19.8, "law": "lognorm", "A": 512,
         "acts": "zipf", "unit": "ns"},
        # a CSV export read on the GPU
        {"name": "csv_2M", "kind": "csv", "events": 2_000_000, "mean": 10.0, "law": "geom", "A": 64, "acts": "zipf",
         "unit": "ms"},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above (sizes log-uniform, activity counts 3 to 600)."""
    kind = rng.choice(["dfg", "discover", "discover", "views", "serve", "drill", "explore", "efg", "csv"])
    law = rng.choice(["geom", "lognorm"])
    c = {"kind": kind, "law": law, "mean": 19.8 if law == "lognorm" else round(rng.uniform(3.0, 25.0), 2),
         "A": _log_uniform(rng, 3, 600), "acts": rng.choice(["zipf", "dirichlet"]), "unit": rng.choice(["ms", "ns"])}
    if kind in ("dfg", "discover"):
        c["events"] = _log_uniform(rng, 1_000, 20_000_000)
        c["ordered"] = rng.random() < 0.25
    elif kind == "views":
        c["events"] = _log_uniform(rng, 50_000, 10_000_000)
        c["views"] = _log_uniform(rng, 1, 512)
        c["slice"] = min(c["events"], _log_uniform(rng, 2_000, 2_000_000))
    elif kind in ("serve", "drill"):
        c["events"] = _log_uniform(rng, 50_000, 10_000_000)
        c["slice"] = min(c["events"], _log_uniform(rng, 2_000, 4_000_000))
    elif kind == "explore":
        c["events"] = _log_uniform(rng, 10_000, 20_000_000)
        c["steps"] = ",".join(rng.sample(["cases", "paths", "df", "window", "sample_cases", "sample_events"], 3))
    elif kind == "efg":
        c["events"] = _log_uniform(rng, 2_000, 3_000_000)
    else:
        c["events"] = _log_uniform(rng, 1_000, 2_000_000)
    return c


# ---- logs -------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _rand(n, g):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _chain(A, acts, g):
    """Initial and row-wise cumulative distributions of the activity chain."""
    e = -torch.log1p(-torch.rand(A + 1, A, generator=g, device=DEV, dtype=torch.float64))
    e = e / e.sum(1, keepdim=True)
    if acts == "zipf":
        w = torch.arange(1, A + 1, device=DEV, dtype=torch.float64) ** -1.1
        pi = (w / w.sum())[torch.randperm(A, generator=g, device=DEV)]
        p0, P = pi, 0.5 * pi[None, :] + 0.5 * e[:A]
    else:
        p0, P = e[A], e[:A]
    c0, cP = p0.cumsum(0), P.cumsum(1)
    c0[-1] = 1.0
    cP[:, -1] = 1.0
    return c0, (cP + torch.arange(A, device=DEV, dtype=torch.float64)[:, None]).reshape(-1)


def make_log(c, seed):
    """(case int32, act int32, ts int64) on the GPU and the number of cases."""
    g = _gen(seed)
    A = c["A"]
    C = max(1, int(round(c["events"] / c["mean"])))
    if c["law"] == "geom":
        L = torch.floor(torch.log1p(-_rand(C, g)) / math.log1p(-1.0 / c["mean"])).long() + 1
    else:
        z = torch.randn(C, generator=g, device=DEV, dtype=torch.float64)
        L = torch.round(torch.exp(math.log(12.0) + z)).long().clamp_(1, 2000)
    L.clamp_(max=2000)
    # the stated number of events exactly: spread what is missing, or over, one event a case
    N = max(C, int(c["events"]))
    while (over := int(L.sum()) - N) != 0:
        some = torch.randperm(C, generator=g, device=DEV)
        some = some[(L[some] > 1) if over > 0 else (L[some] < 2000)][:abs(over)]
        L[some] += -1 if over > 0 else 1
    # activities position by position over the cases still running, longest first
    order = torch.argsort(L, descending=True, stable=True)
    rank = torch.empty_like(order)
    rank[order] = torch.arange(C, device=DEV)
    hist = torch.bincount(L).cpu().numpy()
    running = (C - np.cumsum(hist))[:-1]          # cases longer than k, k = 0, 1, ...
    block = np.zeros(len(running) + 1, np.int64)
    np.cumsum(running, out=block[1:])
    c0, cP = _chain(A, c["acts"], g)
    pm = torch.empty(N, dtype=torch.int32, device=DEV)
    prev = None
    for k, n in enumerate(running.tolist()):
        u = _rand(n, g)
        if k == 0:
            cur = torch.searchsorted(c0, u, right=True).clamp_(max=A - 1)
        else:
            prev = prev[:n]
            cur = (torch.searchsorted(cP, prev + u, right=True) - prev * A).clamp_(0, A - 1)
        pm[int(block[k]):int(block[k]) + n] = cur.int()
        prev = cur
    off = torch.zeros(C + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(L, 0, out=off[1:])
    owner = torch.repeat_interleave(torch.arange(C, device=DEV), L)
    within = torch.arange(N, device=DEV) - off[owner]
    act = pm[torch.from_numpy(block).to(DEV)[within] + rank[owner]]
    del pm, within
    if c["kind"] == "csv":                         # every activity occurs: the dictionary's size is known
        k = min(A, N)
        act[torch.randperm(N, generator=g, device=DEV)[:k]] = torch.arange(k, dtype=torch.int32, device=DEV)
    unit = 1 if c["unit"] == "ms" else 1_000_000
    gap_mean = 3_600_000.0 if c["unit"] == "ms" else 1e10
    gaps = torch.floor(-torch.log1p(-_rand(N, g)) * gap_mean).long()
    gaps[_rand(N, g) < 0.05] = 0                   # equal timestamps inside a case: ties by row
    gaps[off[:-1]] = 0
    run = gaps.cumsum(0)
    start = 1_600_000_000_000 * unit + (_rand(C, g) * (YEAR_MS * unit)).long()
    ts = run + (start - run[off[:-1]])[owner]
    del gaps, run
    case = torch.randperm(C, generator=g, device=DEV)[owner].int()
    if c.get("ordered"):
        rows = torch.sort(case, stable=True).indices
    else:
        rows = torch.randperm(N, generator=g, device=DEV)
    return case[rows].contiguous(), act[rows].contiguous(), ts[rows].contiguous(), C


def _zeroed_prepared(n, A):
    """A prepared log to write into; what a call leaves unwritten stays zero."""
    p = pm4g.Prepared.empty(n, A, DEV)
    for t in (p.case_s, p.act_s, p.ts_s, p.case_off, p.case_code):
        t.zero_()
    return p


def _zeroed_variants(n):
    i64, i32 = dict(dtype=torch.int64, device=DEV), dict(dtype=torch.int32, device=DEV)
    return dict(n_variants=torch.zeros(1, **i64), var_count=torch.zeros(n, **i64), var_len=torch.zeros(n, **i32),
                var_rep=torch.zeros(n, **i32), var_off=torch.zeros(n + 1, **i64), var_acts=torch.zeros(n, **i32),
                case_variant=torch.zeros(n, **i32), status=torch.zeros(1, **i32))


def _fields(p):
    return dict(case_s=p.case_s, act_s=p.act_s, ts_s=p.ts_s, case_off=p.case_off, case_code=p.case_code,
                n_cases=p.n_cases, status=p.status)


def _resident(c, seed):
    """The log formatted once, as a program that keeps it does."""
    case, act, ts, C = make_log(c, seed)
    return pm4g.pm4g_prepare(case, act, ts, c["A"], out=_zeroed_prepared(case.numel(), c["A"])), C, ts


class _Views:
    pass


def _draw_views(c, C, t_lo, t_hi, n, seed):
    """Views as in synth.make_views: slice log-uniform from 1000 events to the
    case's bound, a time window of 5 to 100 % of the span, 8..A activities."""
    r = np.random.default_rng(seed)
    A, v = c["A"], _Views()
    top = max(1, min(C, int(c["slice"] / c["mean"])))
    low = max(1, min(top, int(1000 / c["mean"])))
    width = np.exp(r.uniform(math.log(low), math.log(top), n)).round().astype(np.int64).clip(1, C)
    lo = (r.random(n) * (C - width + 1)).astype(np.int64)
    v.case_lo, v.case_hi = lo.astype(np.int32), (lo + width).astype(np.int32)
    w = (r.uniform(0.05, 1.0, n) * (t_hi - t_lo)).astype(np.int64)
    v.t_lo = t_lo + (r.random(n) * (t_hi - t_lo - w + 1)).astype(np.int64)
    v.t_hi = v.t_lo + w
    keep = r.integers(min(8, A), A + 1, n)
    ranks = np.argsort(np.argsort(r.random((n, A)), axis=1), axis=1)
    bits = np.zeros((n, (A + 63) // 64 * 64), np.uint8)
    bits[:, :A] = ranks < keep[:, None]
    v.masks = np.packbits(bits, axis=1, bitorder="little").view(np.uint64)
    return v


# ---- state and pass -----------------------------------------------------------

def prepare(case, seed):
    c, k = case, case["kind"]
    if k == "dfg":
        cs, act, ts, _ = make_log(c, seed)
        return dict(c=c, log=(cs, act, ts))
    if k == "discover":
        cs, act, ts, _ = make_log(c, seed)
        return dict(c=c, log=(cs, act, ts), prep=_zeroed_prepared(cs.numel(), c["A"]), var=_zeroed_variants(cs.numel()))
    if k == "csv":
        return dict(c=c, text=_csv_text(c, seed))
    prep, C, ts = _resident(c, seed)
    t_lo, t_hi = int(ts.min()), int(ts.max())
    del ts
    s = dict(c=c, prep=prep)
    if k == "views":
        v = _draw_views(c, C, t_lo, t_hi, c["views"], seed)
        s["views"], s["masks"] = pm4g.views_to_device(v, DEV)
        # the capacities of this program's views, learnt from one call
        o = pm4g.pm4g_dfg_batched(prep, s["views"], s["masks"], c["views"], keep_workspace=False)
        need = [int(x) for x in o["required"].tolist()]
        s["tuning"] = pm4g.BatchedTuning(pair_capacity=need[3] * 11 // 10 + 1024, record_capacity=need[1] * 11 // 10 + 1024,
                                         cell_capacity=need[4] * 11 // 10 + 1024)
        E = min(c["views"] * min(c["A"] ** 2, c["slice"]), 3 << 26)
        s["out"] = dict(o, cap_edges=E, **{n: torch.zeros(E, dtype=o[n].dtype, device=DEV) for n in
                                           ("src", "dst", "count", "dt_sum", "dt_min", "dt_max", "dt_mean")})
    elif k == "serve":
        s["executor"] = serve.GpuExecutor({"log": prep}, device=DEV)
        v = _draw_views(c, C, t_lo, t_hi, 4, seed)
        s["requests"] = [serve.Request(rid=i, log="log", kind=("dfg", "filter", "dfg", "variants")[i],
                                       case_lo=int(v.case_lo[i]), case_hi=int(v.case_hi[i]), t_lo=int(v.t_lo[i]),
                                       t_hi=int(v.t_hi[i]), mask=v.masks[i], arrival=0.0) for i in range(4)]
        # where this program collects the answers
        A, n = c["A"], max(1000, c["slice"] * 3 // 2 + 4000)
        cells = dict(src=np.int32, dst=np.int32, count=np.int64, dt_sum=np.int64, dt_min=np.int64, dt_max=np.int64,
                     dt_mean=np.float64, start_count=np.int64, end_count=np.int64, act_count=np.int64)
        s["answers"] = [{k: np.zeros(A if k.endswith("_count") else A * A, t) for k, t in cells.items()}, {},
                        {k: np.zeros(A if k.endswith("_count") else A * A, t) for k, t in cells.items()},
                        dict(var_count=np.zeros(1000, np.int64), var_len=np.zeros(1000, np.int32),
                             var_rep=np.zeros(1000, np.int32), var_off=np.zeros(1001, np.int64),
                             var_acts=np.zeros(n, np.int32))]
    elif k == "drill":
        w = max(1, min(C, int(c["slice"] / c["mean"])))
        v = _draw_views(dict(c, slice=w * c["mean"]), C, t_lo, t_hi, 1, seed)
        v.case_lo[0] = np.random.default_rng(seed).integers(0, C - w + 1)
        v.case_hi[0] = v.case_lo[0] + w
        s["view"], s["mask"] = pm4g.views_to_device(v, DEV)
        n = min(prep.n_events, int(1.5 * w * c["mean"]) + 4000)   # room for the view's events
        s["sub"], s["var"] = _zeroed_prepared(n, c["A"]), _zeroed_variants(n)
    elif k == "explore":
        A = c["A"]
        g = np.random.default_rng(seed)
        bits = np.zeros((A * A + 63) // 64 * 64, np.uint8)
        bits[g.choice(A * A, size=min(A, A * A // 2), replace=False)] = 1
        s["pairs"] = torch.from_numpy(np.packbits(bits, bitorder="little").view(np.int64).copy()).to(DEV)
        s["window"] = (t_lo + (t_hi - t_lo) * 3 // 10, t_lo + (t_hi - t_lo) * 7 // 10)
        s["C"], s["seed"] = C, seed
        s["out"] = [_zeroed_prepared(prep.n_events, A) for _ in range(3)]
    return s


def run(s):
    c, k = s["c"], s["c"]["kind"]
    A = c["A"]
    if k == "dfg":
        return pm4g.pm4g_dfg(*s["log"], A, presorted=bool(c.get("ordered")))
    if k == "discover":
        p = pm4g.pm4g_prepare(*s["log"], A, presorted=bool(c.get("ordered")), out=s["prep"])
        d = pm4g.pm4g_dfg_prepared(p)
        v = pm4g.pm4g_variants_prepared(p, out=s["var"])
        return dict(log=_fields(p), dfg=d, variants=v)
    if k == "csv":
        return pm4g.pm4g_ingest_csv(s["text"], 0, 1, 2, ts_iso=True, ts_scale=3 if c["unit"] == "ms" else 9)
    p = s["prep"]
    if k == "views":
        o = pm4g.pm4g_dfg_batched(p, s["views"], s["masks"], c["views"], tuning=s["tuning"], out=s["out"])
        return {n: x for n, x in o.items() if n not in ("required", "cap_edges")}
    if k == "serve":
        ex, rs = s["executor"], s["requests"]
        ex.run(rs[:3])
        ex.run(rs[3:])
        for r, to in zip(rs, s["answers"]):
            for n, x in r.result.items():
                if isinstance(x, np.ndarray):
                    to[n][:x.size] = x
                else:
                    to[n] = x
        return s["answers"]
    if k == "drill":
        q = pm4g.pm4g_filter_view(p, s["view"], s["mask"], out=s["sub"])
        v = pm4g.pm4g_variants_prepared(q, out=s["var"])
        return dict(log=_fields(q), variants=v)
    if k == "efg":
        return pm4g.pm4g_efg(p)
    df = pm4g.pm4g_cases(p)
    got = [{n: x[:s["C"]] for n, x in df.items()}]
    for step, o in zip(c["steps"].split(","), s["out"]):
        if step == "cases":
            q = pm4g.pm4g_filter_cases(p, min_events=5, max_events=40, out=o)
        elif step == "paths":
            q = pm4g.pm4g_filter_cases(p, path_mask=s["pairs"], path_keep=False, out=o)
        elif step == "window":
            q = pm4g.pm4g_filter_cases(p, contain_lo=s["window"][0], contain_hi=s["window"][1], out=o)
        elif step == "df":
            q = pm4g.pm4g_filter_df_events(p, s["pairs"], 0, False, out=o)
        else:
            q = pm4g.pm4g_sample(p, (s["C"] if step == "sample_cases" else p.n_events) // 10, s["seed"],
                                 step == "sample_events", out=o)
        got.append(_fields(q))
    return got


def _events(c):
    return int(c["events"])


def work(case):
    """Each input column read once, each result written once."""
    c, k, N, A = case, case["kind"], _events(case), case["A"]
    C, cells = N / c["mean"], A * A
    if k == "dfg":
        b = 16 * N + 40 * cells
    elif k == "discover":
        # the formatted log and its case table, the DFG, the variants (about one per case)
        b = 32 * N + 12 * C + 40 * cells + 4 * C + 0.8 * (24 * C + 4 * N)
    elif k == "views":
        kept = min(N, c["views"] * 0.2 * c["slice"] / max(1.0, math.log(max(c["slice"], 1001) / 1000)))
        b = 16 * min(N, c["views"] * c["slice"]) + 48 * min(kept, c["views"] * min(cells, 2000)) + 24 * c["views"] * A
    elif k == "serve":
        b = 4 * 16 * c["slice"] / max(1.0, math.log(max(c["slice"], 1001) / 1000))
    elif k == "drill":
        b = 16 * c["slice"] + 0.3 * c["slice"] * (16 + 4 + 3)
    elif k == "explore":
        b = 28 * C + sum({"cases": 0.6, "paths": 0.8, "df": 1.0, "window": 0.4}.get(x, 0.1) * 32 * N + 12 * C
                         for x in c["steps"].split(","))
    elif k == "efg":
        b = 16 * N + 56 * cells
    else:
        b = N * (52 if c["unit"] == "ms" else 58) + 16 * N
    return {"bytes": float(b), "flops": 0.0}


# ---- CSV text -----------------------------------------------------------------

def _digits(x, width):
    p = 10 ** torch.arange(width - 1, -1, -1, device=DEV, dtype=torch.int64)
    return ((x[:, None] // p) % 10 + 48).to(torch.uint8)


def _csv_text(c, seed):
    """Header and rows "c0000000017,Activity 0003,2021-02-03T04:05:06.789Z"
    (9 fraction digits for ns) as device bytes."""
    case, act, ts, _ = make_log(c, seed)
    n = case.numel()
    per = 1000 if c["unit"] == "ms" else 1_000_000_000
    sec, frac = ts // per, ts % per
    day, tod = sec // 86_400, sec % 86_400
    dates = np.arange("1970-01-01", "2100-01-01", dtype="datetime64[D]").astype("S10")
    dates = torch.from_numpy(dates.view(np.uint8).reshape(-1, 10).copy()).to(DEV)

    def lit(b):
        return torch.frombuffer(bytearray(b), dtype=torch.uint8).to(DEV)[None, :].expand(n, len(b))

    row = torch.cat([lit(b"c"), _digits(case.long() + 2**31, 10), lit(b",Activity "), _digits(act.long(), 4), lit(b","),
                     dates[day], lit(b"T"), _digits(tod // 3600, 2), lit(b":"), _digits(tod // 60 % 60, 2), lit(b":"),
                     _digits(tod % 60, 2), lit(b"."), _digits(frac, 3 if per == 1000 else 9), lit(b"Z\n")], 1)
    head = torch.frombuffer(bytearray(b"case,activity,timestamp\n"), dtype=torch.uint8).to(DEV)
    return torch.cat([head, row.reshape(-1)])


# ---- values in 64 bits, from plain torch ---------------------------------------

def _ordered(case, act, ts):
    i = torch.sort(ts, stable=True).indices
    i = i[torch.sort(case[i], stable=True).indices]
    return case[i], act[i].long(), ts[i]


def _mean_of(case, act, ts, A):
    """Count and mean gap per cell of the pairs of an ordered log."""
    same = case[1:] == case[:-1]
    cell = (act[:-1] * A + act[1:])[same]
    gap = (ts[1:] - ts[:-1])[same]
    n = torch.bincount(cell, minlength=A * A)
    s = torch.zeros(A * A, dtype=torch.int64, device=DEV).index_add_(0, cell, gap)
    return n, s.double() / n.double()              # 0 / 0: not a number, as for an empty cell


def _kept(v, i, case, act, ts):
    bits = torch.from_numpy(np.unpackbits(v.masks[i].view(np.uint8), bitorder="little")).to(DEV).bool()
    m = (case >= int(v.case_lo[i])) & (case < int(v.case_hi[i])) & (ts >= int(v.t_lo[i])) & (ts <= int(v.t_hi[i]))
    m &= bits[act]
    return case[m], act[m], ts[m]


def exact(case, seed):
    """The floating-point outputs (mean gaps, temporal profile); every other
    output is a whole number."""
    c, k, A = case, case["kind"], case["A"]
    if k in ("csv", "drill", "explore") or (k == "views" and c["views"] > 64):
        return None
    case_, act, ts, C = make_log(c, seed)
    t_lo, t_hi = int(ts.min()), int(ts.max())
    case_, act, ts = _ordered(case_, act, ts)
    if k in ("dfg", "discover"):
        mean = _mean_of(case_, act, ts, A)[1]
        return dict(dt_mean=mean) if k == "dfg" else dict(dfg=dict(dt_mean=mean))
    if k in ("views", "serve"):
        v = _draw_views(c, C, t_lo, t_hi, c["views"] if k == "views" else 4, seed)
        got = []
        for i in range(len(v.case_lo)):
            n, mean = _mean_of(*_kept(v, i, case_, act, ts), A)
            got.append(mean[n > 0])
        if k == "views":
            full = torch.zeros(min(c["views"] * min(A * A, c["slice"]), 3 << 26), dtype=torch.float64, device=DEV)
            flat = torch.cat(got)
            full[:flat.numel()] = flat
            return dict(dt_mean=full)
        full = [np.zeros(A * A) for _ in got]
        for f, x in zip(full, got):
            f[:x.numel()] = x.cpu().numpy()
        return [dict(dt_mean=full[0]), None, dict(dt_mean=full[2]), None]
    # temporal profile: two passes over the pairs, one distance in the case at a time
    n = torch.zeros(A * A, dtype=torch.int64, device=DEV)
    s, q = (torch.zeros(A * A, dtype=torch.float64, device=DEV) for _ in range(2))

    def pairs():
        at = torch.arange(case_.numel(), device=DEV)
        d = 1
        while at.numel():
            at = at[at + d < case_.numel()]
            at = at[case_[at] == case_[at + d]]    # a case with no pair at this distance has none further
            if at.numel():
                yield act[at] * A + act[at + d], (ts[at + d] - ts[at]).double()
            d += 1

    for cell, gap in pairs():
        n += torch.bincount(cell, minlength=A * A)
        s.index_add_(0, cell, gap)
    mean = s / n.double()
    for cell, gap in pairs():
        q.index_add_(0, cell, (gap - mean[cell]) ** 2)
    std = torch.sqrt(q / (n - 1).double())
    std = torch.where(n == 1, torch.zeros_like(std), torch.where(n == 0, torch.full_like(std, math.nan), std))
    return dict(mean=mean, std=std)
