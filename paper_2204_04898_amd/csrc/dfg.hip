// Directly-follows graph aggregation over a prepared log (Sec. 3, the
// aggregations over consecutive event pairs: frequency and performance DFG;
// start and end activities; how often each activity occurs).  For position i
// of the ordered log, the event
// directly follows i-1 iff both have the same case; the pair contributes to
// cell act_s[i-1]*A + act_s[i] with gap ts_s[i] - ts_s[i-1] (mod 2^64).
//
// Three aggregation paths:
//   A*A <= 4096  k_dfg_lds: up to 256 blocks, one privatised LDS table each
//                (count u32, sum u64, min, max: 112 KB), partial tables
//                written out and reduced per cell; a log of at most two tiles
//                is one block, which writes the outputs itself.
//   A*A >  4096, few events: k_dfg_direct: the pairs straight into the dense
//                outputs with global atomics.
//   A*A >  4096  cells are cut into buckets of 4096 (cell >> 12) and the
//                edges are partitioned bucket-major, so that each bucket's
//                edges are one contiguous stream:
//                k_dfg_count    per (bucket, chunk of the log) edge counts,
//                               and the start counts;
//                scan           first edge index of every (bucket, chunk);
//                k_dfg_scatter  edges (u16 cell within the bucket, u64 gap)
//                               written to their place via LDS cursors;
//                k_dfg_plan     buckets cut into slots of about E/512 edges
//                               (Zipf-heavy buckets get more slots);
//                k_dfg_agg      one block per slot streams its edges into a
//                               4096-cell LDS table, writes a partial table.
// k_dfg_reduce folds the partial tables, writes the dense outputs and the
// FP64 mean.  Activity and end counts are not counted per event: every event
// starts its case or is the target of one pair, so act(y) = start(y) + the
// column sum of count, and every event ends its case or is the source of one
// pair, so end(x) = act(x) - the row sum of count.
// Per-event global atomics run at ~25 G/s on MI355X, LDS atomics at ~700 G/s,
// so only the few-event path uses the former.
// Bytes per event: 16 read (+ 8 read, 10 write and 10 read per edge on the
// bucketed path).
#include <math.h>

#include "common.hpp"
#include "devsort.hpp"
#include "internal.hpp"
#include "prof.hpp"
#include "../../include/pm4g.h"

namespace pm4g {

constexpr int kLB = 1024;   // threads of k_dfg_lds
constexpr int kAB = 1024;   // threads of k_dfg_agg
constexpr int64_t kDfgSlotMin = 8192;     // edges of a full aggregation slot, at least
constexpr int64_t kDfgDirectMax = 16384;  // events of the few-event path, at most

static int64_t n_buckets(int32_t A) {
    return ((int64_t)A * A + kCellsPerTable - 1) / kCellsPerTable;
}
// chunk of the log per (bucket, chunk) counter: about 64 buckets per 4096 events
static int64_t dfg_chunk(int64_t nbk) { return (int64_t)kDfgTile * (nbk <= 64 ? 1 : (nbk + 63) / 64); }
static int64_t dfg_chunks(int64_t n, int64_t nbk) {
    const int64_t c = dfg_chunk(nbk);
    return (n + c - 1) / c;
}

DfgWs dfg_ws_layout(Bump& b, int64_t n, int32_t A) {
    DfgWs w{};
    if (A <= kDfgLdsMaxA) {
        const int64_t slots = kDfgLdsBlocks;
        w.n_slots_max = (int32_t)slots;
        w.n_act_blocks = kDfgLdsBlocks;
        w.pcount = b.take<uint32_t>(slots * kCellsPerTable);
        w.psum = b.take<uint64_t>(slots * kCellsPerTable);
        w.pmin = b.take<int64_t>(slots * kCellsPerTable);
        w.pmax = b.take<int64_t>(slots * kCellsPerTable);
    } else {
        const int64_t nbk = n_buckets(A);
        const int64_t nch = dfg_chunks(n, nbk);
        const int64_t slots = nbk + kDfgAggTarget;
        w.n_slots_max = (int32_t)slots;
        const int64_t g = nch < kDfgPartBlocks ? (nch < 1 ? 1 : nch) : kDfgPartBlocks;
        w.n_act_blocks = (int32_t)g;
        const size_t m = (size_t)(n > 0 ? n : 1);
        w.pcount = b.take<uint32_t>(slots * kCellsPerTable);
        w.psum = b.take<uint64_t>(slots * kCellsPerTable);
        w.pmin = b.take<int64_t>(slots * kCellsPerTable);
        w.pmax = b.take<int64_t>(slots * kCellsPerTable);
        w.ecell = b.take<uint16_t>(m);
        w.egap = b.take<uint64_t>(m);
        w.ecnt = b.take<uint32_t>((size_t)(nbk * nch) + 1);
        w.escan = b.take<uint32_t>((size_t)(nbk * nch) + 1);
        w.bbase = b.take<uint32_t>(nbk);
        w.btotal = b.take<uint32_t>(nbk);
        w.bfirst = b.take<uint32_t>(nbk);
        w.bslots = b.take<uint32_t>(nbk);
        w.plan = b.take<int4>(slots);
        w.nplan = b.take<uint32_t>(1);
        w.part32 = b.take<uint32_t>(dev::kScanGrid);
        w.scal = b.take<int64_t>(2);
        w.utotal = b.take<uint32_t>(1);
    }
    w.pfreq = b.take<uint32_t>((size_t)w.n_act_blocks * A);
    w.pstart = b.take<uint32_t>((size_t)w.n_act_blocks * A);
    w.pend = b.take<uint32_t>((size_t)w.n_act_blocks * A);
    w.pspan = b.take<uint64_t>(w.n_act_blocks);
    return w;
}

// Four consecutive events [e0, e0 + 4) of the prepared log in registers,
// with the event before e0: 16-byte loads when the quad lies inside [.., lim)
// and the columns are 16-byte aligned, element loads otherwise; the event
// before comes from the adjacent lane (the lanes hold consecutive quads), the
// wave's first lane loads it.  Lanes past `lim` get case ~prev so nothing
// pairs.  fetch_quad only issues loads (so a caller can have the next quad in
// flight while it works on one), join_quad does the lane exchange; every lane
// of the wave must execute both.
struct Quad {
    int32_t c[4], a[4];
    int64_t t[4];
    int32_t cp, ap;   // event e0 - 1 (cp = ~c[0] when there is none)
    int64_t tp;
};

template <bool WANT_TS>
__device__ __forceinline__ Quad fetch_quad(const int32_t* __restrict__ case_s, const int32_t* __restrict__ act_s,
                                           const int64_t* __restrict__ ts_s, int64_t e0, int64_t lim, int64_t n,
                                           bool aligned) {
    Quad q;
    if (aligned && e0 + 3 < lim) {
        const int4 c4 = *reinterpret_cast<const int4*>(case_s + e0);
        const int4 a4 = *reinterpret_cast<const int4*>(act_s + e0);
        q.c[0] = c4.x; q.c[1] = c4.y; q.c[2] = c4.z; q.c[3] = c4.w;
        q.a[0] = a4.x; q.a[1] = a4.y; q.a[2] = a4.z; q.a[3] = a4.w;
        if (WANT_TS) {
            const longlong2 t01 = *reinterpret_cast<const longlong2*>(ts_s + e0);
            const longlong2 t23 = *reinterpret_cast<const longlong2*>(ts_s + e0 + 2);
            q.t[0] = t01.x; q.t[1] = t01.y; q.t[2] = t23.x; q.t[3] = t23.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t i = e0 + j;
            const bool in = i < lim;
            q.c[j] = in ? case_s[i] : (j ? ~q.c[j - 1] : 0);
            q.a[j] = in ? act_s[i] : 0;
            if (WANT_TS) q.t[j] = in ? ts_s[i] : 0;
        }
    }
    q.cp = q.ap = 0;
    q.tp = 0;
    if (lane() == 0 && e0 > 0 && e0 - 1 < n) {
        q.cp = case_s[e0 - 1];
        q.ap = act_s[e0 - 1];
        if (WANT_TS) q.tp = ts_s[e0 - 1];
    }
    return q;
}

template <bool WANT_TS>
__device__ __forceinline__ void join_quad(Quad& q, int64_t e0, int64_t n) {
    const int32_t cp = __shfl_up(q.c[3], 1);
    const int32_t ap = __shfl_up(q.a[3], 1);
    int64_t tp = 0;
    if (WANT_TS) tp = __shfl_up(q.t[3], 1);
    if (lane() != 0) {
        q.cp = cp;
        q.ap = ap;
        q.tp = tp;
    } else if (!(e0 > 0 && e0 - 1 < n)) {
        q.cp = ~q.c[0];
    }
}

template <bool WANT_TS>
__device__ __forceinline__ Quad load_quad(const int32_t* __restrict__ case_s, const int32_t* __restrict__ act_s,
                                          const int64_t* __restrict__ ts_s, int64_t e0, int64_t lim, int64_t n,
                                          bool aligned) {
    Quad q = fetch_quad<WANT_TS>(case_s, act_s, ts_s, e0, lim, n, aligned);
    join_quad<WANT_TS>(q, e0, n);
    return q;
}

// ---------------------------------------------------------------------------
// LDS table of cells: count, gap sum, and min and max side by side (read with
// one 16-byte load before the conditional atomics)

__device__ __forceinline__ void agg_edge(uint32_t* scount, uint64_t* ssum, int64_t* smm, uint32_t cell,
                                         uint64_t gap) {
    const int64_t gg = (int64_t)gap;
    atomicAdd(&scount[cell], 1u);
    atomicAdd(reinterpret_cast<unsigned long long*>(&ssum[cell]), (unsigned long long)gap);
    const longlong2 mm = *reinterpret_cast<const longlong2*>(&smm[2 * cell]);
    if (gg < mm.x) __hip_atomic_fetch_min(&smm[2 * cell], gg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (gg > mm.y) __hip_atomic_fetch_max(&smm[2 * cell + 1], gg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void store_cell(const DfgOutDev& out, int64_t e, uint64_t cnt, uint64_t sum, int64_t mn,
                                           int64_t mx) {
    out.count[e] = (int64_t)cnt;
    out.dt_sum[e] = (int64_t)sum;
    out.dt_min[e] = mn;
    out.dt_max[e] = mx;
    if (out.dt_mean) out.dt_mean[e] = cnt ? (double)(int64_t)sum / (double)(int64_t)cnt : (double)NAN;
}

// The call's scalars.  bad: an activity outside [0, A) was seen; status_in (may
// be NULL): the producing prepare's status.
__device__ __forceinline__ void store_scalars(const DfgOutDev& out, uint64_t span, int64_t n_cases, bool bad,
                                              const int32_t* status_in) {
    *out.overflow = span > (uint64_t)INT64_MAX ? 1 : 0;
    *out.n_cases = n_cases;
    *out.status = bad ? PM4G_E_RANGE : (status_in ? *status_in : 0);
}

__device__ __forceinline__ uint64_t wave_sat_sum(uint64_t v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = sat_add63(v, __shfl_xor(v, o));
    return v;
}

// ---------------------------------------------------------------------------
// A*A <= 4096: privatised LDS tables

// Span partial of a block that saw an invalid activity (a saturated span is
// 2^63 at most).
constexpr uint64_t kBadSpan = ~0ull;

// Tile of kDfgTile events per block and step, one quad per thread, the next
// tile's loads in flight while one is aggregated.  Bound by LDS atomics (two
// per pair, one per case, and the rare min/max): no counter per event for the
// activities and case ends, which follow from the table (header).  With fewer
// than 64 activities each cell is kept `1 << clog` times side by side, lane l
// adding to copy l mod copies, so that a wave's adds to a frequent cell do not
// queue on one address (16 activities: 256 cells, 16 copies).
// Measured on 10M events of 64 activities: 37 us, 4.3 TB/s (84 us with element
// loads and 7 atomics per event), and the fold of its 256 tables 15 us (84).
__global__ __launch_bounds__(kLB) void k_dfg_lds(const int32_t* __restrict__ case_s,
                                                 const int32_t* __restrict__ act_s,
                                                 const int64_t* __restrict__ ts_s, int64_t n, int32_t A, int clog,
                                                 DfgWs ws, const int32_t* status_in, DfgOutDev out,
                                                 const int64_t* skip) {
    if (skip && *skip) n = 0;
    __shared__ uint32_t scount[kCellsPerTable];
    __shared__ uint64_t ssum[kCellsPerTable];
    __shared__ alignas(16) int64_t smm[2 * kCellsPerTable];
    __shared__ uint32_t sstart[kDfgLdsMaxA], sfreq[kDfgLdsMaxA], srow[kDfgLdsMaxA];
    __shared__ uint64_t sspan[kLB / kWave];

    const int cells = A * A, copies = 1 << clog;
    for (int c = threadIdx.x; c < cells << clog; c += kLB) {
        scount[c] = 0;
        ssum[c] = 0;
        smm[2 * c] = INT64_MAX;
        smm[2 * c + 1] = INT64_MIN;
    }
    if (threadIdx.x < A) sstart[threadIdx.x] = sfreq[threadIdx.x] = srow[threadIdx.x] = 0;
    const bool aligned = ((reinterpret_cast<uintptr_t>(case_s) | reinterpret_cast<uintptr_t>(act_s) |
                           reinterpret_cast<uintptr_t>(ts_s)) & 15) == 0;
    static_assert(kDfgTile == 4 * kLB, "one quad per thread and tile");
    const int64_t tiles = (n + kDfgTile - 1) / kDfgTile;
    int64_t tile = blockIdx.x;
    Quad nx{};
    if (tile < tiles)
        nx = fetch_quad<true>(case_s, act_s, ts_s, tile * kDfgTile + 4 * (int64_t)threadIdx.x, n, n, aligned);
    __syncthreads();

    uint64_t span = 0;
    bool bad = false;
    const uint32_t copy = (uint32_t)lane() & (uint32_t)(copies - 1);
    for (; tile < tiles; tile += gridDim.x) {
        const int64_t e0 = tile * kDfgTile + 4 * (int64_t)threadIdx.x;
        Quad qd = nx;
        if (tile + gridDim.x < tiles)
            nx = fetch_quad<true>(case_s, act_s, ts_s, e0 + (int64_t)gridDim.x * kDfgTile, n, n, aligned);
        join_quad<true>(qd, e0, n);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (e0 + j >= n) break;
            const int32_t a = qd.a[j];
            if ((uint32_t)a >= (uint32_t)A) {
                bad = true;
                continue;
            }
            const int32_t p = j ? qd.a[j - 1] : qd.ap;
            if ((j ? qd.c[j - 1] : qd.cp) != qd.c[j]) {
                atomicAdd(&sstart[a], 1u);
            } else if ((uint32_t)p < (uint32_t)A) {
                const uint64_t gap = (uint64_t)qd.t[j] - (uint64_t)(j ? qd.t[j - 1] : qd.tp);
                agg_edge(scount, ssum, smm, ((uint32_t)(p * A + a) << clog) | copy, gap);
                span = sat_add63(span, cap63(gap));
            }
        }
    }
    span = wave_sat_sum(span);
    if (__ballot(bad) != 0) span = kBadSpan;
    if (lane() == 0) sspan[threadIdx.x / kWave] = span;
    __syncthreads();

    // the copies of each cell folded; the table's outputs (one block) or its partial
    const bool direct = gridDim.x == 1;
    const size_t slot = (size_t)blockIdx.x * kCellsPerTable;
    for (int c = threadIdx.x; c < cells; c += kLB) {
        uint32_t cnt = 0;
        uint64_t sum = 0;
        int64_t mn = INT64_MAX, mx = INT64_MIN;
        for (int k = 0; k < copies; ++k) {
            const int at = (c << clog) + k;
            cnt += scount[at];
            sum += ssum[at];
            mn = smm[2 * at] < mn ? smm[2 * at] : mn;
            mx = smm[2 * at + 1] > mx ? smm[2 * at + 1] : mx;
        }
        scount[c << clog] = cnt;   // only this thread reads the cell's copies
        if (direct) {
            store_cell(out, c, cnt, sum, mn, mx);
        } else {
            ws.pcount[slot + c] = cnt;
            ws.psum[slot + c] = sum;
            ws.pmin[slot + c] = mn;
            ws.pmax[slot + c] = mx;
        }
    }
    __syncthreads();
    // column and row sums of the counts: thread (a, g) takes every 16th entry of
    // column a and of row a (the row from entry a on: the lanes' banks differ)
    {
        const int a = threadIdx.x & (kDfgLdsMaxA - 1);
        if (a < A) {
            uint32_t col = 0, row = 0;
            for (int x = threadIdx.x / kDfgLdsMaxA; x < A; x += kLB / kDfgLdsMaxA) {
                const int y = x + a < A ? x + a : x + a - A;
                col += scount[(x * A + a) << clog];
                row += scount[(a * A + y) << clog];
            }
            atomicAdd(&sfreq[a], col);
            atomicAdd(&srow[a], row);
        }
    }
    __syncthreads();
    if (threadIdx.x < kWave) {   // kDfgLdsMaxA activities: one wave
        const int a = threadIdx.x;
        const uint32_t st = a < A ? sstart[a] : 0u;
        const uint32_t fr = a < A ? st + sfreq[a] : 0u;
        const int64_t en = a < A ? (int64_t)fr - (int64_t)srow[a] : 0;   // of a part of the log: may be negative
        uint64_t sp = 0;
        bool any_bad = false;
        for (int k = 0; k < kLB / kWave; ++k) {
            any_bad |= sspan[k] == kBadSpan;
            sp = sat_add63(sp, cap63(sspan[k]));
        }
        if (direct) {
            if (a < A) {
                out.act_count[a] = fr;
                out.start_count[a] = st;
                out.end_count[a] = en;
            }
            const uint32_t nc = wave_sum(st);
            if (a == 0) store_scalars(out, sp, nc, any_bad, status_in);
        } else {
            if (a < A) {
                const size_t ab = (size_t)blockIdx.x * A + a;
                ws.pfreq[ab] = fr;
                ws.pstart[ab] = st;
                ws.pend[ab] = (uint32_t)(int32_t)en;
            }
            if (a == 0) ws.pspan[blockIdx.x] = any_bad ? kBadSpan : sp;
        }
    }
}

// ---------------------------------------------------------------------------
// A*A > 4096: bucket-major edges

constexpr int kCB = 512;                  // threads of k_dfg_count / k_dfg_scatter


// Per chunk: edge counts per bucket; per block: start counts, its cases (in
// pend[block]) and whether it saw an invalid activity (pend[blocks + block]).
// Dynamic LDS: (A + nbk) u32.
__global__ __launch_bounds__(kCB) void k_dfg_count(const int32_t* __restrict__ case_s,
                                                   const int32_t* __restrict__ act_s, int64_t n,
                                                   int32_t A, int64_t nbk, int64_t nch, int64_t chunk,
                                                   DfgWs ws, const int64_t* skip) {
    if (skip && *skip) n = 0;
    extern __shared__ uint32_t dsm[];
    uint32_t* sstart = dsm;
    uint32_t* bcnt = dsm + A;
    __shared__ uint32_t scase[kCB / kWave];
    for (int a = threadIdx.x; a < A; a += kCB) sstart[a] = 0;
    const bool aligned = ((reinterpret_cast<uintptr_t>(case_s) | reinterpret_cast<uintptr_t>(act_s)) & 15) == 0;
    bool bad = false;
    uint32_t cases = 0;
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
        for (int64_t k = threadIdx.x; k < nbk; k += kCB) bcnt[k] = 0;
        __syncthreads();
        const int64_t i1 = (ch + 1) * chunk < n ? (ch + 1) * chunk : n;
        for (int64_t t0 = ch * chunk; t0 < i1; t0 += kDfgTile) {
#pragma unroll
            for (int h = 0; h < kDfgTile / (4 * kCB); ++h) {
                const int64_t e0 = t0 + 4 * (h * kCB + (int64_t)threadIdx.x);
                if (t0 + 4 * h * kCB >= i1) break;   // block-uniform
                const Quad qd = load_quad<false>(case_s, act_s, nullptr, e0, i1, n, aligned);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (e0 + j >= i1) break;
                    const int32_t c = qd.c[j], a = qd.a[j];
                    if ((uint32_t)a >= (uint32_t)A) {
                        bad = true;
                        continue;
                    }
                    const int32_t cp = j ? qd.c[j - 1] : qd.cp;
                    const int32_t ap = j ? qd.a[j - 1] : qd.ap;
                    if (cp != c) {
                        atomicAdd(&sstart[a], 1u);
                        ++cases;
                    } else if ((uint32_t)ap < (uint32_t)A)
                        atomicAdd(&bcnt[((uint32_t)ap * (uint32_t)A + (uint32_t)a) >> 12], 1u);
                }
            }
        }
        __syncthreads();
        for (int64_t k = threadIdx.x; k < nbk; k += kCB) ws.ecnt[k * nch + ch] = bcnt[k];
        __syncthreads();
    }
    cases = wave_sum(cases);
    if (lane() == 0) scase[threadIdx.x / kWave] = cases;
    const int any_bad = __syncthreads_or(bad);   // (a block without chunks: also the zeroing above)
    const size_t ab = (size_t)blockIdx.x * A;
    for (int a = threadIdx.x; a < A; a += kCB) ws.pstart[ab + a] = sstart[a];
    if (threadIdx.x == 0) {
        uint32_t c = 0;
        for (int k = 0; k < kCB / kWave; ++k) c += scase[k];
        ws.pend[blockIdx.x] = c;
        ws.pend[gridDim.x + blockIdx.x] = any_bad ? 1u : 0u;
        if (blockIdx.x == 0) ws.scal[0] = nbk * nch;
    }
}

// Per chunk: every edge goes to its bucket's run (cursor seeded from the scan).
// Per 4096-event tile the edges are first grouped by bucket in LDS, then
// written out in bucket order, so each bucket's piece is one coalesced run.
// Span partial per block.  Dynamic LDS: 3 * nbk u32.
__global__ __launch_bounds__(kCB) void k_dfg_scatter(const int32_t* __restrict__ case_s,
                                                     const int32_t* __restrict__ act_s,
                                                     const int64_t* __restrict__ ts_s, int64_t n, int32_t A,
                                                     int64_t nbk, int64_t nch, int64_t chunk, DfgWs ws,
                                                     const int64_t* skip) {
    if (skip && *skip) n = 0;
    extern __shared__ uint32_t dsm[];
    uint32_t* cur = dsm;              // global cursor of each bucket
    uint32_t* lcnt = dsm + nbk;       // edges per bucket in this tile
    uint32_t* lstart = dsm + 2 * nbk; // their start in the staged tile
    __shared__ uint16_t s_cell[kDfgTile];
    __shared__ uint64_t s_gap[kDfgTile];
    __shared__ uint16_t s_bk[kDfgTile];
    __shared__ uint32_t tmp[kCB / kWave + 1];
    __shared__ uint64_t sspan[kCB / kWave];
    constexpr int kQ = kDfgTile / (4 * kCB);   // quads per thread per tile (2)
    const bool aligned = ((reinterpret_cast<uintptr_t>(case_s) | reinterpret_cast<uintptr_t>(act_s) |
                           reinterpret_cast<uintptr_t>(ts_s)) & 15) == 0;
    uint64_t span = 0;
    // chunks XCD-contiguous: a bucket's runs from neighbouring chunks are
    // neighbours in the output and meet in the same L2
    const XcdSplit xs = xcd_split(nch);
    for (int64_t ch = xs.first; ch < xs.end; ch += xs.stride) {
        for (int64_t k = threadIdx.x; k < nbk; k += kCB) cur[k] = ws.escan[k * nch + ch];
        const int64_t i1 = (ch + 1) * chunk < n ? (ch + 1) * chunk : n;
        for (int64_t t0 = ch * chunk; t0 < i1; t0 += kDfgTile) {
            for (int64_t k = threadIdx.x; k < nbk; k += kCB) lcnt[k] = 0;
            __syncthreads();
            // 1. edges of this thread's quads: bucket, slot in the bucket, cell, gap
            uint32_t eb[4 * kQ], ec[4 * kQ];
            uint64_t eg[4 * kQ];
#pragma unroll
            for (int h = 0; h < kQ; ++h) {
                const int64_t e0 = t0 + 4 * (h * kCB + (int64_t)threadIdx.x);
                Quad qd{};
                if (t0 + 4 * h * kCB < i1)   // block-uniform
                    qd = load_quad<true>(case_s, act_s, ts_s, e0, i1, n, aligned);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int u = 4 * h + j;
                    eb[u] = 0xFFFFFFFFu;
                    if (t0 + 4 * h * kCB >= i1) continue;
                    const int32_t cp = j ? qd.c[j - 1] : qd.cp;
                    const int32_t ap = j ? qd.a[j - 1] : qd.ap;
                    const int64_t tp = j ? qd.t[j - 1] : qd.tp;
                    if (e0 + j >= i1 || qd.c[j] != cp || (uint32_t)qd.a[j] >= (uint32_t)A ||
                        (uint32_t)ap >= (uint32_t)A)
                        continue;
                    const uint32_t cell = (uint32_t)ap * (uint32_t)A + (uint32_t)qd.a[j];
                    const uint64_t gap = (uint64_t)qd.t[j] - (uint64_t)tp;
                    span = sat_add63(span, cap63(gap));
                    const uint32_t b = cell >> 12;
                    const uint32_t slot = atomicAdd(&lcnt[b], 1u);
                    eb[u] = b | (slot << 16);   // nbk <= 4096, slot < 4096
                    ec[u] = cell & (kCellsPerTable - 1);
                    eg[u] = gap;
                }
            }
            __syncthreads();
            // 2. bucket starts inside the staged tile
            uint32_t E = 0;
            for (int64_t k0 = 0; k0 < nbk; k0 += kCB) {
                const int64_t k = k0 + threadIdx.x;
                const uint32_t v = k < nbk ? lcnt[k] : 0u;
                uint32_t total;
                const uint32_t ex = block_excl_sum<kCB>(v, tmp, &total);
                if (k < nbk) lstart[k] = E + ex;
                E += total;
            }
            __syncthreads();
            // 3. stage in bucket order
#pragma unroll
            for (int u = 0; u < 4 * kQ; ++u) {
                if (eb[u] == 0xFFFFFFFFu) continue;
                const uint32_t b = eb[u] & 0xFFFFu;
                const uint32_t at = lstart[b] + (eb[u] >> 16);
                s_cell[at] = (uint16_t)ec[u];
                s_gap[at] = eg[u];
                s_bk[at] = (uint16_t)b;
            }
            __syncthreads();
            // 4. coalesced runs out
            for (uint32_t i = threadIdx.x; i < E; i += kCB) {
                const uint32_t b = s_bk[i];
                const uint32_t g = cur[b] + (i - lstart[b]);
                ws.ecell[g] = s_cell[i];
                ws.egap[g] = s_gap[i];
            }
            __syncthreads();
            for (int64_t k = threadIdx.x; k < nbk; k += kCB) cur[k] += lcnt[k];
        }
        __syncthreads();
    }
    span = wave_sat_sum(span);
    if (lane() == 0) sspan[threadIdx.x / kWave] = span;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s = 0;
        for (int k = 0; k < kCB / kWave; ++k) s = sat_add63(s, sspan[k]);
        ws.pspan[blockIdx.x] = s;
    }
}

// Bucket bases and totals from the scan; every bucket cut into slots of about
// E/kDfgAggTarget edges, at least kDfgSlotMin: a slot's table costs 112 KB
// written and read again, so a log of 700k events in 512 slots spent more on
// tables (agg 18 + reduce 26 us) than on its edges.
__global__ __launch_bounds__(1024) void k_dfg_plan(int64_t nbk, int64_t nch, DfgWs ws) {
    __shared__ uint32_t tmp[1024 / kWave + 1];
    const uint64_t all = *ws.utotal;
    uint64_t chunk = (all + kDfgAggTarget - 1) / kDfgAggTarget;
    if (chunk < kDfgSlotMin) chunk = kDfgSlotMin;
    uint32_t run = 0;
    for (int64_t b0 = 0; b0 < nbk; b0 += 1024) {
        const int64_t b = b0 + threadIdx.x;
        uint32_t sl = 0, tb = 0, base = 0;
        if (b < nbk && nch > 0) {   // no chunks (empty log): empty buckets
            base = ws.escan[b * nch];
            const uint32_t next = b + 1 < nbk ? ws.escan[(b + 1) * nch] : (uint32_t)all;
            tb = next - base;
            sl = (uint32_t)((tb + chunk - 1) / chunk);
        }
        uint32_t total;
        const uint32_t ex = block_excl_sum<1024>(sl, tmp, &total);
        if (b < nbk) {
            const uint32_t first = run + ex;
            ws.bbase[b] = base;
            ws.btotal[b] = tb;
            ws.bfirst[b] = first;
            ws.bslots[b] = sl;
            for (uint32_t s = 0; s < sl; ++s) {
                const uint64_t v0 = (uint64_t)s * chunk;
                const uint64_t v1 = v0 + chunk < tb ? v0 + chunk : tb;
                ws.plan[first + s] = make_int4((int)b, (int)v0, (int)v1, 0);
            }
        }
        run += total;
    }
    if (threadIdx.x == 0) *ws.nplan = run;
}

// One block per slot: its edges are one contiguous range of its bucket.
__global__ __launch_bounds__(kAB) void k_dfg_agg(DfgWs ws) {
    __shared__ uint32_t scount[kCellsPerTable];
    __shared__ uint64_t ssum[kCellsPerTable];
    __shared__ alignas(16) int64_t smm[2 * kCellsPerTable];

    const uint32_t g = blockIdx.x;
    if (g >= *ws.nplan) return;
    const int4 pl = ws.plan[g];
    for (int c = threadIdx.x; c < kCellsPerTable; c += kAB) {
        scount[c] = 0;
        ssum[c] = 0;
        smm[2 * c] = INT64_MAX;
        smm[2 * c + 1] = INT64_MIN;
    }
    __syncthreads();
    const size_t at0 = (size_t)ws.bbase[pl.x];
    const int64_t v1 = pl.z;
    constexpr int kU = 4;   // edges in flight per thread
    int64_t v = pl.y + threadIdx.x;
    for (; v + (kU - 1) * kAB < v1; v += kU * kAB) {
        uint32_t cell[kU];
        uint64_t gap[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            cell[u] = ws.ecell[at0 + v + u * kAB];
            gap[u] = ws.egap[at0 + v + u * kAB];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) agg_edge(scount, ssum, smm, cell[u], gap[u]);
    }
    for (; v < v1; v += kAB) agg_edge(scount, ssum, smm, ws.ecell[at0 + v], ws.egap[at0 + v]);
    __syncthreads();
    const size_t slot = (size_t)g * kCellsPerTable;
    for (int c = threadIdx.x; c < kCellsPerTable; c += kAB) {
        ws.pcount[slot + c] = scount[c];
        ws.psum[slot + c] = ssum[c];
        ws.pmin[slot + c] = smm[2 * c];
        ws.pmax[slot + c] = smm[2 * c + 1];
    }
}

// ---------------------------------------------------------------------------
// Fold partial tables into the dense outputs.
// direct_slots > 0: every cell's partials are slots 0..direct_slots-1 (LDS path);
// block gridDim.x - 1 folds the activity counts and the scalars instead.
// direct_slots == 0: cell -> bucket cell>>12 -> slots bfirst..bfirst+bslots.
// A block takes CPB cells; GROUPS threads share a cell's slots (one thread per
// cell walked up to 256 slots one after the other: 84 us on 256 tables of 64
// activities).
template <int CPB, int GROUPS>
__global__ __launch_bounds__(CPB* GROUPS) void k_dfg_reduce(int32_t A, int32_t direct_slots, DfgWs ws,
                                                           const int32_t* status_in, DfgOutDev out) {
    constexpr int kT = CPB * GROUPS, kNW = kT / kWave;
    struct Part {
        uint64_t cnt, sum;
        int64_t mn, mx;
    };
    __shared__ Part red[GROUPS > 1 ? kNW * CPB : 1];
    const int64_t cells = (int64_t)A * A;
    if (direct_slots > 0 && blockIdx.x == gridDim.x - 1) {
        // thread (a, g): every (kT / 64)th slot of activity a
        __shared__ unsigned long long sf[3][kDfgLdsMaxA];
        __shared__ uint64_t sspan[kNW];
        for (int k = threadIdx.x; k < 3 * kDfgLdsMaxA; k += kT) (&sf[0][0])[k] = 0;
        __syncthreads();
        const int a = threadIdx.x & (kDfgLdsMaxA - 1);
        uint64_t f = 0, st = 0;
        int64_t en = 0;
        if (a < A) {
#pragma unroll 4
            for (int k = threadIdx.x / kDfgLdsMaxA; k < direct_slots; k += kT / kDfgLdsMaxA) {
                f += ws.pfreq[(size_t)k * A + a];
                st += ws.pstart[(size_t)k * A + a];
                en += (int32_t)ws.pend[(size_t)k * A + a];
            }
            atomicAdd(&sf[0][a], (unsigned long long)f);
            atomicAdd(&sf[1][a], (unsigned long long)st);
            atomicAdd(&sf[2][a], (unsigned long long)en);
        }
        uint64_t sp = 0;
        bool bad = false;
        for (int k = threadIdx.x; k < direct_slots; k += kT) {
            bad |= ws.pspan[k] == kBadSpan;
            sp = sat_add63(sp, cap63(ws.pspan[k]));
        }
        sp = wave_sat_sum(sp);
        if (lane() == 0) sspan[threadIdx.x / kWave] = sp;
        const int any_bad = __syncthreads_or(bad);
        if (threadIdx.x < kWave) {
            if (a < A) {
                out.act_count[a] = (int64_t)sf[0][a];
                out.start_count[a] = (int64_t)sf[1][a];
                out.end_count[a] = (int64_t)sf[2][a];
            }
            const uint64_t nc = wave_sum(a < A ? (uint64_t)sf[1][a] : 0ull);
            if (a == 0) {
                uint64_t t = 0;
                for (int k = 0; k < kNW; ++k) t = sat_add63(t, sspan[k]);
                store_scalars(out, t, (int64_t)nc, any_bad != 0, status_in);
            }
        }
        return;
    }
    const int cl = threadIdx.x % CPB;
    const int64_t e = (int64_t)blockIdx.x * CPB + cl;
    Part p{0, 0, INT64_MAX, INT64_MIN};
    if (e < cells) {
        int64_t lc = e, s0 = 0, s1 = direct_slots;
        if (direct_slots == 0) {
            const int64_t b = e >> 12;
            lc = e & (kCellsPerTable - 1);
            s0 = ws.bfirst[b];
            s1 = s0 + ws.bslots[b];
        }
#pragma unroll 4
        for (int64_t s = s0 + threadIdx.x / CPB; s < s1; s += GROUPS) {
            const size_t at = (size_t)s * kCellsPerTable + lc;
            const int64_t a = ws.pmin[at], b = ws.pmax[at];
            p.cnt += ws.pcount[at];
            p.sum += ws.psum[at];
            p.mn = a < p.mn ? a : p.mn;
            p.mx = b > p.mx ? b : p.mx;
        }
    }
    if constexpr (GROUPS > 1) {
        static_assert(CPB < kWave && kWave % CPB == 0, "a wave holds whole groups");
#pragma unroll
        for (int o = CPB; o < kWave; o <<= 1) {
            p.cnt += __shfl_xor(p.cnt, o);
            p.sum += __shfl_xor(p.sum, o);
            const int64_t a = __shfl_xor(p.mn, o), b = __shfl_xor(p.mx, o);
            p.mn = a < p.mn ? a : p.mn;
            p.mx = b > p.mx ? b : p.mx;
        }
        if (lane() < CPB) red[threadIdx.x / kWave * CPB + cl] = p;
        __syncthreads();
        if (threadIdx.x >= CPB || e >= cells) return;
        for (int k = 1; k < kNW; ++k) {
            const Part o = red[k * CPB + cl];
            p.cnt += o.cnt;
            p.sum += o.sum;
            p.mn = o.mn < p.mn ? o.mn : p.mn;
            p.mx = o.mx > p.mx ? o.mx : p.mx;
        }
    }
    if (e < cells) store_cell(out, e, p.cnt, p.sum, p.mn, p.mx);
}

// A*A > 4096, after the cells are final.  Blocks [0, ceil(A / 16)): activity,
// start and end counts of 16 activities (header).  start_rows > 0: the start
// counts are folded from that many partial rows; 0: out.start_count holds them.
// The next block: the scalars, from `nparts` partials (start_rows > 0: case
// counts and bad flags in pend, spans in pspan; 0: spans in egap, bad flags in
// ecell, the cases are the start counts).  Any further blocks: the means.
constexpr int kActs = 16;
constexpr int kAT = 1024;
__global__ __launch_bounds__(kAT) void k_dfg_acts(int32_t A, int32_t start_rows, int32_t nparts, DfgWs ws,
                                                  const int32_t* status_in, DfgOutDev out) {
    constexpr int kNW = kAT / kWave, kG = kAT / kActs;
    const int ablk = (A + kActs - 1) / kActs;
    if ((int)blockIdx.x > ablk) {
        const int64_t cells = (int64_t)A * A, stride = (int64_t)(gridDim.x - ablk - 1) * kAT;
        for (int64_t e = (int64_t)(blockIdx.x - ablk - 1) * kAT + threadIdx.x; e < cells; e += stride) {
            const int64_t c = out.count[e];
            out.dt_mean[e] = c ? (double)out.dt_sum[e] / (double)c : (double)NAN;
        }
        return;
    }
    if ((int)blockIdx.x == ablk) {
        __shared__ uint64_t r1[kNW], r2[kNW];
        uint64_t sp = 0, c = 0;
        bool bad = false;
        for (int k = threadIdx.x; k < nparts; k += kAT) {
            if (start_rows > 0) {
                sp = sat_add63(sp, ws.pspan[k]);
                c += ws.pend[k];
                bad |= ws.pend[nparts + k] != 0;
            } else {
                sp = sat_add63(sp, ws.egap[k]);
                bad |= ws.ecell[k] != 0;
            }
        }
        if (start_rows == 0)
            for (int a = threadIdx.x; a < A; a += kAT) c += (uint64_t)out.start_count[a];
        sp = wave_sat_sum(sp);
        c = wave_sum(c);
        if (lane() == 0) {
            r1[threadIdx.x / kWave] = sp;
            r2[threadIdx.x / kWave] = c;
        }
        const int any_bad = __syncthreads_or(bad);
        if (threadIdx.x == 0) {
            uint64_t s = 0, t = 0;
            for (int k = 0; k < kNW; ++k) {
                s = sat_add63(s, r1[k]);
                t += r2[k];
            }
            store_scalars(out, s, (int64_t)t, any_bad != 0, status_in);
        }
        return;
    }
    __shared__ unsigned long long sst[kActs], scol[kActs], srow[kActs];
    if (threadIdx.x < kActs) sst[threadIdx.x] = scol[threadIdx.x] = srow[threadIdx.x] = 0;
    __syncthreads();
    const int a0 = blockIdx.x * kActs, al = threadIdx.x % kActs, a = a0 + al, g = threadIdx.x / kActs;
    if (a < A) {
        uint64_t st = 0, col = 0;
#pragma unroll 8
        for (int k = g; k < start_rows; k += kG) st += ws.pstart[(size_t)k * A + a];
        if (start_rows == 0 && g == 0) st = (uint64_t)out.start_count[a];
#pragma unroll 8
        for (int b = g; b < A; b += kG) col += (uint64_t)out.count[(size_t)b * A + a];
        atomicAdd(&sst[al], (unsigned long long)st);
        atomicAdd(&scol[al], (unsigned long long)col);
    }
    for (int r = threadIdx.x / kWave; r < kActs && a0 + r < A; r += kNW) {   // wave-uniform
        uint64_t row = 0;
#pragma unroll 4
        for (int y = lane(); y < A; y += kWave) row += (uint64_t)out.count[(size_t)(a0 + r) * A + y];
        row = wave_sum(row);
        if (lane() == 0) srow[r] = row;
    }
    __syncthreads();
    if (threadIdx.x < kActs && a < A) {
        const uint64_t f = sst[al] + scol[al];
        out.act_count[a] = (int64_t)f;
        out.start_count[a] = (int64_t)sst[al];
        out.end_count[a] = (int64_t)(f - srow[al]);
    }
}

// ---------------------------------------------------------------------------
// A*A > 4096, few events: the pairs straight into the dense outputs

__global__ __launch_bounds__(256) void k_dfg_direct_init(int32_t A, DfgOutDev out) {
    const int64_t cells = (int64_t)A * A, stride = (int64_t)gridDim.x * 256;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < cells; e += stride) {
        out.count[e] = 0;
        out.dt_sum[e] = 0;
        out.dt_min[e] = INT64_MAX;
        out.dt_max[e] = INT64_MIN;
        if (e < A) out.start_count[e] = 0;
    }
}

// One wave per 256 events; its span and bad flag in egap[wave], ecell[wave]
// (free on this path, one entry per event).  The wave's lanes with the same pair
// (or the same start) add up first, for the first kRounds different ones: the
// atomics of a log's frequent pair otherwise queue on its cell at 8 ns each
// (16384 events of 65 activities, all one pair: 22 us, 225 without; all
// different: 21 and 20).
constexpr int kDirectRounds = 3;
__global__ __launch_bounds__(kWave) void k_dfg_direct(const int32_t* __restrict__ case_s,
                                                      const int32_t* __restrict__ act_s,
                                                      const int64_t* __restrict__ ts_s, int64_t n, int32_t A,
                                                      DfgWs ws, DfgOutDev out) {
    const bool aligned = ((reinterpret_cast<uintptr_t>(case_s) | reinterpret_cast<uintptr_t>(act_s) |
                           reinterpret_cast<uintptr_t>(ts_s)) & 15) == 0;
    const int64_t e0 = 4 * ((int64_t)blockIdx.x * kWave + lane());
    const Quad qd = load_quad<true>(case_s, act_s, ts_s, e0, n, n, aligned);
    uint64_t span = 0;
    bool bad = false;
    const auto add = [&](uint32_t cell, uint64_t k, uint64_t sum, int64_t mn, int64_t mx) {
        atomicAdd(reinterpret_cast<unsigned long long*>(&out.count[cell]), (unsigned long long)k);
        atomicAdd(reinterpret_cast<unsigned long long*>(&out.dt_sum[cell]), (unsigned long long)sum);
        __hip_atomic_fetch_min(&out.dt_min[cell], mn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_max(&out.dt_max[cell], mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int32_t a = qd.a[j], p = j ? qd.a[j - 1] : qd.ap;
        const bool in = e0 + j < n, ok = in && (uint32_t)a < (uint32_t)A;
        bad |= in && !ok;
        const bool first = (j ? qd.c[j - 1] : qd.cp) != qd.c[j];
        const bool pair = ok && !first && (uint32_t)p < (uint32_t)A;
        const uint64_t gap = pair ? (uint64_t)qd.t[j] - (uint64_t)(j ? qd.t[j - 1] : qd.tp) : 0;
        const uint32_t cell = pair ? (uint32_t)p * (uint32_t)A + (uint32_t)a : 0u;
        if (pair) span = sat_add63(span, cap63(gap));
        uint64_t starts = __ballot(ok && first), pairs = __ballot(pair);
        for (int r = 0; r < kDirectRounds && starts; ++r) {   // wave-uniform, as the next one
            const int l = __ffsll((unsigned long long)starts) - 1;
            const uint64_t same = __ballot(a == wave_lane(a, l)) & starts;
            if (lane() == l)
                atomicAdd(reinterpret_cast<unsigned long long*>(&out.start_count[a]), (unsigned long long)__popcll(same));
            starts &= ~same;
        }
        uint64_t alone = 0;   // pairs that too few lanes share
        for (int r = 0; r < kDirectRounds && pairs; ++r) {
            const int l = __ffsll((unsigned long long)pairs) - 1;
            const uint64_t same = __ballot(cell == wave_lane(cell, l)) & pairs;
            pairs &= ~same;
            if (__popcll(same) < 4) {
                alone |= same;
                continue;
            }
            const bool mine = (same >> lane()) & 1ull;
            const uint64_t sum = wave_sum(mine ? gap : 0);
            const int64_t mn = wave_min(mine ? (int64_t)gap : INT64_MAX), mx = wave_max(mine ? (int64_t)gap : INT64_MIN);
            if (lane() == l) add(cell, __popcll(same), sum, mn, mx);
        }
        if ((starts >> lane()) & 1ull) atomicAdd(reinterpret_cast<unsigned long long*>(&out.start_count[a]), 1ull);
        if (((pairs | alone) >> lane()) & 1ull) add(cell, 1, gap, (int64_t)gap, (int64_t)gap);
    }
    span = wave_sat_sum(span);
    const bool any_bad = __ballot(bad) != 0;
    if (lane() == 0) {
        ws.egap[blockIdx.x] = span;
        ws.ecell[blockIdx.x] = any_bad ? 1 : 0;
    }
}

hipError_t launch_dfg(const int32_t* case_s, const int32_t* act_s, const int64_t* ts_s, int64_t n, int32_t A,
                      const int32_t* status_in, DfgWs ws, DfgOutDev out, hipStream_t s, const int64_t* skip) {
    const int64_t cells = (int64_t)A * A;
    if (A <= kDfgLdsMaxA) {
        // one tile per block until every block has one; up to two tiles are one
        // block's, which saves the partial tables and the reduce launch
        const int64_t tiles = (n + kDfgTile - 1) / kDfgTile;
        const int64_t g = tiles <= 2 ? 1 : (tiles > kDfgLdsBlocks ? kDfgLdsBlocks : tiles);
        // copies of each cell: folding 16 of them costs a block some 5 us, more
        // than the conflicts of a few tiles (100k events, 16 activities, one tile
        // per block: 12.5 us with 16 copies)
        const int cmax = tiles >= 8 * g ? 4 : 1;
        int clog = 0;
        while (clog < cmax && (cells << (clog + 1)) <= kCellsPerTable) ++clog;
        {
            ProfScope p(P_DFG_MAIN, s);
            k_dfg_lds<<<(unsigned)g, kLB, 0, s>>>(case_s, act_s, ts_s, n, A, clog, ws, status_in, out, skip);
        }
        if (g > 1) {
            ProfScope p(P_DFG_REDUCE, s);
            k_dfg_reduce<16, 64><<<(unsigned)((cells + 15) / 16 + 1), 1024, 0, s>>>(A, (int32_t)g, ws, status_in, out);
        }
    } else if (n <= kDfgDirectMax) {
        const int64_t waves = (n + 4 * kWave - 1) / (4 * kWave);
        const int64_t gi = (cells + 255) / 256;
        {
            ProfScope p(P_DFG_MAIN, s);
            k_dfg_direct_init<<<(unsigned)(gi < 4096 ? gi : 4096), 256, 0, s>>>(A, out);
            if (waves > 0) k_dfg_direct<<<(unsigned)waves, kWave, 0, s>>>(case_s, act_s, ts_s, n, A, ws, out);
        }
        ProfScope p(P_DFG_REDUCE, s);
        const int64_t gm = out.dt_mean ? ((cells + kAT - 1) / kAT < 1024 ? (cells + kAT - 1) / kAT : 1024) : 0;
        k_dfg_acts<<<(unsigned)((A + kActs - 1) / kActs + 1 + gm), kAT, 0, s>>>(A, 0, (int32_t)waves, ws, status_in, out);
    } else {
        const int64_t nbk = n_buckets(A);
        const int64_t nch = dfg_chunks(n, nbk);
        const int64_t chunk = dfg_chunk(nbk);
        const unsigned g = (unsigned)ws.n_act_blocks;
        {
            ProfScope p(P_DFG_COUNT, s);
            k_dfg_count<<<g, kCB, (size_t)(A + nbk) * sizeof(uint32_t), s>>>(case_s, act_s, n, A, nbk, nch, chunk, ws,
                                                                             skip);
            dev::excl_scan<uint32_t>(ws.ecnt, &ws.scal[0], ws.escan, ws.part32, ws.utotal, s);
        }
        {
            ProfScope p(P_DFG_MAIN, s);
            k_dfg_scatter<<<g, kCB, (size_t)3 * nbk * sizeof(uint32_t), s>>>(case_s, act_s, ts_s, n, A, nbk,
                                                                           nch, chunk, ws, skip);
        }
        {
            ProfScope p(P_DFG_PLAN, s);
            k_dfg_plan<<<1, 1024, 0, s>>>(nbk, nch, ws);
        }
        {
            // every slot but one per bucket holds kDfgSlotMin edges or more
            ProfScope p(P_DFG_AGG, s);
            const int64_t full = n / kDfgSlotMin;
            k_dfg_agg<<<(unsigned)(nbk + (full < kDfgAggTarget ? full : kDfgAggTarget)), kAB, 0, s>>>(ws);
        }
        ProfScope p(P_DFG_REDUCE, s);
        // many buckets hold one slot or two each: a thread per cell; few buckets
        // share up to 512 slots, the frequent ones half of them: 16 threads per
        // cell; in between eight, so that a block has twice the cells (a call on
        // 100,000 events of 1000 activities, 245 buckets: 117 us with 16, 85 with
        // eight, 73 with one; on 20M events of Zipf activities 329, 296 and 356.
        // 65 activities, 20M such events, two buckets: 296, 303 and 431)
        if (nbk > 256)
            k_dfg_reduce<256, 1><<<(unsigned)((cells + 255) / 256), 256, 0, s>>>(A, 0, ws, status_in, out);
        else if (nbk > 32)
            k_dfg_reduce<32, 8><<<(unsigned)((cells + 31) / 32), 256, 0, s>>>(A, 0, ws, status_in, out);
        else
            k_dfg_reduce<16, 16><<<(unsigned)((cells + 15) / 16), 256, 0, s>>>(A, 0, ws, status_in, out);
        k_dfg_acts<<<(unsigned)((A + kActs - 1) / kActs + 1), kAT, 0, s>>>(A, (int32_t)g, (int32_t)g, ws, status_in, out);
    }
    return hipGetLastError();
}

}  // namespace pm4g
