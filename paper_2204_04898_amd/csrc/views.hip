// Batched drill-down views over a prepared log (Sec. 1 drill-down: each view
// is a filtered part of the log; Sec. 3: event-level timestamp filter,
// attribute filter on the activity, and the DFG re-discovered on what is kept).
//
// A view v keeps event i iff case_lo <= c_i < case_hi, t_lo <= t_i <= t_hi and
// bit a_i of its activity mask is set.  Its DFG pairs each kept event with the
// previous kept event of the same case.  Every kept event is either the first
// kept event of its case (a start) or the destination of exactly one pair, and
// either the last one (an end) or the source of exactly one pair, so
//   act_count(y) = start(y) + sum_x count(x, y),  end(x) = act_count(x) - sum_y count(x, y).
//
// Pipeline (sizes stay on the device and so do the capacity checks: the call
// never waits for the device; when a capacity is short, the kernels after the
// check return at once and the status word and the required sizes say so):
//   k_view_slice     case range -> event slice [p0, p1) (binary search in the
//                    case table); a slice always holds whole cases
//   k_view_tile_scan per-tile counts of overlapping views, offsets
//   k_view_fill      per-tile lists of overlapping views
//   k_view_count /   tile-major: a block stages one tile of the log in LDS;
//   k_view_write     its waves walk the overlapping views' parts of the tile:
//                    the view's predicate lists the kept positions (ballots),
//                    and the kept events, 64 at a time, find the previous kept
//                    event in the neighbouring lane, carried across groups and
//                    (by a backward search) across tiles.  A pair gives a
//                    record (cell = x*A+y, gap); a start gives (A*A + y, 0).
//                    The walk runs twice:
//                    count per cell bucket (cell >> 12) and take each run's
//                    place in its (view, bucket) segment with one atomic (kept
//                    per (tile, view, bucket)), then write the runs
//   k_view_place_*   (view, bucket) counters -> segment places, segment list, gate
//   k_view_agg       a block (large segments: several) per (view, bucket)
//                    segment: 4096-cell LDS table;
//                    non-empty pair cells -> temporary sparse records, start
//                    cells -> start counts
//   k_view_out_*     places of the output cells, required sizes, status
//   k_view_out       per-view lists ordered by (src, dst), offsets, FP64 mean;
//                    per view: activity and end counts from the start counts
//                    and the row / column sums
#include <math.h>

#include <atomic>
#include <random>

#include "common.hpp"
#include "devsort.hpp"
#include "internal.hpp"
#include "prof.hpp"
#include "../../include/pm4g.h"

namespace pm4g {

namespace {

constexpr int kWalkFew = 16, kWalkMany = 8;   // waves per walk block (by activities: what LDS holds)
constexpr int kMaxBuckets = 264;          // >= ceil(1024 * 1025 / 4096) = 257
constexpr int kAB2 = 1024;                // threads per aggregation block
constexpr int kFT = 1024;                 // threads per block of the persistent launch
constexpr uint64_t kRecGapLimit = 1ull << 52;   // gaps below it share a u64 with the cell

// A phase's view of the grid: block bid of nblk.  A phase launched as a
// kernel of its own takes blockIdx / gridDim; the single persistent launch
// runs every phase on its own grid, with grid barriers in between.
struct Grid {
    int64_t bid, nblk;
};
__device__ __forceinline__ Grid hw_grid() { return Grid{(int64_t)blockIdx.x, (int64_t)gridDim.x}; }


}  // namespace

int64_t view_buckets(int32_t A) {
    return ((int64_t)A * (A + 1) + kCellsPerTable - 1) / kCellsPerTable;
}

// Blocks that may share a tile's views in the walks: a log of few tiles would
// otherwise leave most of the chip idle (512 blocks fill it).  Calls in us, a
// block per tile and shared: 4096 views of 50k events (13 tiles) 2320, 451; 300
// of 200k (49 tiles) 373, 192; 100 of 1.05M (256 tiles) 457, 427.  Above 256
// tiles, or with few views, it would only stage tiles again: 16 views of 1.05M
// events 229, 243; 48 of 2M (489 tiles) 247, 281.
static int32_t walk_parts(int64_t n_tiles, int32_t V) {
    if (n_tiles < 1 || n_tiles > 256 || V < 32) return 1;
    const int64_t fill = (511 + n_tiles) / n_tiles, most = V / 16 < 16 ? V / 16 : 16;
    return (int32_t)(fill < most ? fill : most);
}

ViewWs view_ws_layout(Bump& b, int64_t n, int32_t A, int32_t V, int32_t tile, int64_t pair_cap,
                      int64_t rec_cap, int64_t cell_cap) {
    ViewWs w{};
    const size_t cc = (size_t)(cell_cap > 0 ? cell_cap : 1);
    w.cell_cap = cell_cap;
    const int64_t tiles = (n + tile - 1) / tile;
    const size_t vm = (size_t)(V > 0 ? V : 1);
    const size_t rc = (size_t)(rec_cap > 0 ? rec_cap : 1);
    w.tile = tile;
    w.n_tiles = tiles;
    w.n_buckets = (int32_t)view_buckets(A);
    w.parts = walk_parts(tiles, V);
    w.pair_cap = pair_cap;
    w.rec_cap = rec_cap;
    w.p0 = b.take<int64_t>(vm);
    w.p1 = b.take<int64_t>(vm);
    w.tcount = b.take<uint32_t>((size_t)tiles + 2);
    w.toff = b.take<uint32_t>((size_t)tiles + 2);
    w.tcursor = b.take<uint32_t>((size_t)tiles + 2);
    w.list = b.take<uint32_t>((size_t)(pair_cap > 0 ? pair_cap : 1));
    w.scal = b.take<int64_t>(16);
    w.part32 = b.take<uint32_t>(dev::kScanGrid);
    w.part64 = b.take<int64_t>(dev::kScanGrid);
    w.part64b = b.take<int64_t>(dev::kScanGrid);
    w.bar = b.take<uint64_t>(kViewMaxBlocks + 1);
    w.rec_cell = b.take<uint16_t>(rc);
    w.rec_gap = b.take<uint64_t>(rc);
    w.pair_carry = b.take<uint4>((size_t)(pair_cap > 0 ? pair_cap : 1));
    w.pair_rel = b.take<uint32_t>((size_t)(pair_cap > 0 ? pair_cap : 1) * (size_t)w.n_buckets);
    w.n_vb = (int64_t)(V > 0 ? V : 0) * w.n_buckets;
    const size_t nvb = (size_t)(w.n_vb > 0 ? w.n_vb : 1);
    w.vb_cnt = b.take<uint32_t>(nvb);
    w.vb_base = b.take<int64_t>(nvb);
    w.vb_flag = b.take<uint32_t>(nvb);
    w.vb_seg = b.take<uint32_t>(nvb);
    w.seg_key = b.take<uint32_t>(nvb);
    w.seg_rec = b.take<int64_t>(nvb + 1);
    w.seg_cells = b.take<uint32_t>(nvb);
    w.seg_tmp = b.take<int64_t>(nvb);
    w.seg_out = b.take<int64_t>(nvb);
    w.view_cells = b.take<uint32_t>(vm);
    w.t_cell = b.take<uint32_t>(cc);
    w.t_count = b.take<uint32_t>(cc);
    w.t_sum = b.take<uint64_t>(cc);
    w.t_min = b.take<int64_t>(cc);
    w.t_max = b.take<int64_t>(cc);
    w.agg_item = b.take<uint4>(kViewAggItems);
    w.agg_done = b.take<uint32_t>(kViewAggItems);
    return w;
}

namespace {

// scal: [2] #segments, [3] temporary cell cursor, [4] total output cells, [7]
// #pairs, [9] records, [10] nonzero when some case lasts 2^52 time units or
// more (records then keep the cell in a separate array), [12] the gate after
// the count walk: 0, or the status that stops the call, [13] work taken by the
// aggregation's blocks, [14] aggregation items (parts of split segments)
//
// Record places.  The count walk adds each (tile, view) pair's records per
// bucket to the (view, bucket) counter with one atomic, whose old value is the
// run's place inside that (view, bucket) segment (kept per pair and bucket);
// an exclusive scan of the counters in (view, bucket) order gives the
// segments' places, so every segment's records form one contiguous range in
// (view, bucket) order.
//
// Records.  A record's gap is at most its case's duration, so when every case
// of the log lasts less than 2^52 units a record is one u64 in rec_gap:
// cell within its bucket (12 bits) << 52 | gap.  Otherwise the cell goes to
// rec_cell and the full gap to rec_gap.

__device__ __forceinline__ void ph_init(Grid gd, ViewWs w, int32_t V, int32_t A, const int32_t* status_in,
                                        BatchedOutDev out) {
    const int64_t stride = (int64_t)gd.nblk * blockDim.x;
    const int64_t i0 = (int64_t)gd.bid * blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < w.n_tiles + 2; i += stride) {
        w.tcount[i] = 0;
        w.tcursor[i] = 0;
    }
    for (int64_t i = i0; i < V; i += stride) w.view_cells[i] = 0;
    for (int64_t i = i0; i < w.n_vb; i += stride) w.vb_cnt[i] = 0;
    for (int64_t i = i0; i < (int64_t)V * A; i += stride) out.start_count[i] = 0;
    for (int64_t i = i0; i < kViewAggItems; i += stride) w.agg_done[i] = 0;
    if (i0 < 16) w.scal[i0] = 0;
    if (i0 == 0) {
        *out.status = (status_in && *status_in) ? *status_in : 0;
        out.required[0] = 0;
        out.required[1] = 0;
        out.required[2] = 0;
        out.required[3] = 0;
        out.required[4] = 0;
    }
}

__global__ void k_view_init(ViewWs w, int32_t V, int32_t A, const int32_t* status_in, BatchedOutDev out) {
    ph_init(hw_grid(), w, V, A, status_in, out);
}

// Sets scal[10] when a case of the log lasts 2^52 time units or more (its
// last timestamp minus its first; the prepared log is sorted by (case, ts)).
__device__ __forceinline__ void ph_span(Grid gd, const int64_t* __restrict__ case_off,
                                        const int64_t* __restrict__ ts_s, const int64_t* n_cases, ViewWs w) {
    const int64_t C = *n_cases;
    bool wide = false;
    for (int64_t c = (int64_t)gd.bid * blockDim.x + threadIdx.x; c < C;
         c += (int64_t)gd.nblk * blockDim.x) {
        const uint64_t d = (uint64_t)ts_s[case_off[c + 1] - 1] - (uint64_t)ts_s[case_off[c]];
        wide |= d >= kRecGapLimit;
    }
    if (__ballot(wide) != 0 && lane() == 0) atomicOr(reinterpret_cast<unsigned long long*>(&w.scal[10]), 1ull);
}

// Event slice of every view (whole cases) and the per-tile overlap differences:
// one wave per view, whose lanes search the case table together.
__device__ __forceinline__ void ph_slice(Grid gd, const pm4g_view* views, int32_t V, const int64_t* case_off,
                                         const int32_t* case_code, const int64_t* n_cases, ViewWs w) {
    const int64_t C = *n_cases;
    const int64_t wv = ((int64_t)gd.bid * blockDim.x + threadIdx.x) / kWave;
    const int64_t nw = (int64_t)gd.nblk * blockDim.x / kWave;
    for (int64_t v = wv; v < V; v += nw) {   // wave-uniform
        const pm4g_view vw = views[v];
        int64_t p0 = 0, p1 = 0;
        if (vw.case_lo < vw.case_hi && vw.t_lo <= vw.t_hi) {
            p0 = case_off[lb_i32(case_code, C, vw.case_lo)];
            p1 = case_off[lb_i32(case_code, C, vw.case_hi)];
        }
        if (lane() != 0) continue;
        w.p0[v] = p0;
        w.p1[v] = p1;
        if (p1 > p0) {
            atomicAdd(&w.tcount[p0 / w.tile], 1u);
            atomicAdd(&w.tcount[(p1 - 1) / w.tile + 1], 0xFFFFFFFFu);   // -1
        }
    }
}

// The case spans and the views' slices: both follow the zeroing of their words
// and nothing of one depends on the other.
__global__ void k_view_slice(const pm4g_view* views, int32_t V, const int64_t* __restrict__ case_off,
                             const int64_t* __restrict__ ts_s, const int32_t* case_code, const int64_t* n_cases,
                             ViewWs w) {
    ph_slice(hw_grid(), views, V, case_off, case_code, n_cases, w);
    ph_span(hw_grid(), case_off, ts_s, n_cases, w);
}

// tcount holds differences; one block turns them into counts and offsets (each
// thread a contiguous run of tiles: two block scans in all).
__device__ __forceinline__ void ph_tile_scan(Grid gd, ViewWs w) {
    __shared__ uint32_t tmp[1024 / kWave + 1];
    if (gd.bid != 0) return;   // one block (of 1024 threads)
    const int64_t nt = w.n_tiles;
    const int64_t per = (nt + 1023) / 1024;
    const int64_t a = per * threadIdx.x < nt ? per * threadIdx.x : nt;
    const int64_t b = a + per < nt ? a + per : nt;
    uint32_t d = 0, total;
#pragma unroll 8
    for (int64_t t = a; t < b; ++t) d += w.tcount[t];
    uint32_t cnt = block_excl_sum<1024>(d, tmp, &total);
    const uint32_t cnt0 = cnt;
    uint32_t pairs = 0;
#pragma unroll 8
    for (int64_t t = a; t < b; ++t) pairs += (cnt += w.tcount[t]);
    uint32_t off = block_excl_sum<1024>(pairs, tmp, &total);
    cnt = cnt0;
#pragma unroll 8
    for (int64_t t = a; t < b; ++t) {
        cnt += w.tcount[t];
        w.tcount[t] = cnt;
        w.toff[t] = off;
        off += cnt;
    }
    if (threadIdx.x == 0) {
        w.toff[nt] = total;
        w.scal[7] = total;
    }
}

__global__ __launch_bounds__(1024) void k_view_tile_scan(ViewWs w) { ph_tile_scan(hw_grid(), w); }

// One wave per view, its lanes over the view's tiles (a view can span
// thousands of tiles; one thread per view made that a serial atomic chain).
__device__ __forceinline__ void ph_fill(Grid gd, int32_t V, ViewWs w) {
    const int64_t wv = ((int64_t)gd.bid * blockDim.x + threadIdx.x) / kWave;
    const int64_t nw = (int64_t)gd.nblk * blockDim.x / kWave;
    for (int64_t v = wv; v < V; v += nw) {
        const int64_t p0 = w.p0[v], p1 = w.p1[v];
        if (p1 <= p0) continue;
        const int64_t t1 = (p1 - 1) / w.tile;
        for (int64_t t = p0 / w.tile + lane(); t <= t1; t += kWave) {
            const int64_t at = (int64_t)w.toff[t] + atomicAdd(&w.tcursor[t], 1u);
            if (at < w.pair_cap) w.list[at] = (uint32_t)v;
        }
    }
}

__global__ void k_view_fill(int32_t V, ViewWs w) { ph_fill(hw_grid(), V, w); }

__device__ __forceinline__ bool kept(int32_t a, int64_t t, int64_t tlo, int64_t thi, const uint8_t* mask) {
    return t >= tlo && t <= thi && mask[a] != 0;
}

struct WalkState {
    bool cr_valid;   // a kept event before the window belongs to the case at its first event
    int32_t cr_a;
    int64_t cr_t;
};

// Initial state for a walk that starts at e0 inside slice [p0, p1): if the case
// at e0 - 1 continues at e0, its last kept event before e0.
__device__ WalkState walk_init(const int32_t* case_s, const int32_t* act_s, const int64_t* ts_s,
                               int64_t e0, int64_t p0, int64_t tlo, int64_t thi, int32_t A, const uint8_t* mask) {
    WalkState st{false, 0, 0};
    if (e0 <= p0) return st;   // slices start at a case start
    const int32_t cur = case_s[e0 - 1];
    if (case_s[e0] != cur) return st;
    for (int64_t hi = e0; hi > p0; hi -= kWave) {
        const int64_t i = hi - 1 - lane();
        bool same = false, k = false;
        int32_t a = 0;
        int64_t t = 0;
        if (i >= p0) {
            same = case_s[i] == cur;
            if (same) {
                a = act_s[i];
                t = ts_s[i];
                k = (uint32_t)a < (uint32_t)A && kept(a, t, tlo, thi, mask);
            }
        }
        const uint64_t kb = __ballot(k);
        const int l = kb ? (__ffsll((long long)kb) - 1) : 0;   // lowest lane = latest position
        const int32_t al = __shfl(a, l);
        const int64_t tl = __shfl(t, l);
        if (kb) {
            st.cr_valid = true;
            st.cr_a = al;
            st.cr_t = tl;
            return st;
        }
        if (__ballot(i >= p0 && !same) != 0) return st;   // reached the case start
    }
    return st;
}

// LDS of a walk block: NW waves over a TILE-event tile, for logs of up to ACTS
// activities.
//
// A block with many views on its tile counts a view per wave, the views taken
// in turn.  Otherwise, and always when records are written, waves share views:
// each wave sets one up (its slot: the activities as bytes, the window, the
// cursors), then teams of TILE / SLICE waves walk the slots, each wave its own
// slice of the tile, taking record places from the view's shared cursors.  So
// a view's runs grow by a team of waves at once and the lines that a CU has
// open in its L2 are those of a few views, where a view per wave kept more of
// them open than the L2s hold and half-filled lines went to memory; and a tile
// that few views overlap still occupies all waves.
// The walks are otherwise bound by LDS and vector instructions, so a staged
// event is one word, its case's ordinal in the tile over its activity (one
// gather, one DPP move, one comparison of high halves), a view's activity is a
// byte, where a bit took a shift, an address and a field extract, and 16 waves
// of 64 registers let two blocks fill a CU.
// 4096 views of a 99M-event log, 8.2G events tested, 2.2G kept: count walk 7.5
// to 5.8 ms, write walk 12.9 to 9.4 ms (18 GB of records: 4 ms at copy rate);
// 200 views of 2M events, 30 activities: 56 to 21 and 59 to 39 us.
constexpr int kFewActs = 512;
constexpr int kSub = 512;             // events per round (8 windows of 64)
constexpr int kList = kSub + kWave;   // a round's kept positions plus the previous round's rest
constexpr int kSlice = 1024;          // events of a wave's slice when writing (512: 9.75 ms, 1024: 9.45, 2048: 11.4)
struct PairSlot {
    int64_t tlo, thi, cr_t;   // window; the carry's timestamp
    int32_t e0, e1;           // the view's events in the tile
    uint32_t cr_ca;           // the carry: activity (of the tile's first case), or kNoCase
    uint32_t pad;
};
constexpr uint32_t kNoCase = 0xFFFF0000u;   // an ordinal that no staged event has
template <int TILE, int NW, int ACTS>
struct WalkSmem {
    static constexpr int kBuckets = (ACTS * (ACTS + 1) + kCellsPerTable - 1) / kCellsPerTable;
    static constexpr int kMaskBytes = ACTS + 4;   // a view's activities, and one never kept
    uint32_t s_ca[TILE];   // case ordinal in the tile << 16 | activity
    int64_t s_ts[TILE];
    PairSlot s_pair[NW];
    uint32_t s_cur[NW][kBuckets];
    uint32_t s_bnd[TILE / kWave];   // case boundaries of each 64 events
    uint32_t s_next;
    uint16_t s_list[NW][kList];
    uint8_t s_mask[NW][kMaskBytes];
};

// Appends the kept positions of [r0, r1) (FULL: r1 = r0 + kSub) to the wave's
// list (LIST; else they are only counted): all loads issued before any use;
// returns the list length.
template <bool FULL, bool LIST>
__device__ __forceinline__ int list_kept(const uint32_t* __restrict__ s_ca, const int64_t* __restrict__ s_ts,
                                         int r0, int r1, int64_t tlo, int64_t thi,
                                         const uint8_t* __restrict__ mask, uint16_t* __restrict__ list, int n) {
    constexpr int kU = kSub / kWave;
    const int i0 = r0 + lane();
    uint32_t av[kU];
    int64_t tv[kU];
    uint32_t mv[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int i = i0 + u * kWave;
        const int ii = FULL ? i : (i < r1 ? i : r1 - 1);   // past the end: the last event, not kept
        av[u] = s_ca[ii] & 0xFFFFu;
        tv[u] = s_ts[ii];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) mv[u] = mask[av[u]];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        // one ballot per comparison (each folds to the comparison's lane mask)
        uint64_t K = __builtin_amdgcn_ballot_w64(mv[u] != 0) & __builtin_amdgcn_ballot_w64(tv[u] >= tlo) &
                     __builtin_amdgcn_ballot_w64(tv[u] <= thi);
        if (!FULL) K &= __builtin_amdgcn_ballot_w64(i0 + u * kWave < r1);
        const uint32_t at =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(K >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)K, (uint32_t)n));
        if (LIST && __builtin_amdgcn_inverse_ballot_w64(K)) list[at] = (uint16_t)(i0 + u * kWave);
        n += __popcll(K);
    }
    return n;
}

// The carry of a walk that starts at r0 > e0 inside a view's events [e0, ..) of
// the staged tile: the last kept event before r0 of the case at r0; the view's
// own carry (pca, pt as passed) if that case reaches back to e0.
__device__ __forceinline__ void slice_carry(const uint32_t* __restrict__ s_ca, const int64_t* __restrict__ s_ts, int r0,
                                            int e0, int64_t tlo, int64_t thi, const uint8_t* __restrict__ mask,
                                            uint32_t& pca, int64_t& pt) {
    const uint32_t ord = wave_lane(s_ca[r0], 0) >> 16;
    for (int hi = r0; hi > e0; hi -= kWave) {   // wave-uniform
        const int i = hi - 1 - lane();
        uint32_t ca = kNoCase;
        int64_t t = 0;
        if (i >= e0) {
            ca = s_ca[i];
            t = s_ts[i];
        }
        const bool same = (ca >> 16) == ord;
        const uint64_t K = __ballot(same && t >= tlo && t <= thi && mask[ca & 0xFFFFu] != 0);
        if (K != 0) {
            const int l = __ffsll((long long)K) - 1;   // lowest lane = latest position
            pca = wave_lane(ca, l);
            pt = wave_lane(t, l);
            return;
        }
        if (__ballot(i >= e0 && !same) != 0) {   // the case's start
            pca = kNoCase;
            return;
        }
    }
}

// A wave's walk over [r0, r1) of the staged tile (positions in it, the same in
// every lane, as all of the walk's bounds are: they live in scalar registers),
// in rounds of kSub events; pca, pt: the last kept event before r0 in the case
// at r0.  Pass 1 tests the view's predicate on the round's events and appends
// the kept positions to the wave's list; pass 2 takes the listed kept events
// 64 at a time (a partial group waits for the next round, except in the last
// one): lane l's previous kept event of the slice is lane l - 1's (a DPP
// shift; lane 0 takes the carry, the last kept event before the group), and
// the event starts its case's kept events iff that previous one lies in
// another case or does not exist (cases are contiguous).  Every kept event
// yields one record: WRITE=false counts per bucket in cursor[], WRITE=true
// takes record places from cursor[] (each bucket's cursor starts at its run)
// and writes the records.  With one bucket (ONE: logs of up to 63 activities)
// a group's records take consecutive places and nothing but the kept events'
// number is counted: every lane's atomic would meet in one word.
template <bool WRITE, bool ONE>
__device__ __forceinline__ void walk(const uint32_t* __restrict__ s_ca, const int64_t* __restrict__ s_ts, int r0,
                                     int r1, uint32_t pca, int64_t pt, uint32_t A, int64_t tlo, int64_t thi,
                                     const uint8_t* __restrict__ mask, uint16_t* __restrict__ list,
                                     uint32_t* __restrict__ cursor, uint16_t* __restrict__ rec_cell,
                                     uint64_t* __restrict__ rec_gap, bool wide) {
    const uint32_t AA = A * A;
    int n = 0;   // listed kept positions
    for (int q0 = r0; q0 < r1; q0 += kSub) {
        const int q1 = q0 + kSub < r1 ? q0 + kSub : r1;
        constexpr bool kListed = WRITE || !ONE;
        if (q1 - q0 == kSub) n = list_kept<true, kListed>(s_ca, s_ts, q0, q1, tlo, thi, mask, list, n);
        else n = list_kept<false, kListed>(s_ca, s_ts, q0, q1, tlo, thi, mask, list, n);
        if (!kListed) continue;
        __builtin_amdgcn_wave_barrier();
        const bool last = q1 >= r1;
        int c0 = 0;
        for (; c0 + kWave <= n || (last && c0 < n); c0 += kWave) {
            const bool in = c0 + lane() < n;
            uint32_t ca = 0;
            int64_t t = 0;
            if (in) {
                const int q = list[c0 + lane()];
                ca = s_ca[q];
                if (WRITE) t = s_ts[q];
            }
            // lane l - 1's event: a DPP wave shift right by one, whose lane 0
            // (no source lane) keeps the first operand, the carry
            const uint32_t cq = (uint32_t)__builtin_amdgcn_update_dpp((int)pca, (int)ca, 0x138, 0xF, 0xF, false);
            uint64_t tq = 0;
            if (WRITE) {
                const uint32_t tql = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)pt, (int)(uint32_t)t,
                                                                           0x138, 0xF, 0xF, false);
                const uint32_t tqh = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)((uint64_t)pt >> 32),
                                                                           (int)(uint32_t)((uint64_t)t >> 32),
                                                                           0x138, 0xF, 0xF, false);
                tq = ((uint64_t)tqh << 32) | tql;
            }
            const bool starts = ((ca ^ cq) >> 16) != 0;
            const int m = n - c0 < kWave ? n - c0 : kWave;
            uint32_t first = 0;
            if (ONE && lane() == 0) first = atomicAdd(&cursor[0], (uint32_t)m);
            if (ONE) first = wave_lane(first, 0) + lane();
            if (in) {
                const uint32_t a = ca & 0xFFFFu;
                const uint32_t cell = (starts ? AA : (cq & 0xFFFFu) * A) + a;
                const uint32_t slot = ONE ? first : atomicAdd(&cursor[cell >> 12], 1u);
                if (WRITE) {   // slot: the record's place (the cursor starts at its run)
                    const uint64_t gap = starts ? 0ull : (uint64_t)t - tq;
                    const uint64_t qc = (uint64_t)(cell & (uint32_t)(kCellsPerTable - 1));
                    if (wide) {
                        rec_cell[slot] = (uint16_t)qc;
                        rec_gap[slot] = gap;
                    } else {
                        rec_gap[slot] = (qc << 52) | gap;
                    }
                }
            }
            pca = wave_lane(ca, m - 1);
            if (WRITE) pt = wave_lane(t, m - 1);
        }
        // the rest (fewer than 64) moves to the front of the list
        if (c0 > 0 && c0 < n) {
            const int rest = n - c0;
            uint16_t x = 0;
            if (lane() < rest) x = list[c0 + lane()];
            __builtin_amdgcn_wave_barrier();
            if (lane() < rest) list[lane()] = x;
        }
        n = c0 < n ? n - c0 : 0;
        __builtin_amdgcn_wave_barrier();
    }
    if (!WRITE && ONE && lane() == 0) atomicAdd(&cursor[0], (uint32_t)n);
}

// Stages tile [T0, T1): the case ordinals count the boundaries from the tile's
// start (ballots, and one scan of the counts of each 64 events).  An activity
// outside the log's range takes the mask's last byte, which no view keeps.
template <int TILE, int NW, int ACTS>
__device__ __forceinline__ void stage_tile(const int32_t* __restrict__ case_s, const int32_t* __restrict__ act_s,
                                           const int64_t* __restrict__ ts_s, int64_t T0, int64_t T1, int32_t A,
                                           WalkSmem<TILE, NW, ACTS>& S) {
    constexpr int kPer = TILE / (NW * kWave);
    static_assert(TILE / kWave <= kWave && kPer * NW * kWave == TILE, "one wave scans the counts");
    const int n = (int)(T1 - T0);
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    if (threadIdx.x == 0) S.s_next = NW;
    uint32_t ca[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = u * NW * kWave + (int)threadIdx.x;
        bool bnd = false;
        uint32_t a = 0;
        if (i < n) {
            const int32_t c = case_s[T0 + i];
            bnd = i > 0 && case_s[T0 + i - 1] != c;
            a = (uint32_t)act_s[T0 + i];
            if (a >= (uint32_t)A) a = S.kMaskBytes - 1;
            S.s_ts[i] = ts_s[T0 + i];
        }
        const uint64_t B = __ballot(bnd);
        if (lane() == 0) S.s_bnd[u * NW + wv] = (uint32_t)__popcll(B);
        ca[u] = ((uint32_t)(__popcll(B & lanes_below()) + bnd) << 16) | a;
    }
    __syncthreads();
    const uint32_t b = lane() < TILE / kWave ? S.s_bnd[lane()] : 0u;
    const uint32_t before = wave_incl_sum(b) - b;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = u * NW * kWave + (int)threadIdx.x;
        const uint32_t ord = wave_lane(before, u * NW + wv);
        if (i < n) S.s_ca[i] = ca[u] + (ord << 16);
    }
}

// The view's activities as bytes (byte a: kept), by a wave.
template <int BYTES>
__device__ __forceinline__ void stage_mask(const uint64_t* __restrict__ words, int MW, uint8_t (&mask)[BYTES]) {
    for (int q = 0; q < MW; ++q) mask[q * kWave + lane()] = (uint8_t)((words[q] >> lane()) & 1ull);
    if (lane() == 0) mask[BYTES - 1] = 0;
    __builtin_amdgcn_wave_barrier();
}

// The first `pairs` slots, walked by teams of waves.
template <bool WRITE, int SLICE, int TILE, int NW, int ACTS>
__device__ __forceinline__ void walk_slots(uint32_t A, const ViewWs& w, int pairs, bool wide,
                                           WalkSmem<TILE, NW, ACTS>& S) {
    constexpr int kTeam = TILE / SLICE;
    static_assert(NW % kTeam == 0, "whole teams");
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int s0 = (wv % kTeam) * SLICE, s1 = s0 + SLICE;
    for (int k = wv / kTeam; k < pairs; k += NW / kTeam) {
        const PairSlot& P = S.s_pair[k];
        const int e0 = wave_lane(P.e0, 0), e1 = wave_lane(P.e1, 0);
        const int r0 = s0 > e0 ? s0 : e0, r1 = s1 < e1 ? s1 : e1;
        if (r0 >= r1) continue;
        const int64_t tlo = wave_lane(P.tlo, 0), thi = wave_lane(P.thi, 0);
        uint32_t pca = wave_lane(P.cr_ca, 0);
        int64_t pt = wave_lane(P.cr_t, 0);
        if (r0 > e0 && (WRITE || w.n_buckets > 1))
            slice_carry(S.s_ca, S.s_ts, r0, e0, tlo, thi, S.s_mask[k], pca, pt);
        if (w.n_buckets == 1)
            walk<WRITE, true>(S.s_ca, S.s_ts, r0, r1, pca, pt, A, tlo, thi, S.s_mask[k], S.s_list[wv], S.s_cur[k],
                              w.rec_cell, w.rec_gap, wide);
        else
            walk<WRITE, false>(S.s_ca, S.s_ts, r0, r1, pca, pt, A, tlo, thi, S.s_mask[k], S.s_list[wv], S.s_cur[k],
                               w.rec_cell, w.rec_gap, wide);
    }
}

// The block's i-th piece of work in the walks (walk_item), or -1 past the end.
__device__ __forceinline__ int64_t walk_tile(Grid gd, int64_t i, int64_t n_items) {
    return walk_item(gd.bid, gd.nblk, i, n_items);
}

// The tile's views beyond the first NW, taken in turn by the block's waves.
__device__ __forceinline__ uint32_t next_pair(uint32_t* s_next) {
    uint32_t j = 0;
    if (lane() == 0) j = atomicAdd(s_next, 1u);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)j);
}

// Views per wave from which a block counts one view per wave (below it, waves
// left without a view cost more than the shared walk's barriers: 48 views of a
// 3M-event log, 6 views a tile, 52 us by views and 36 us shared; with 82 views a
// tile 5.8 ms by views, 9.1 ms shared).
constexpr uint32_t kManyViews = 2;

// Views of a tile per block that shares it (w.parts blocks at most): sixteen or
// more, one per wave; with fewer a block would stage the tile for less work than
// the staging.
__device__ __forceinline__ uint32_t walk_share(uint32_t views, uint32_t parts) {
    const uint32_t even = (views + parts - 1) / parts;
    return even < 16 ? 16 : even;
}

// Count walk.  After a view's walk, each non-empty bucket's run takes its
// place in the (view, bucket) segment with one atomic on the segment's
// counter; the walk's initial carry and whether the pair keeps an event are
// kept for the write walk (pair_carry: ts, 0, act | valid << 30 | kept << 31).
template <int TILE, int NW, int ACTS>
__device__ __forceinline__ void ph_count(Grid gd, const int32_t* __restrict__ case_s,
                                        const int32_t* __restrict__ act_s,
                                        const int64_t* __restrict__ ts_s, int64_t n, int32_t A,
                                        const pm4g_view* __restrict__ views,
                                        const uint64_t* __restrict__ masks, ViewWs w,
                                        WalkSmem<TILE, NW, ACTS>& S) {

    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int NB = w.n_buckets;
    const int MW = (A + 63) / 64;
    auto& mask = S.s_mask[wv];
    uint32_t* cur = S.s_cur[wv];
    if (w.scal[7] > w.pair_cap) return;   // the tile lists are incomplete: the gate stops the call
    const uint32_t parts = (uint32_t)w.parts;
    for (int64_t it = 0, at; (at = walk_tile(gd, it, w.n_tiles * parts)) >= 0; ++it) {
        const int64_t tile = (uint32_t)at / parts;
        const uint32_t part = (uint32_t)at % parts;
        const uint32_t views_n = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.tcount[tile]);
        const uint32_t share = walk_share(views_n, parts);
        const uint32_t j_lo = share * part < views_n ? share * part : views_n;
        const uint32_t cnt = views_n - j_lo < share ? views_n - j_lo : share;
        if (cnt == 0) continue;   // no view of the tile is this block's (block-uniform)
        const int64_t T0 = tile * TILE;
        const int64_t T1 = (T0 + TILE) < n ? (T0 + TILE) : n;
        stage_tile(case_s, act_s, ts_s, T0, T1, A, S);
        const int64_t off = wave_lane((int64_t)w.toff[tile] + j_lo, 0);
        __syncthreads();
        // many views: one per wave, taken in turn (no barriers); few: shared,
        // NW at a time (block-uniform)
        const bool many = cnt >= kManyViews * NW;
        for (uint32_t j = wv, j0 = 0; many ? j < cnt : j0 < cnt;) {
            const int pairs = (int)(cnt - j0 < NW ? cnt - j0 : NW);
            WalkState st{false, 0, 0};
            uint32_t v = 0;
            int64_t tlo = 0, thi = 0;
            int r0 = 0, r1 = 0;
            uint32_t cr_ca = kNoCase;
            if (j < cnt) {
                v = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.list[off + j]);
                const pm4g_view vw = views[v];
                tlo = wave_lane(vw.t_lo, 0);
                thi = wave_lane(vw.t_hi, 0);
                const int64_t p0 = wave_lane(w.p0[v], 0), p1 = wave_lane(w.p1[v], 0);
                stage_mask(masks + (size_t)v * MW, MW, mask);
                const int64_t e0 = T0 > p0 ? T0 : p0;
                r0 = (int)(e0 - T0);
                r1 = (int)((T1 < p1 ? T1 : p1) - T0);
                st = walk_init(case_s, act_s, ts_s, e0, p0, tlo, thi, A, mask);
                cr_ca = st.cr_valid ? (uint32_t)st.cr_a : kNoCase;
                for (int q = lane(); q < NB; q += kWave) cur[q] = 0;
                __builtin_amdgcn_wave_barrier();
            }
            if (many) {
                if (NB == 1)
                    walk<false, true>(S.s_ca, S.s_ts, r0, r1, cr_ca, st.cr_t, (uint32_t)A, tlo, thi, mask, S.s_list[wv],
                                      cur, w.rec_cell, w.rec_gap, false);
                else
                    walk<false, false>(S.s_ca, S.s_ts, r0, r1, cr_ca, st.cr_t, (uint32_t)A, tlo, thi, mask,
                                       S.s_list[wv], cur, w.rec_cell, w.rec_gap, false);
            } else {
                if (j < cnt && lane() == 0) S.s_pair[wv] = PairSlot{tlo, thi, st.cr_t, r0, r1, cr_ca, 0};
                __syncthreads();
                walk_slots<false, kSub>((uint32_t)A, w, pairs, false, S);
                __syncthreads();
            }
            const uint32_t jt = j;
            j0 += NW;
            j = many ? next_pair(&S.s_next) : j0 + wv;
            if (jt >= cnt) continue;
            uint32_t* rel = w.pair_rel + (size_t)(off + jt) * (size_t)NB;
            uint64_t any = 0;
            for (int q0 = 0; q0 < NB; q0 += kWave) {
                const int q = q0 + lane();
                const uint32_t c = q < NB ? cur[q] : 0u;
                any |= __ballot(c != 0);
                if (c != 0) rel[q] = atomicAdd(&w.vb_cnt[(size_t)v * NB + q], c);
            }
            if (lane() == 0) {
                const uint32_t aw = (uint32_t)(st.cr_valid ? st.cr_a : 0) | (st.cr_valid ? 1u << 30 : 0u) |
                                    (any != 0 ? 1u << 31 : 0u);
                w.pair_carry[off + jt] = make_uint4((uint32_t)(uint64_t)st.cr_t, (uint32_t)((uint64_t)st.cr_t >> 32), 0u,
                                                   aw);
            }
        }
        __syncthreads();
    }
}

template <int TILE, int NW, int ACTS>
__global__ __launch_bounds__(NW* kWave, NW == 16 ? 8 : 4) void k_view_count(const int32_t* __restrict__ case_s,
                                        const int32_t* __restrict__ act_s,
                                        const int64_t* __restrict__ ts_s, int64_t n, int32_t A,
                                        const pm4g_view* __restrict__ views,
                                        const uint64_t* __restrict__ masks, ViewWs w) {
    __shared__ WalkSmem<TILE, NW, ACTS> S;
    ph_count<TILE, NW, ACTS>(hw_grid(), case_s, act_s, ts_s, n, A, views, masks, w, S);
}

// Write walk: each (tile, view) pair's buckets start at their runs' places in
// the segment-contiguous record layout; the walk starts from the carry the
// count walk found.
template <int TILE, int NW, int ACTS>
__device__ __forceinline__ void ph_write(Grid gd, const int32_t* __restrict__ case_s,
                                        const int32_t* __restrict__ act_s,
                                        const int64_t* __restrict__ ts_s, int64_t n, int32_t A,
                                        const pm4g_view* __restrict__ views,
                                        const uint64_t* __restrict__ masks, ViewWs w,
                                        WalkSmem<TILE, NW, ACTS>& S) {
    constexpr int kQ = (WalkSmem<TILE, NW, ACTS>::kBuckets + kWave - 1) / kWave;   // buckets per lane

    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int NB = w.n_buckets;
    const int MW = (A + 63) / 64;
    const bool wide = w.scal[10] != 0;
    auto& mask = S.s_mask[wv];
    uint32_t* cur = S.s_cur[wv];
    if (w.scal[12] != 0) return;   // a capacity is short: no record is written
    const uint32_t parts = (uint32_t)w.parts;
    for (int64_t it = 0, at; (at = walk_tile(gd, it, w.n_tiles * parts)) >= 0; ++it) {
        const int64_t tile = (uint32_t)at / parts;
        const uint32_t part = (uint32_t)at % parts;
        const uint32_t views_n = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.tcount[tile]);
        const uint32_t share = walk_share(views_n, parts);
        const uint32_t j_lo = share * part < views_n ? share * part : views_n;
        const uint32_t cnt = views_n - j_lo < share ? views_n - j_lo : share;
        if (cnt == 0) continue;   // no view of the tile is this block's (block-uniform)
        const int64_t T0 = tile * TILE;
        const int64_t T1 = (T0 + TILE) < n ? (T0 + TILE) : n;
        stage_tile(case_s, act_s, ts_s, T0, T1, A, S);
        const int64_t off = wave_lane((int64_t)w.toff[tile] + j_lo, 0);
        for (uint32_t j0 = 0; j0 < cnt; j0 += NW) {   // block-uniform
            const uint32_t j = j0 + wv;
            const int pairs = (int)(cnt - j0 < NW ? cnt - j0 : NW);
            if (j < cnt) {
                const uint4 cy = w.pair_carry[off + j];
                const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)w.list[off + j]);
                // the runs' first records (buckets without a run get no record),
                // loaded before anything waits
                const uint32_t* rel = w.pair_rel + (size_t)(off + j) * (size_t)NB;
                const int64_t* vbb = w.vb_base + (size_t)v * NB;
                uint32_t qv[kQ];
#pragma unroll
                for (int u = 0; u < kQ; ++u) {
                    const int q = u * kWave + lane();
                    qv[u] = q < NB ? (uint32_t)vbb[q] + rel[q] : 0u;
                }
                const pm4g_view vw = views[v];
                const int64_t p0 = wave_lane(w.p0[v], 0), p1 = wave_lane(w.p1[v], 0);
                stage_mask(masks + (size_t)v * MW, MW, mask);
#pragma unroll
                for (int u = 0; u < kQ; ++u) {
                    const int q = u * kWave + lane();
                    if (q < NB) cur[q] = qv[u];
                }
                const int64_t e0 = T0 > p0 ? T0 : p0;
                const int64_t e1 = cy.w >> 31 ? (T1 < p1 ? T1 : p1) : e0;   // (no kept event: nothing to walk)
                if (lane() == 0)
                    S.s_pair[wv] = PairSlot{vw.t_lo, vw.t_hi, (int64_t)(((uint64_t)cy.y << 32) | cy.x), (int)(e0 - T0),
                                            (int)(e1 - T0), (cy.w >> 30) & 1u ? cy.w & 0x3FFFFFFFu : kNoCase, 0};
            }
            __syncthreads();
            walk_slots<true, kSlice>((uint32_t)A, w, pairs, wide, S);
            __syncthreads();
        }
        __syncthreads();
    }
}

template <int TILE, int NW, int ACTS>
__global__ __launch_bounds__(NW* kWave, NW == 16 ? 8 : 4) void k_view_write(const int32_t* __restrict__ case_s,
                                        const int32_t* __restrict__ act_s,
                                        const int64_t* __restrict__ ts_s, int64_t n, int32_t A,
                                        const pm4g_view* __restrict__ views,
                                        const uint64_t* __restrict__ masks, ViewWs w) {
    __shared__ WalkSmem<TILE, NW, ACTS> S;
    ph_write<TILE, NW, ACTS>(hw_grid(), case_s, act_s, ts_s, n, A, views, masks, w, S);
}

// Blocks that share a segment's records.  One block takes a segment unless
// the segment alone is a sizeable part (1/512) of the call's records: a few
// views of a few buckets would otherwise leave the chip idle behind their
// largest segment.  A block adds up about 3000 records per us and folds
// another block's table in about 2.5 us, so sqrt(count) / 96 parts make the
// two times meet, and below 65536 records (22 us) sharing gains nothing;
// count * 1024 / records bounds the parts of all segments by kViewAggItems.
// Parts have more than 16384 records each (a segment has 9216 parts^2 records
// at least), so a part's table of kCellsPerTable cells (28 bytes each) fits
// over the records it was made of.  One view of 4M events, one bucket: 1343 us
// by one block, 137 us shared; 48 views of a 3M-event log: 193 and 68 us.
__device__ __forceinline__ uint32_t seg_parts(int64_t count, int64_t records) {
    if (count < 65536 || count * 512 < records) return 1;
    const uint32_t a = (uint32_t)(sqrtf((float)count) * (1.0f / 96.0f));
    const uint32_t b = (uint32_t)(count * 1024 / records);
    return a < b ? a : b;
}

// Places of the segments: the non-empty (view, bucket) pairs in increasing
// order, each with its first record.  Every block takes a contiguous range of
// the counters: its sums first (ph_place_sum); with all blocks' sums at hand,
// each block places its own range (ph_place), and the first one, which knows
// the totals too, closes the lists and sets the gate: every capacity the later
// kernels write into is known now; if one is short (or the records exceed
// 32-bit places) the call stops here, reported at the end.  Two launches
// where flags, two scans, gate and segment list took seven.
constexpr int kPB = 256;   // threads per block of the placing kernels
__device__ __forceinline__ int64_t place_chunk(Grid gd, int64_t n) {
    return ((n + gd.nblk - 1) / gd.nblk + 3) & ~int64_t(3);
}

template <int BLOCK>
struct PlaceSmem {
    int64_t tmp[BLOCK / kWave + 1];
};

template <int BLOCK>
__device__ __forceinline__ void ph_place_sum(Grid gd, ViewWs w, PlaceSmem<BLOCK>& L) {
    const int64_t chunk = place_chunk(gd, w.n_vb);
    const int64_t b0 = gd.bid * chunk;
    const int64_t b1 = (b0 + chunk) < w.n_vb ? (b0 + chunk) : w.n_vb;
    int64_t recs = 0;
    uint32_t segs = 0;
    for (int64_t i = b0 + 4 * threadIdx.x; i < b1; i += 4 * BLOCK) {
        const uint4 c = dev::scan_load(w.vb_cnt, i, b1);
        recs += (int64_t)c.x + c.y + c.z + c.w;
        segs += (c.x != 0) + (c.y != 0) + (c.z != 0) + (c.w != 0);
    }
    int64_t r, g;
    block_excl_sum<BLOCK>(recs, L.tmp, &r);
    block_excl_sum<BLOCK>((int64_t)segs, L.tmp, &g);
    if (threadIdx.x == 0) {
        w.part64[gd.bid] = r;
        w.part32[gd.bid] = (uint32_t)g;
    }
}

__global__ __launch_bounds__(kPB) void k_view_place_sum(ViewWs w) {
    __shared__ PlaceSmem<kPB> L;
    ph_place_sum<kPB>(hw_grid(), w, L);
}

template <int BLOCK>
__device__ __forceinline__ void ph_place(Grid gd, ViewWs w, PlaceSmem<BLOCK>& L) {
    int64_t rb = 0, rt = 0, sb = 0, st = 0;   // records, segments: before this block, of all blocks
    for (int64_t k = threadIdx.x; k < gd.nblk; k += BLOCK) {
        const int64_t r = w.part64[k], g = w.part32[k];
        rt += r;
        st += g;
        if (k < gd.bid) {
            rb += r;
            sb += g;
        }
    }
    int64_t run, seg, R, S;
    block_excl_sum<BLOCK>(rb, L.tmp, &run);
    block_excl_sum<BLOCK>(sb, L.tmp, &seg);
    block_excl_sum<BLOCK>(rt, L.tmp, &R);
    block_excl_sum<BLOCK>(st, L.tmp, &S);
    if (gd.bid == 0 && threadIdx.x == 0) {
        int64_t g = 0;
        if (w.scal[7] > w.pair_cap || R > w.rec_cap) g = PM4G_E_CAPACITY;
        if (w.scal[7] <= w.pair_cap && R > (int64_t)0xFFFFFFFF) g = PM4G_E_INVALID;
        w.scal[12] = g;
        w.scal[9] = R;
        w.scal[2] = S;
        w.seg_rec[S] = R;
    }
    const int64_t chunk = place_chunk(gd, w.n_vb);
    const int64_t b0 = gd.bid * chunk;
    const int64_t b1 = (b0 + chunk) < w.n_vb ? (b0 + chunk) : w.n_vb;
    for (int64_t c0 = b0; c0 < b1; c0 += 4 * BLOCK) {   // block-uniform
        const int64_t i0 = c0 + 4 * threadIdx.x;
        const uint4 c = dev::scan_load(w.vb_cnt, i0, b1);
        const uint32_t cnt[4] = {c.x, c.y, c.z, c.w};
        // records (below 2^43) and segments of the step in one word
        int64_t v = 0, total;
#pragma unroll
        for (int q = 0; q < 4; ++q) v += (int64_t)cnt[q] + (cnt[q] ? int64_t(1) << 48 : 0);
        const int64_t ex = block_excl_sum<BLOCK>(v, L.tmp, &total);
        int64_t rec = run + (ex & ((int64_t(1) << 48) - 1));
        uint32_t g = (uint32_t)(seg + (ex >> 48));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = i0 + q;
            if (i >= b1) break;
            w.vb_base[i] = rec;
            w.vb_seg[i] = g;
            if (cnt[q] == 0) continue;
            w.seg_key[g] = (uint32_t)i;
            w.seg_rec[g] = rec;
            const uint32_t parts = seg_parts(cnt[q], R);
            if (parts > 1) {   // a segment that several blocks share is listed part by part
                const uint32_t at = (uint32_t)atomicAdd(reinterpret_cast<unsigned long long*>(&w.scal[14]),
                                                        (unsigned long long)parts);
                for (uint32_t p = 0; p < parts; ++p) w.agg_item[at + p] = make_uint4(g, p, parts, at);
            }
            rec += cnt[q];
            ++g;
        }
        run += total & ((int64_t(1) << 48) - 1);
        seg += total >> 48;
    }
}

__global__ __launch_bounds__(kPB) void k_view_place(ViewWs w) {
    __shared__ PlaceSmem<kPB> L;
    ph_place<kPB>(hw_grid(), w, L);
}

// LDS of an aggregation block: one 4096-cell table.
struct AggSmem {
    alignas(16) uint32_t scount[kCellsPerTable];
    alignas(16) uint64_t ssum[kCellsPerTable];
    alignas(16) int64_t smm[2 * kCellsPerTable];   // min, max of each cell side by side
    uint32_t tmp[kAB2 / kWave + 1];
    uint32_t s_last;
    int64_t s_next[2], s_base;
};

// LDS of an activity-count block.
template <int BLOCK>
struct ActsSmem {
    uint32_t rows[PM4G_BATCHED_MAX_ACTIVITIES];
    uint32_t cols[PM4G_BATCHED_MAX_ACTIVITIES];
    int64_t s_src[kMaxBuckets];
    uint32_t s_m[kMaxBuckets];
    int64_t red[2][BLOCK / kWave];
};

// smm: each cell's min and max side by side, read with one 16-byte load (a
// stale pair only makes an atomic run that was not needed: min only falls
// and max only rises).
__device__ __forceinline__ void view_agg_rec(uint32_t* scount, uint64_t* ssum, int64_t* smm,
                                             uint32_t cell, uint64_t gap) {
    const int64_t gg = (int64_t)gap;
    atomicAdd(&scount[cell], 1u);
    atomicAdd(reinterpret_cast<unsigned long long*>(&ssum[cell]), (unsigned long long)gap);
    const longlong2 mm = *reinterpret_cast<const longlong2*>(&smm[2 * cell]);
    if (gg < mm.x) __hip_atomic_fetch_min(&smm[2 * cell], gg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (gg > mm.y) __hip_atomic_fetch_max(&smm[2 * cell + 1], gg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A batch of records: kAggU per thread (stride kAB2) from r0 on, those before
// r1; WIDE: the cell sits in rec_cell, else in the top 12 bits.
constexpr int kAggU = 8;
constexpr int kAggBatch = kAggU * kAB2;
template <bool WIDE>
struct AggRecs {
    uint64_t x[kAggU];
    uint32_t cell[WIDE ? kAggU : 1];
};
template <bool WIDE>
__device__ __forceinline__ void agg_load(const ViewWs& w, int64_t r0, int64_t r1, AggRecs<WIDE>& a) {
    const int left = (int)(r1 - r0 < kAggBatch ? r1 - r0 : kAggBatch);   // block-uniform, may be negative
    const uint64_t* g = w.rec_gap + r0;
#pragma unroll
    for (int u = 0; u < kAggU; ++u) {
        const int i = u * kAB2 + threadIdx.x;
        if (left == kAggBatch || i < left) a.x[u] = g[i];
    }
    if constexpr (WIDE) {
        const uint16_t* c = w.rec_cell + r0;
#pragma unroll
        for (int u = 0; u < kAggU; ++u) {
            const int i = u * kAB2 + threadIdx.x;
            if (i < left) a.cell[u] = c[i];
        }
    }
}
template <bool WIDE>
__device__ __forceinline__ void agg_add(const AggRecs<WIDE>& a, int64_t r0, int64_t r1, AggSmem& L) {
    const int left = (int)(r1 - r0 < kAggBatch ? r1 - r0 : kAggBatch);
#pragma unroll
    for (int u = 0; u < kAggU; ++u) {
        if (u * kAB2 + (int)threadIdx.x >= left) break;
        if constexpr (WIDE) view_agg_rec(L.scount, L.ssum, L.smm, a.cell[u], a.x[u]);
        else view_agg_rec(L.scount, L.ssum, L.smm, (uint32_t)(a.x[u] >> 52), a.x[u] & (kRecGapLimit - 1));
    }
}

// One piece of work of an aggregation block: records [r0, r1) of segment g
// (view, bucket) = key; it: the item (segment, part, parts, first item), parts
// = 0 for a segment that is not an item.
struct AggWork {
    uint4 it;
    uint32_t key;
    int64_t r0, r1;   // the segment's records
    bool any, end;
};
__device__ __forceinline__ AggWork agg_work(const ViewWs& w, int64_t t, int64_t items, int64_t S) {
    AggWork k;
    k.end = t >= items + S;
    k.it = make_uint4(0, 0, 0, 0);
    k.key = 0;
    k.r0 = k.r1 = 0;
    if (t < items) k.it = w.agg_item[t];
    else if (!k.end) k.it.x = (uint32_t)(t - items);
    if (!k.end) {
        k.key = w.seg_key[k.it.x];
        k.r0 = w.seg_rec[k.it.x];
        k.r1 = w.seg_rec[k.it.x + 1];
    }
    return k;
}
__device__ __forceinline__ int64_t part_begin(int64_t r0, int64_t count, uint32_t part, uint32_t parts) {
    return r0 + count * part / parts;
}

// Where a part's table lies: over its own records, on a cache line of its own.
__device__ __forceinline__ uint4* part_table(const ViewWs& w, int64_t r0) {
    return reinterpret_cast<uint4*>((reinterpret_cast<uintptr_t>(w.rec_gap + r0) + 255) & ~(uintptr_t)255);
}

// A (view, bucket) segment's records are one contiguous range, streamed by a
// block into a 4096-cell LDS table; after compaction only the touched cells
// are reset, so the table is cleared once per block.  The table fills a CU's
// LDS: one block runs per CU and no other hides its waits, so the block runs
// ahead of itself.  Segments are taken from one counter (they differ by orders
// of magnitude in size), two segments before they are added up; the first
// records of the next segment are on their way while this one's cells are
// read out; and these cells wait in registers for their place (one atomic on
// the cells' cursor) while the next segment is added up.  4096 views of a 99M
// event log (2.2G records, 266,000 segments): 8.1 ms with the waits, 7.3 ms
// without; what remains is LDS time (three to five operations per record).
// A segment shared by several blocks (seg_parts): each writes its table over
// the records it has read, and the last to arrive folds the others' in.
template <bool WIDE>
__device__ __forceinline__ void agg_segments(int32_t A, const ViewWs& w, const BatchedOutDev& out, AggSmem& L) {
    uint32_t* scount = L.scount;
    uint64_t* ssum = L.ssum;
    int64_t* smm = L.smm;
    const int64_t S = w.scal[2], R = w.scal[9], items = w.scal[14];
    const int64_t AA = (int64_t)A * A;
    const int NB = w.n_buckets;
    constexpr int kPer = kCellsPerTable / kAB2;   // 4 cells per thread, blocked
    const int c0 = threadIdx.x * kPer;
    unsigned long long* ticket = reinterpret_cast<unsigned long long*>(&w.scal[13]);
    unsigned long long* cursor = reinterpret_cast<unsigned long long*>(&w.scal[3]);
    if (threadIdx.x == 0) {
        L.s_next[0] = (int64_t)atomicAdd(ticket, 1ull);
        L.s_next[1] = (int64_t)atomicAdd(ticket, 1ull);
    }
    for (int c = threadIdx.x; c < kCellsPerTable; c += kAB2) {
        scount[c] = 0;
        ssum[c] = 0;
        smm[2 * c] = INT64_MAX;
        smm[2 * c + 1] = INT64_MIN;
    }
    __syncthreads();
    // trims a work's records to its part; none for a segment whose parts are items
    auto trim = [&](AggWork& k) {
        const int64_t a = k.r0, n = k.r1 - k.r0;
        if (k.it.z != 0) {
            k.r0 = part_begin(a, n, k.it.y, k.it.z);
            k.r1 = part_begin(a, n, k.it.y + 1, k.it.z);
        }
        k.any = !k.end && (k.it.z != 0 || seg_parts(n, R) == 1);
        if (!k.any) k.r1 = k.r0;
    };
    AggRecs<WIDE> recs;
    AggWork k = agg_work(w, wave_lane(L.s_next[0], 0), items, S);
    int64_t tn = wave_lane(L.s_next[1], 0);   // the same in every lane
    trim(k);
    agg_load(w, k.r0, k.r1, recs);
    __syncthreads();
    // cells read out, not yet written: their place (thread 0), rank, values
    int64_t base0 = 0;
    uint32_t rr = 0, flags = 0, cellb = 0, total = 0;
    uint32_t cnt[kPer];
    uint64_t sum[kPer];
    int64_t mn[kPer], mx[kPer];
    uint32_t done_seg = 0;
    bool done = false;
    for (;;) {   // block-uniform
        AggWork kn = agg_work(w, tn, items, S);
        int64_t nt = 0;
        if (threadIdx.x == 0 && !k.end) nt = (int64_t)atomicAdd(ticket, 1ull);
        agg_add(recs, k.r0, k.r1, L);
        for (int64_t r = k.r0 + kAggBatch; r < k.r1; r += kAggBatch) {
            agg_load(w, r, k.r1, recs);
            agg_add(recs, r, k.r1, L);
        }
        if (threadIdx.x == 0) {
            L.s_next[0] = nt;
            L.s_base = base0;
            if (done) {
                w.seg_cells[done_seg] = total;
                w.seg_tmp[done_seg] = base0;
            }
        }
        __syncthreads();
        trim(kn);
        tn = wave_lane(L.s_next[0], 0);
        agg_load(w, kn.r0, kn.r1, recs);
        if (done) {   // the segment before this one
            const int64_t base = wave_lane(L.s_base, 0);
            if (base + (int64_t)total > w.cell_cap) flags = 0;   // over capacity: counted, not written
            int64_t at = base + rr;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                if (!(flags & (1u << q))) continue;
                w.t_cell[at] = cellb + c0 + q;
                w.t_count[at] = cnt[q];
                w.t_sum[at] = sum[q];
                w.t_min[at] = mn[q];
                w.t_max[at] = mx[q];
                ++at;
            }
        }
        if (k.end) break;
        bool mine = k.any;
        if (k.it.z > 1) {
            uint4* tab = part_table(w, k.r0);
            tab[threadIdx.x] = *reinterpret_cast<const uint4*>(&scount[c0]);
#pragma unroll
            for (int q = 0; q < kPer / 2; ++q)
                tab[kAB2 + q * kAB2 + threadIdx.x] = *reinterpret_cast<const uint4*>(&ssum[c0 + 2 * q]);
#pragma unroll
            for (int q = 0; q < kPer; ++q)
                tab[3 * kAB2 + q * kAB2 + threadIdx.x] = *reinterpret_cast<const uint4*>(&smm[2 * (c0 + q)]);
            // every wave's part has reached the L2 before one thread writes the L2
            // back, announces the table and, as the last, drops stale lines
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (threadIdx.x == 0) {
                __threadfence();
                __builtin_amdgcn_s_waitcnt(0);   // the write-back too
                L.s_last = atomicAdd(&w.agg_done[k.it.w], 1u) == k.it.z - 1;
                __threadfence();
            }
            __syncthreads();
            mine = L.s_last != 0;
            if (mine) {
                const int64_t a = w.seg_rec[k.it.x], n = w.seg_rec[k.it.x + 1] - a;
                for (uint32_t p = 0; p < k.it.z; ++p) {
                    if (p == k.it.y) continue;
                    const uint4* o = part_table(w, part_begin(a, n, p, k.it.z));
                    const uint4 oc = o[threadIdx.x];
                    uint4 os[kPer / 2], om[kPer];
#pragma unroll
                    for (int q = 0; q < kPer / 2; ++q) os[q] = o[kAB2 + q * kAB2 + threadIdx.x];
#pragma unroll
                    for (int q = 0; q < kPer; ++q) om[q] = o[3 * kAB2 + q * kAB2 + threadIdx.x];
                    const uint32_t cc[4] = {oc.x, oc.y, oc.z, oc.w};
#pragma unroll
                    for (int q = 0; q < kPer; ++q) {
                        const uint4 ov = os[q / 2];
                        scount[c0 + q] += cc[q];
                        ssum[c0 + q] += q % 2 ? ((uint64_t)ov.w << 32 | ov.z) : ((uint64_t)ov.y << 32 | ov.x);
                        const int64_t on = (int64_t)((uint64_t)om[q].y << 32 | om[q].x);
                        const int64_t ox = (int64_t)((uint64_t)om[q].w << 32 | om[q].z);
                        if (on < smm[2 * (c0 + q)]) smm[2 * (c0 + q)] = on;
                        if (ox > smm[2 * (c0 + q) + 1]) smm[2 * (c0 + q) + 1] = ox;
                    }
                }
            }
        }
        // the cells, in cell order; start cells go straight to the start counts
        const uint32_t v = k.key / (uint32_t)NB;
        cellb = (k.key % (uint32_t)NB) * (uint32_t)kCellsPerTable;
        const uint4 n4 = *reinterpret_cast<const uint4*>(&scount[c0]);
        cnt[0] = n4.x;
        cnt[1] = n4.y;
        cnt[2] = n4.z;
        cnt[3] = n4.w;
        flags = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            sum[q] = 0;   // (nothing of the segment before stays live)
            mn[q] = mx[q] = 0;
            if (cnt[q] == 0) continue;
            const int c = c0 + q;
            const int64_t cell = (int64_t)cellb + c;
            sum[q] = ssum[c];
            mn[q] = smm[2 * c];
            mx[q] = smm[2 * c + 1];
            scount[c] = 0;   // reset for the next segment
            ssum[c] = 0;
            smm[2 * c] = INT64_MAX;
            smm[2 * c + 1] = INT64_MIN;
            if (!mine) continue;
            if (cell < AA) flags |= 1u << q;
            else if (cell < AA + A) out.start_count[(size_t)v * A + (cell - AA)] = cnt[q];
        }
        rr = block_excl_sum<kAB2>((uint32_t)__popc(flags), L.tmp, &total);
        if (mine && threadIdx.x == 0) {
            base0 = (int64_t)atomicAdd(cursor, (unsigned long long)total);
            atomicAdd(&w.view_cells[v], total);
        }
        done = mine;
        done_seg = k.it.x;
        k = kn;
    }
}

__device__ __forceinline__ void ph_agg(int32_t A, const ViewWs& w, const BatchedOutDev& out, AggSmem& L) {
    if (w.scal[12] != 0) return;
    if (w.scal[10] != 0) agg_segments<true>(A, w, out, L);
    else agg_segments<false>(A, w, out, L);
}

__global__ __launch_bounds__(kAB2) void k_view_agg(int32_t A, ViewWs w, BatchedOutDev out) {
    __shared__ AggSmem S;
    ph_agg(A, w, out, S);
}

// Places of the output cells: per segment and per view, by block sums and
// then each block's own range, as for the segments; the first block ends the
// call's bookkeeping (totals, required sizes, status).
template <int BLOCK>
__device__ __forceinline__ void ph_out_sum(Grid gd, int32_t V, ViewWs w, PlaceSmem<BLOCK>& L) {
    const int64_t S = w.scal[12] ? 0 : w.scal[2];
    const int64_t ns[2] = {S, (int64_t)V};
    const uint32_t* in[2] = {w.seg_cells, w.view_cells};
    int64_t* part[2] = {w.part64, w.part64b};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int64_t chunk = place_chunk(gd, ns[k]);
        const int64_t b0 = gd.bid * chunk;
        const int64_t b1 = (b0 + chunk) < ns[k] ? (b0 + chunk) : ns[k];
        int64_t c = 0, t;
        for (int64_t i = b0 + 4 * threadIdx.x; i < b1; i += 4 * BLOCK) {
            const uint4 x = dev::scan_load(in[k], i, b1);
            c += (int64_t)x.x + x.y + x.z + x.w;
        }
        block_excl_sum<BLOCK>(c, L.tmp, &t);
        if (threadIdx.x == 0) part[k][gd.bid] = t;
    }
}

__global__ __launch_bounds__(kPB) void k_view_out_sum(int32_t V, ViewWs w) {
    __shared__ PlaceSmem<kPB> L;
    ph_out_sum<kPB>(hw_grid(), V, w, L);
}

template <int BLOCK>
__device__ __forceinline__ void ph_out_place(Grid gd, int32_t V, ViewWs w, BatchedOutDev out, PlaceSmem<BLOCK>& L) {
    const int64_t gate = w.scal[12];
    const int64_t ns[2] = {gate ? 0 : w.scal[2], (int64_t)V};
    const uint32_t* in[2] = {w.seg_cells, w.view_cells};
    const int64_t* part[2] = {w.part64, w.part64b};
    int64_t* to[2] = {w.seg_out, out.edge_off};
    int64_t cells = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        int64_t b = 0, t = 0, run, all;
        for (int64_t j = threadIdx.x; j < gd.nblk; j += BLOCK) {
            const int64_t x = part[k][j];
            t += x;
            if (j < gd.bid) b += x;
        }
        block_excl_sum<BLOCK>(b, L.tmp, &run);
        block_excl_sum<BLOCK>(t, L.tmp, &all);
        if (k == 0) cells = all;
        const int64_t chunk = place_chunk(gd, ns[k]);
        const int64_t b0 = gd.bid * chunk;
        const int64_t b1 = (b0 + chunk) < ns[k] ? (b0 + chunk) : ns[k];
        for (int64_t c0 = b0; c0 < b1; c0 += 4 * BLOCK) {   // block-uniform
            const int64_t i0 = c0 + 4 * threadIdx.x;
            const uint4 x = dev::scan_load(in[k], i0, b1);
            const uint32_t c[4] = {x.x, x.y, x.z, x.w};
            int64_t total;
            int64_t at = run + block_excl_sum<BLOCK>((int64_t)c[0] + c[1] + c[2] + c[3], L.tmp, &total);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (i0 + q < b1) to[k][i0 + q] = at;
                at += c[q];
            }
            run += total;
        }
    }
    if (gd.bid == 0 && threadIdx.x == 0) {
        const bool pairs_short = w.scal[7] > w.pair_cap;   // then the count walk did not run
        w.scal[4] = cells;
        out.edge_off[V] = cells;
        out.required[0] = cells;                            // 0 (unknown) until the records are placed
        out.required[1] = pairs_short ? 0 : w.scal[9];
        out.required[2] = w.scal[7] * (int64_t)w.n_buckets;   // run places: pairs x buckets
        out.required[3] = w.scal[7];
        out.required[4] = gate ? 0 : w.scal[3];
        if (gate) set_status(out.status, (int32_t)gate);
        else if (cells > out.cap_edges || w.scal[3] > w.cell_cap) set_status(out.status, PM4G_E_CAPACITY);
    }
}

__global__ __launch_bounds__(kPB) void k_view_out_place(int32_t V, ViewWs w, BatchedOutDev out) {
    __shared__ PlaceSmem<kPB> L;
    ph_out_place<kPB>(hw_grid(), V, w, out, L);
}

__device__ __forceinline__ void ph_copy(Grid gd, int32_t A, ViewWs w, BatchedOutDev out) {
    const int64_t S = w.scal[2];
    const bool fits = w.scal[12] == 0 && w.scal[4] <= out.cap_edges && w.scal[3] <= w.cell_cap;
    if (!fits) return;
    constexpr int kU = 4;                                      // all loads of kU steps issued before the stores
    constexpr int kMost = kCellsPerTable / (kU * kWave);       // waves that a segment can use
    const int64_t wv = ((int64_t)gd.bid * blockDim.x + threadIdx.x) / kWave;
    const int64_t nw = (int64_t)gd.nblk * blockDim.x / kWave;
    // few segments: several waves per segment, so that none copies 4096 cells alone
    const int64_t spare = S > 0 ? nw / S : 1;
    const int64_t per = spare < 1 ? 1 : (spare < kMost ? spare : kMost);
    for (int64_t q = wv; q < S * per; q += nw) {
        const int64_t g = q / per;
        const int64_t src = w.seg_tmp[g], dst = w.seg_out[g];
        const uint32_t m = w.seg_cells[g];
        for (uint32_t r0 = (uint32_t)(q % per) * kU * kWave; r0 < m; r0 += (uint32_t)per * kU * kWave) {
            uint32_t cell[kU], cnt[kU];
            uint64_t sum[kU];
            int64_t mn[kU], mx[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const uint32_t r = r0 + u * kWave + lane();
                if (r < m) {
                    cell[u] = w.t_cell[src + r];
                    cnt[u] = w.t_count[src + r];
                    sum[u] = w.t_sum[src + r];
                    mn[u] = w.t_min[src + r];
                    mx[u] = w.t_max[src + r];
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const uint32_t r = r0 + u * kWave + lane();
                if (r < m) {
                    out.src[dst + r] = (int32_t)(cell[u] / (uint32_t)A);
                    out.dst[dst + r] = (int32_t)(cell[u] % (uint32_t)A);
                    out.count[dst + r] = cnt[u];
                    out.dt_sum[dst + r] = (int64_t)sum[u];
                    out.dt_min[dst + r] = mn[u];
                    out.dt_max[dst + r] = mx[u];
                    if (out.dt_mean) out.dt_mean[dst + r] = (double)(int64_t)sum[u] / (double)(int64_t)cnt[u];
                }
            }
        }
    }
}



// Per view: its segments form a run of the sorted segment list; fold their
// cells into row and column sums; derive activity and end counts.
template <int BLOCK>
__device__ __forceinline__ void ph_acts(Grid gd, int32_t V, int32_t A, ViewWs w, BatchedOutDev out,
                                        ActsSmem<BLOCK>& L) {
    uint32_t* rows = L.rows;   // at most the view's kept events (< 2^31)
    uint32_t* cols = L.cols;
    int64_t* s_src = L.s_src;
    uint32_t* s_m = L.s_m;
    const int64_t S = w.scal[2];
    const int64_t NB = w.n_buckets;
    if (w.scal[12] != 0 || w.scal[3] > w.cell_cap) return;   // temporary cells were not all written
    for (int64_t v = gd.bid; v < V; v += gd.nblk) {
        for (int a = threadIdx.x; a < A; a += BLOCK) rows[a] = cols[a] = 0;
        __syncthreads();
        // the view's segments (at most NB): their places and cell counts to LDS
        const int64_t lo = w.vb_seg[v * NB];
        const int ns = (int)((v + 1 < V ? (int64_t)w.vb_seg[(v + 1) * NB] : S) - lo);
        for (int k = threadIdx.x; k < ns; k += BLOCK) {
            s_src[k] = w.seg_tmp[lo + k];
            s_m[k] = w.seg_cells[lo + k];
        }
        __syncthreads();
        for (int g = 0; g < ns; ++g) {
            const int64_t src = s_src[g];
            const uint32_t m = s_m[g];
            constexpr int kU = 2;
            for (uint32_t r0 = 0; r0 < m; r0 += kU * BLOCK) {
                uint32_t cell[kU], c[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const uint32_t r = r0 + u * BLOCK + threadIdx.x;
                    cell[u] = 0;
                    c[u] = 0;
                    if (r < m) {
                        cell[u] = w.t_cell[src + r];
                        c[u] = w.t_count[src + r];
                    }
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    if (c[u]) {
                        atomicAdd(&rows[cell[u] / (uint32_t)A], c[u]);
                        atomicAdd(&cols[cell[u] % (uint32_t)A], c[u]);
                    }
                }
            }
        }
        __syncthreads();
        int64_t ne = 0, nc = 0;
        for (int a = threadIdx.x; a < A; a += BLOCK) {
            const size_t at = (size_t)v * A + a;
            const int64_t st = out.start_count[at];
            const int64_t act = st + (int64_t)cols[a];
            out.act_count[at] = act;
            out.end_count[at] = act - (int64_t)rows[a];
            ne += act;
            nc += st;
        }
        ne = wave_sum(ne);
        nc = wave_sum(nc);
        if (lane() == 0) {
            L.red[0][threadIdx.x / kWave] = ne;
            L.red[1][threadIdx.x / kWave] = nc;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t a = 0, b = 0;
            for (int k = 0; k < BLOCK / kWave; ++k) {
                a += L.red[0][k];
                b += L.red[1][k];
            }
            out.n_events[v] = a;
            out.n_cases[v] = b;
        }
        __syncthreads();
    }
}

// The copy and the activity counts read the same temporary cells and write
// disjoint outputs: one launch, its first kOutCopyBlocks blocks copying and the
// others counting, so that the two latency-bound phases overlap.
constexpr int64_t kOutCopyBlocks = 2048;

__global__ __launch_bounds__(256) void k_view_out(int32_t V, int32_t A, ViewWs w, BatchedOutDev out) {
    __shared__ ActsSmem<256> S;
    if ((int64_t)blockIdx.x < kOutCopyBlocks)
        ph_copy(Grid{(int64_t)blockIdx.x, kOutCopyBlocks}, A, w, out);
    else
        ph_acts<256>(Grid{(int64_t)blockIdx.x - kOutCopyBlocks, (int64_t)gridDim.x - kOutCopyBlocks}, V, A, w,
                     out, S);
}

// ---- the single persistent launch ----

// Grid barrier of the persistent launch (every block resident: a cooperative
// launch).  Block b announces its arrival at barrier k by writing the tag
// (call epoch << 6 | k) into bar[b]; block 0 waits until every block has
// announced it and publishes the tag in bar[kViewMaxBlocks]; the others wait
// for that.  Tags are unique per call, so words left in the workspace by
// earlier calls never match.  The release fence before the arrival and the
// acquire fence after the wait make each phase's writes visible to the next
// phase on every XCD; the waits beside them are explicit, for every wave's
// stores before the block announces itself, and for the write-back of the L2
// that the release fence starts (the compiler leaves that one out where the wave
// itself has nothing outstanding).  A wait is bounded: past kBarrierPolls polls (seconds,
// far beyond any phase) the call's status becomes PM4G_E_DEVICE and the
// block goes on, so a broken schedule ends the call instead of hanging it.
constexpr int64_t kBarrierPolls = int64_t(1) << 22;

__device__ void grid_barrier(Grid gd, uint64_t* bar, uint64_t tag, int32_t* status) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x < kWave) {
        __threadfence();
        __builtin_amdgcn_s_waitcnt(0);
        if (lane() == 0) __hip_atomic_store(&bar[gd.bid], tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool late = false;
        if (gd.bid == 0) {
            for (int64_t b0 = 0; b0 < gd.nblk; b0 += kWave) {
                const int64_t b = b0 + lane();
                int64_t polls = 0;
                for (;;) {
                    const bool here = b >= gd.nblk ||
                                      __hip_atomic_load(&bar[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag;
                    if (__ballot(!here) == 0) break;
                    if (++polls > kBarrierPolls) {
                        late = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __threadfence();
            __builtin_amdgcn_s_waitcnt(0);
            if (lane() == 0) __hip_atomic_store(&bar[kViewMaxBlocks], tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (lane() == 0) {
            int64_t polls = 0;
            while (__hip_atomic_load(&bar[kViewMaxBlocks], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != tag) {
                if (++polls > kBarrierPolls) {
                    late = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        if (late && lane() == 0) set_status(status, PM4G_E_DEVICE);
        __threadfence();
        __builtin_amdgcn_s_waitcnt(0);   // the stale lines are gone before the block's other waves read
    }
    __syncthreads();
}

struct FusedArgs {
    const int32_t* case_s;
    const int32_t* act_s;
    const int64_t* ts_s;
    const int64_t* case_off;
    const int32_t* case_code;
    const int64_t* n_cases;
    const int32_t* status_in;
    const pm4g_view* views;
    const uint64_t* masks;
    int64_t n;
    int32_t A, V;
    uint64_t epoch;
    ViewWs w;
    BatchedOutDev out;
};

template <int TILE>
union FusedSmem {
    WalkSmem<TILE, kFT / kWave, PM4G_BATCHED_MAX_ACTIVITIES> walk;
    AggSmem agg;
    ActsSmem<kFT> acts;
    PlaceSmem<kFT> place;
};

// The whole batched call in one launch: the phases of the per-phase kernels,
// in the same order, separated by grid barriers.
// The kernel's arguments are read through a pointer that each phase takes
// anew from an empty register move the compiler cannot see through, so a
// phase loads the fields it uses instead of the whole set staying live (in
// scalar registers, then spilled) across the launch.
typedef const FusedArgs __attribute__((address_space(4))) KernArgs;   // the kernel-argument segment
__device__ __forceinline__ FusedArgs fresh(KernArgs* p) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+s"(p));
    return *p;
#else
    (void)p;   // the host pass compiles device code it never runs
    return FusedArgs{};
#endif
}

template <int TILE>
__global__ __launch_bounds__(kFT) void k_view_fused(FusedArgs args) {
    __shared__ FusedSmem<TILE> sm;
    const Grid gd = hw_grid();
    KernArgs* ap = (KernArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    uint64_t k = args.epoch << 6;
    int32_t* st = args.out.status;
    uint64_t* bar = args.w.bar;
#define PA (fresh(ap))
    ph_init(gd, PA.w, PA.V, PA.A, PA.status_in, PA.out);
    grid_barrier(gd, bar, ++k, st);
    ph_span(gd, PA.case_off, PA.ts_s, PA.n_cases, PA.w);
    ph_slice(gd, PA.views, PA.V, PA.case_off, PA.case_code, PA.n_cases, PA.w);
    grid_barrier(gd, bar, ++k, st);
    ph_tile_scan(gd, PA.w);
    grid_barrier(gd, bar, ++k, st);
    ph_fill(gd, PA.V, PA.w);
    grid_barrier(gd, bar, ++k, st);
    {
        const FusedArgs a = PA;
        ph_count<TILE, kFT / kWave, PM4G_BATCHED_MAX_ACTIVITIES>(gd, a.case_s, a.act_s, a.ts_s, a.n, a.A, a.views, a.masks, a.w, sm.walk);
    }
    grid_barrier(gd, bar, ++k, st);
    ph_place_sum<kFT>(gd, PA.w, sm.place);
    grid_barrier(gd, bar, ++k, st);
    ph_place<kFT>(gd, PA.w, sm.place);
    grid_barrier(gd, bar, ++k, st);
    {
        const FusedArgs a = PA;
        ph_write<TILE, kFT / kWave, PM4G_BATCHED_MAX_ACTIVITIES>(gd, a.case_s, a.act_s, a.ts_s, a.n, a.A, a.views, a.masks, a.w, sm.walk);
    }
    grid_barrier(gd, bar, ++k, st);
    ph_agg(PA.A, PA.w, PA.out, sm.agg);
    grid_barrier(gd, bar, ++k, st);
    ph_out_sum<kFT>(gd, PA.V, PA.w, sm.place);
    grid_barrier(gd, bar, ++k, st);
    ph_out_place<kFT>(gd, PA.V, PA.w, PA.out, sm.place);
    grid_barrier(gd, bar, ++k, st);
    {   // the copy on half of the blocks, the activity counts on the other half
        const int64_t half = gd.nblk / 2 > 0 ? gd.nblk / 2 : 1;
        if (gd.bid < half || gd.nblk < 2) ph_copy(Grid{gd.bid, half}, PA.A, PA.w, PA.out);
        if (gd.bid >= half || gd.nblk < 2)
            ph_acts<kFT>(gd.nblk < 2 ? gd : Grid{gd.bid - half, gd.nblk - half}, PA.V, PA.A, PA.w, PA.out, sm.acts);
    }
#undef PA
}

}  // namespace

// Grid of the persistent launch on the current device: every block resident
// (blocks per CU from the occupancy query, times the CUs), at most
// kViewMaxBlocks.
static int fused_grid(int tile) {
    static int cache[64][2] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    int& g = cache[dev][tile == 2048 ? 0 : 1];
    if (g == 0) {
        int cus = 0, per = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        const void* fn = tile == 2048 ? (const void*)k_view_fused<2048> : (const void*)k_view_fused<4096>;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kFT, 0) != hipSuccess) return 0;
        const int64_t t = (int64_t)cus * per;
        g = (int)(t < kViewMaxBlocks ? t : kViewMaxBlocks);
    }
    return g;
}

hipError_t launch_views_fused(const pm4g_prepared* p, const pm4g_view* views, const uint64_t* masks, int32_t V,
                              ViewWs w, BatchedOutDev out, hipStream_t s) {
    ProfScope ps(P_VIEW_FUSED, s);
    // call epochs: distinct per call (and, from a random start, from any word
    // an earlier owner of the workspace left behind)
    static std::atomic<uint64_t> epoch{std::random_device{}() * 0x9E3779B97F4A7C15ull};
    const int grid = fused_grid(w.tile);
    if (grid <= 0) return hipErrorInvalidConfiguration;
    FusedArgs a{p->case_s, p->act_s, p->ts_s, p->case_off, p->case_code, p->n_cases, p->status, views, masks,
                p->n_events, p->n_activities, V, epoch.fetch_add(1) & ((uint64_t(1) << 57) - 1), w, out};
    void* args[] = {&a};
    const void* fn = w.tile == 2048 ? (const void*)k_view_fused<2048> : (const void*)k_view_fused<4096>;
    return hipLaunchCooperativeKernel(fn, dim3((unsigned)grid), dim3(kFT), args, 0, s);
}

// Blocks of the placing kernels: a step of four entries per thread each, at
// most one partial sum per kScanGrid.
static unsigned place_grid(int64_t n) {
    const int64_t g = (n + 4 * kPB - 1) / (4 * kPB);
    return (unsigned)(g < 1 ? 1 : (g < dev::kScanGrid ? g : dev::kScanGrid));
}

hipError_t launch_views_plan(const pm4g_prepared* p, const pm4g_view* views, int32_t V, ViewWs w,
                             BatchedOutDev out, hipStream_t s) {
    ProfScope ps(P_VIEW_PLAN, s);
    const int32_t A = p->n_activities;
    k_view_init<<<1024, 256, 0, s>>>(w, V, A, p->status, out);
    k_view_slice<<<1024, 256, 0, s>>>(views, V, p->case_off, p->ts_s, p->case_code, p->n_cases, w);
    k_view_tile_scan<<<1, 1024, 0, s>>>(w);
    if (V > 0) k_view_fill<<<(unsigned)((V + 3) / 4), 256, 0, s>>>(V, w);
    return hipGetLastError();
}

hipError_t launch_views_count(const pm4g_prepared* p, const pm4g_view* views, const uint64_t* masks,
                              ViewWs w, int grid, hipStream_t s) {
    ProfScope ps(P_VIEW_EMIT, s);
    const int64_t n = p->n_events;
    if (w.n_tiles > 0) {
        const int64_t work = w.n_tiles * w.parts;
        const unsigned g = (unsigned)(work < grid ? work : grid);
        auto go = [&](auto kernel, int waves) {
            kernel<<<g, (unsigned)(waves * kWave), 0, s>>>(p->case_s, p->act_s, p->ts_s, n, p->n_activities, views,
                                                           masks, w);
        };
        constexpr int kMost = PM4G_BATCHED_MAX_ACTIVITIES;
        const bool few = p->n_activities <= kFewActs;
        if (w.tile == 2048 && few) go(k_view_count<2048, kWalkFew, kFewActs>, kWalkFew);
        else if (w.tile == 2048) go(k_view_count<2048, kWalkMany, kMost>, kWalkMany);
        else if (few) go(k_view_count<4096, kWalkFew, kFewActs>, kWalkFew);
        else go(k_view_count<4096, kWalkMany, kMost>, kWalkMany);
    }
    return hipGetLastError();
}

hipError_t launch_views_write(const pm4g_prepared* p, const pm4g_view* views, const uint64_t* masks,
                              ViewWs w, int grid, hipStream_t s) {
    ProfScope ps(P_VIEW_WRITE, s);
    const int64_t n = p->n_events;
    if (w.n_tiles > 0) {
        const int64_t work = w.n_tiles * w.parts;
        const unsigned g = (unsigned)(work < grid ? work : grid);
        auto go = [&](auto kernel, int waves) {
            kernel<<<g, (unsigned)(waves * kWave), 0, s>>>(p->case_s, p->act_s, p->ts_s, n, p->n_activities, views,
                                                           masks, w);
        };
        constexpr int kMost = PM4G_BATCHED_MAX_ACTIVITIES;
        const bool few = p->n_activities <= kFewActs;
        if (w.tile == 2048 && few) go(k_view_write<2048, kWalkFew, kFewActs>, kWalkFew);
        else if (w.tile == 2048) go(k_view_write<2048, kWalkMany, kMost>, kWalkMany);
        else if (few) go(k_view_write<4096, kWalkFew, kFewActs>, kWalkFew);
        else go(k_view_write<4096, kWalkMany, kMost>, kWalkMany);
    }
    return hipGetLastError();
}

// Places the (view, bucket) segments, writes the records (write walk),
// aggregates per segment.
hipError_t launch_views_reduce(const pm4g_prepared* p, const pm4g_view* views, const uint64_t* masks, int32_t V,
                               ViewWs w, BatchedOutDev out, int emit_grid, int agg_grid, hipStream_t s) {
    const int32_t A = p->n_activities;
    {
        ProfScope ps(P_VIEW_PLACE, s);
        const unsigned g = place_grid(w.n_vb);
        k_view_place_sum<<<g, kPB, 0, s>>>(w);
        k_view_place<<<g, kPB, 0, s>>>(w);
    }
    {
        const hipError_t e = launch_views_write(p, views, masks, w, emit_grid, s);
        if (e != hipSuccess) return e;
    }
    {
        ProfScope ps(P_VIEW_AGG, s);
        k_view_agg<<<(unsigned)agg_grid, kAB2, 0, s>>>(A, w, out);
    }
    {
        ProfScope ps(P_VIEW_OUT, s);
        const unsigned g = place_grid(w.n_vb);   // segments: at most the (view, bucket) pairs
        k_view_out_sum<<<g, kPB, 0, s>>>(V, w);
        k_view_out_place<<<g, kPB, 0, s>>>(V, w, out);
        k_view_out<<<(unsigned)(kOutCopyBlocks + 2048), 256, 0, s>>>(V, A, w, out);
    }
    return hipGetLastError();
}

}  // namespace pm4g
