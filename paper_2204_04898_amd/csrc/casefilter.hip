// Cases dataframe and case-level filters of a prepared log (Sec. 3: the cases
// dataframe holds, per case, its number of events and its throughput time;
// case-level filtering on them; the DFG module's paths filtering, which keeps
// or drops the cases that contain given directly-follows pairs; timestamp
// filters on whole cases; start/end activity and variant filters).
//
//   k_cases_df      per case: events = case_off[c+1] - case_off[c], throughput
//                   = ts of its last event - ts of its first (mod 2^64)
//   k_cf_contains   only with an activity or path set: a wave walks the events
//                   of 64 consecutive cases coalesced; an event whose activity
//                   (or whose pair with the previous event of its case) is in
//                   the set marks its case in LDS
//   k_cf_decide     per case: all predicates -> kept; kept events, kept flag
//                   (range, time-window, start/end activity and variant
//                   predicates read the case's first and last event and its
//                   variant id)
//   k_cf_emit       kept cases' events copied in order (a block takes a range of
//                   cases, the totals of the ranges before it summed by itself;
//                   a wave per 64 cases, coalesced writes), case table rows,
//                   case count, case_off[K], status
// Three launches at most (two scans, a check and a finish beside them were 11).
// Counts stay on the device; nothing synchronises.  Bytes: per case 16 read +
// 24 written (tables), 16 per kept event read + 16 written; the containment
// pass reads 4-8 B per event.
#include "common.hpp"
#include "devsort.hpp"
#include "internal.hpp"
#include "prof.hpp"
#include "../../include/pm4g.h"

namespace pm4g {

// Segment of event position p among 64 consecutive segments, as seg_at, with
// 32-bit starts: event positions stay below 2^31 (the log's size limit), so
// each search step exchanges one dword instead of two.  INT32_MAX marks an
// absent lane; every lane of the wave must execute it.
__device__ __forceinline__ int seg_at32(int32_t vstart, int64_t p) {
    int lo = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        const int cand = lo + step;
        if ((int64_t)__shfl(vstart, cand) <= p) lo = cand;
    }
    return lo;
}

CaseFilterWs case_filter_ws_layout(Bump& b, int64_t n) {
    CaseFilterWs w{};
    const size_t m = (size_t)(n > 0 ? n : 1);
    w.flags = b.take<uint32_t>(m);
    w.cnt = b.take<uint32_t>(m);
    w.kept = b.take<uint32_t>(m);
    w.eoff = b.take<int64_t>(m);
    w.koff = b.take<uint32_t>(m);
    w.part32 = b.take<uint32_t>(dev::kScanGrid);
    w.part64 = b.take<int64_t>(dev::kScanGrid);
    w.scal = b.take<int64_t>(8);
    w.uscal = b.take<uint32_t>(8);
    return w;
}

namespace {

constexpr int kCB = 512;
constexpr int kCGrid = 1024;

// Four cases per thread and step, their loads issued first: each case's first
// and last timestamp sit in lines of their own (with few events per case, the
// whole column is read).
__global__ __launch_bounds__(kCB) void k_cases_df(const int64_t* __restrict__ case_off,
                                                  const int64_t* __restrict__ ts_s, const int64_t* n_cases,
                                                  int64_t* __restrict__ n_events, int64_t* __restrict__ thr) {
    const int64_t C = *n_cases;
    constexpr int kU = 4;
    const int64_t stride = (int64_t)gridDim.x * kCB;
    for (int64_t c0 = (int64_t)blockIdx.x * kCB + threadIdx.x; c0 < C; c0 += kU * stride) {
        int64_t a[kU], b[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t c = c0 + u * stride < C ? c0 + u * stride : c0;
            a[u] = case_off[c];
            b[u] = case_off[c + 1];
        }
        int64_t t0[kU], t1[kU];
        if (thr) {
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                t0[u] = ts_s[a[u]];
                t1[u] = ts_s[b[u] - 1];
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t c = c0 + u * stride;
            if (c >= C) break;
            if (n_events) n_events[c] = b[u] - a[u];
            if (thr) thr[c] = (int64_t)((uint64_t)t1[u] - (uint64_t)t0[u]);
        }
    }
}

__device__ __forceinline__ bool bit_of(const uint64_t* m, int64_t b) { return (m[b >> 6] >> (b & 63)) & 1ull; }

// flags[c]: bit 0 = the case has an activity of act_mask, bit 1 = it has a
// directly-follows pair of path_mask.  A wave takes 64 cases, a lane four
// consecutive events from an aligned one on: one 16-byte load, one search for
// the first one's case, which the following ones leave at its end; the event
// before the lane's first is the lane below's last.  The path bits lie in LDS
// where they fit (LDS): a look-up of 64 scattered words took longer than all
// the rest from the caches.  20M events, 512 activities: 71 us with a search
// and a look-up in memory per event, 38 us (the activities alone: 17
// us at copy rate).
constexpr size_t kPathLds = 40 * 1024;   // bytes of path bits held in LDS: three blocks per CU at least
template <bool LDS>
__global__ __launch_bounds__(kCB) void k_cf_contains(const int32_t* __restrict__ act_s,
                                                     const int64_t* __restrict__ case_off, const int64_t* n_cases,
                                                     int32_t A, const uint64_t* __restrict__ act_mask,
                                                     const uint64_t* __restrict__ path_mask,
                                                     uint32_t* __restrict__ flags) {
    extern __shared__ uint32_t pbits[];
    __shared__ uint32_t lflag[kCB / kWave][kWave];
    __shared__ uint32_t lst[kCB / kWave][kWave + 1];   // the cases' starts, after the wave's first position
    const int64_t C = *n_cases;
    const int wl = threadIdx.x / kWave;
    const int64_t wv = ((int64_t)blockIdx.x * kCB + threadIdx.x) / kWave;
    const int64_t nw = (int64_t)gridDim.x * kCB / kWave;
    if (LDS) {
        stage_bits<kCB>(path_mask, (int64_t)A * A, pbits);
        __syncthreads();
    }
    for (int64_t c0 = wv * kWave; c0 < C; c0 += nw * kWave) {
        const int64_t c = c0 + lane();
        const bool has = c < C;
        const int64_t st = has ? case_off[c] : INT64_MAX;
        const int64_t en = has ? case_off[c + 1] : 0;
        const int last = (C - 1 - c0) < (kWave - 1) ? (int)(C - 1 - c0) : (kWave - 1);
        const int64_t base = wave_lane(st, 0);
        const int64_t end = wave_lane(en, last);
        // offsets from an aligned position fit 32 bits (a log has fewer than 2^31 events)
        const uint32_t skip = (uint32_t)((reinterpret_cast<uintptr_t>(act_s + base) / 4) & 3);
        const int32_t* from = act_s + base - skip;
        const uint32_t top = (uint32_t)(end - base) + skip;
        const uint32_t first = has ? (uint32_t)(st - base) + skip : UINT32_MAX;
        lflag[wl][lane()] = 0;
        lst[wl][lane()] = first;
        if (lane() == 0) lst[wl][kWave] = UINT32_MAX;
        wave_sync();
        int32_t carry = 0;   // the event before the step's first: none before the first case
        for (uint32_t q0 = 0; q0 < top; q0 += 4 * kWave) {   // wave-uniform
            const uint32_t q = q0 + 4 * lane();
            int32_t a[4];
            if (q >= skip && q + 3 < top) {
                const int4 x = *reinterpret_cast<const int4*>(from + q);
                a[0] = x.x;
                a[1] = x.y;
                a[2] = x.z;
                a[3] = x.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) a[j] = q + j >= skip && q + j < top ? from[q + j] : 0;
            }
            int m = seg_of32(first, q < skip ? skip : q);
            uint32_t start = lst[wl][m], nxt = lst[wl][m + 1], bits = 0;
            int32_t before = __builtin_amdgcn_update_dpp(carry, a[3], 0x138, 0xF, 0xF, false);   // lane l - 1's last
            carry = wave_lane(a[3], kWave - 1);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t p = q + j;
                if (p >= nxt) {   // cases are non-empty: one step at a time
                    if (bits) atomicOr(&lflag[wl][m], bits);
                    bits = 0;
                    ++m;
                    start = nxt;
                    nxt = lst[wl][m + 1];
                }
                if (p >= skip && p < top) {
                    if (act_mask) bits |= (uint32_t)(act_mask[a[j] >> 6] >> (a[j] & 63)) & 1u;
                    if (path_mask && p > start) {
                        const uint32_t cell = (uint32_t)before * (uint32_t)A + (uint32_t)a[j];   // below 2^24
                        const uint32_t hit = LDS ? pbits[cell >> 5] >> (cell & 31)
                                                 : (uint32_t)(path_mask[cell >> 6] >> (cell & 63));
                        bits |= (hit & 1u) << 1;
                    }
                }
                before = a[j];
            }
            if (bits) atomicOr(&lflag[wl][m], bits);
        }
        wave_sync();
        if (has) flags[c] = lflag[wl][lane()];
        wave_sync();
    }
}

// Cases [first, end) of this block, in both kernels that follow: equal ranges.
__device__ __forceinline__ int64_t range_first(int64_t C) {
    const int64_t a = (int64_t)blockIdx.x * ((C + gridDim.x - 1) / gridDim.x);
    return a < C ? a : C;
}
__device__ __forceinline__ int64_t range_end(int64_t C) {
    const int64_t per = (C + gridDim.x - 1) / gridDim.x;
    const int64_t e = (int64_t)blockIdx.x * per + per;
    return e < C ? e : C;
}

// The block's kept events and cases.
__device__ __forceinline__ void store_totals(CaseFilterWs w, int64_t ev, uint32_t cases) {
    __shared__ int64_t tmp[kCB / kWave + 1];
    __shared__ uint32_t tmp2[kCB / kWave + 1];
    int64_t te;
    uint32_t tc;
    block_excl_sum<kCB>(ev, tmp, &te);
    block_excl_sum<kCB>(cases, tmp2, &tc);
    if (threadIdx.x == 0) {
        w.part64[blockIdx.x] = te;
        w.part32[blockIdx.x] = tc;
    }
}

__global__ __launch_bounds__(kCB) void k_cf_decide(const int32_t* __restrict__ act_s,
                                                   const int64_t* __restrict__ case_off,
                                                   const int64_t* __restrict__ ts_s, const int64_t* n_cases,
                                                   pm4g_case_filter f, CaseFilterWs w) {
    const int64_t C = *n_cases;
    const bool use_act = f.act_mask != nullptr, use_path = f.path_mask != nullptr;
    int64_t events = 0;
    uint32_t cases = 0;
    for (int64_t c = range_first(C) + threadIdx.x; c < range_end(C); c += kCB) {
        const int64_t a = case_off[c], b = case_off[c + 1];
        const int64_t ev = b - a;
        const int64_t t0 = ts_s[a], t1 = ts_s[b - 1];
        const int64_t thr = (int64_t)((uint64_t)t1 - (uint64_t)t0);
        bool keep = ev >= f.min_events && ev <= f.max_events && thr >= f.min_throughput &&
                    thr <= f.max_throughput && t0 >= f.contain_lo && t1 <= f.contain_hi && t0 <= f.meet_hi &&
                    t1 >= f.meet_lo;
        if (use_act || use_path) {
            const uint32_t fl = w.flags[c];
            if (use_act) keep = keep && (fl & 1u);
            if (use_path) keep = keep && (((fl >> 1) & 1u) == (f.path_keep ? 1u : 0u));
        }
        if (f.start_mask) keep = keep && bit_of(f.start_mask, act_s[a]);
        if (f.end_mask) keep = keep && bit_of(f.end_mask, act_s[b - 1]);
        if (f.variant_mask) {
            const int64_t v = f.case_variant[c];
            const bool in = v >= 0 && v < f.n_variant_bits && bit_of(f.variant_mask, v);
            keep = keep && (in == (f.variant_keep != 0));
        }
        w.cnt[c] = keep ? (uint32_t)ev : 0u;
        events += keep ? ev : 0;
        cases += keep ? 1u : 0u;
    }
    store_totals(w, events, cases);
}

__global__ __launch_bounds__(kCB) void k_cf_emit(const int32_t* __restrict__ case_s,
                                                 const int32_t* __restrict__ act_s,
                                                 const int64_t* __restrict__ ts_s,
                                                 const int64_t* __restrict__ case_off,
                                                 const int32_t* __restrict__ case_code, const int64_t* n_cases,
                                                 CaseFilterWs w, int64_t cap, int32_t* __restrict__ o_case,
                                                 int32_t* __restrict__ o_act, int64_t* __restrict__ o_ts,
                                                 int64_t* __restrict__ o_off, int32_t* __restrict__ o_code,
                                                 int64_t* o_n_cases, int32_t* o_status, const int32_t* status_in) {
    __shared__ int64_t tmp[kCB / kWave + 1];
    const int64_t C = *n_cases;
    // kept events and cases of the ranges before this one, and of all
    int64_t run, krun, total, kept;
    {
        int64_t e = 0, k = 0, et = 0, kt = 0;
        for (int b = threadIdx.x; b < (int)gridDim.x; b += kCB) {
            const int64_t x = w.part64[b], y = w.part32[b];
            et += x;
            kt += y;
            if (b < (int)blockIdx.x) {
                e += x;
                k += y;
            }
        }
        block_excl_sum<kCB>(e, tmp, &run);
        block_excl_sum<kCB>(k, tmp, &krun);
        block_excl_sum<kCB>(et, tmp, &total);
        block_excl_sum<kCB>(kt, tmp, &kept);
    }
    const bool over = total > cap;   // the output cannot hold them: nothing is written
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        o_off[over ? 0 : kept] = over ? 0 : total;
        *o_n_cases = over ? 0 : kept;
        *o_status = (status_in && *status_in) ? *status_in : (over ? PM4G_E_CAPACITY : 0);
    }
    if (over) return;
    const int64_t c1 = range_end(C);
    for (int64_t s0 = range_first(C); s0 < c1; s0 += kCB) {   // block-uniform
        const int64_t c0 = s0 + threadIdx.x / kWave * kWave;
        const int64_t c = c0 + lane();
        const bool has = c < c1;
        int64_t src = 0, len = 0;
        if (has) {
            src = case_off[c];
            len = w.cnt[c];
        }
        // kept events below 2^31 (the log's size limit), kept cases above them
        int64_t all;
        const int64_t before = block_excl_sum<kCB>(len + (len ? int64_t(1) << 32 : 0), tmp, &all);
        const int64_t dst = run + (int64_t)(uint32_t)before;
        if (len) {
            const int64_t k = krun + (before >> 32);
            o_off[k] = dst;
            o_code[k] = case_code[c];
        }
        run += (int64_t)(uint32_t)all;
        krun += all >> 32;
        if (c0 >= c1) continue;   // wave-uniform; the block scan above is every wave's
        const int last = (c1 - 1 - c0) < (kWave - 1) ? (int)(c1 - 1 - c0) : (kWave - 1);
        const int64_t base = __shfl(dst, 0);
        const int64_t end = __shfl(dst + len, last);
        // positions fit 32 bits: output starts and the source-minus-output shift
        // are exchanged as dwords
        const int32_t dst32 = has ? (int32_t)dst : INT32_MAX;
        const int32_t shift = (int32_t)(src - (has ? dst : 0));
        // dropped cases are empty segments: the last segment starting at or before
        // p is the kept case that holds p.  Wave-uniform trip count; four 64-event
        // steps per trip, their loads issued before the stores
        constexpr int kU = 4;
        for (int64_t p0 = base; p0 < end; p0 += kU * kWave) {
            int32_t cv[kU], av[kU];
            int64_t tv[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t p = p0 + u * kWave + lane();
                const int m = seg_at32(dst32, p);
                const int32_t sh = __shfl(shift, m);
                if (p < end) {
                    const int64_t i = p + sh;
                    cv[u] = case_s[i];
                    av[u] = act_s[i];
                    tv[u] = ts_s[i];
                }
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t p = p0 + u * kWave + lane();
                if (p < end) {
                    o_case[p] = cv[u];
                    o_act[p] = av[u];
                    o_ts[p] = tv[u];
                }
            }
        }
    }
}

}  // namespace

hipError_t launch_cases_df(const pm4g_prepared* p, int64_t* n_events, int64_t* thr, hipStream_t s) {
    ProfScope ps(P_CASES, s);
    const int64_t n = p->n_events;
    const int64_t g = (n + kCB - 1) / kCB;
    k_cases_df<<<(unsigned)(g < kCGrid ? (g < 1 ? 1 : g) : kCGrid), kCB, 0, s>>>(p->case_off, p->ts_s, p->n_cases,
                                                                                n_events, thr);
    return hipGetLastError();
}

namespace {

// Sampling by cases: a case is kept iff its id's SplitMix64 key is at most the
// selected threshold.
__global__ __launch_bounds__(kCB) void k_cf_sample(const int64_t* __restrict__ case_off,
                                                   const int32_t* __restrict__ case_code, const int64_t* n_cases,
                                                   uint64_t seed, const SelState* sel, CaseFilterWs w) {
    const int64_t C = *n_cases;
    const uint64_t T = sel->T;
    const bool none = sel->none != 0, all = sel->all != 0;
    int64_t events = 0;
    uint32_t cases = 0;
    for (int64_t c = range_first(C) + threadIdx.x; c < range_end(C); c += kCB) {
        const bool keep = !none && (all || splitmix64(seed, (uint64_t)(uint32_t)case_code[c]) <= T);
        const int64_t ev = keep ? case_off[c + 1] - case_off[c] : 0;
        w.cnt[c] = (uint32_t)ev;
        events += ev;
        cases += keep ? 1u : 0u;
    }
    store_totals(w, events, cases);
}

// Blocks of the deciding and the copying kernel (the same ranges): at most the
// partials' room; n bounds the case count, which is on the device.
unsigned range_grid(int64_t n) {
    const int64_t g = (n + kCB - 1) / kCB;
    return (unsigned)(g < 1 ? 1 : (g < dev::kScanGrid ? g : dev::kScanGrid));
}

// Blocks of the containment kernel: n bounds the cases.
unsigned contains_grid(int64_t n) {
    const int64_t g = (n + kCB - 1) / kCB;
    return (unsigned)(g < 1 ? 1 : (g < kCGrid ? g : kCGrid));
}

// The kept cases (w.cnt and the ranges' totals) copied into out.
void materialise_cases(const pm4g_prepared* p, const pm4g_prepared* out, CaseFilterWs w, hipStream_t s) {
    k_cf_emit<<<range_grid(p->n_events), kCB, 0, s>>>(p->case_s, p->act_s, p->ts_s, p->case_off, p->case_code,
                                                      p->n_cases, w, out->n_events, out->case_s, out->act_s, out->ts_s,
                                                      out->case_off, out->case_code, out->n_cases, out->status,
                                                      p->status);
}

}  // namespace

hipError_t launch_filter_cases(const pm4g_prepared* p, const pm4g_case_filter* f, const pm4g_prepared* out,
                               CaseFilterWs w, hipStream_t s) {
    ProfScope ps(P_CASE_FILTER, s);
    const pm4g_case_filter fv = *f;
    if (fv.act_mask || fv.path_mask) {
        const size_t bytes = bits_bytes((int64_t)p->n_activities * p->n_activities);
        if (fv.path_mask && bytes <= kPathLds)
            k_cf_contains<true><<<contains_grid(p->n_events), kCB, bytes, s>>>(p->act_s, p->case_off, p->n_cases,
                                                                               p->n_activities, fv.act_mask,
                                                                               fv.path_mask, w.flags);
        else
            k_cf_contains<false><<<contains_grid(p->n_events), kCB, 0, s>>>(p->act_s, p->case_off, p->n_cases,
                                                                            p->n_activities, fv.act_mask, fv.path_mask,
                                                                            w.flags);
    }
    k_cf_decide<<<range_grid(p->n_events), kCB, 0, s>>>(p->act_s, p->case_off, p->ts_s, p->n_cases, fv, w);
    materialise_cases(p, out, w, s);
    return hipGetLastError();
}

hipError_t launch_sample_cases(const pm4g_prepared* p, uint64_t seed, const SelState* sel,
                               const pm4g_prepared* out, CaseFilterWs w, hipStream_t s) {
    k_cf_sample<<<range_grid(p->n_events), kCB, 0, s>>>(p->case_off, p->case_code, p->n_cases, seed, sel, w);
    materialise_cases(p, out, w, s);
    return hipGetLastError();
}

}  // namespace pm4g
