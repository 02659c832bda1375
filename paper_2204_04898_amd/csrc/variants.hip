// Trace variants of a prepared log (Sec. 3, variant level: cases grouped by
// their activity sequence, an aggregation of the per-case aggregation; the
// cases dataframe carries numbers from which each case's variant follows).
//
// Grouping is exact: cases enter an open-addressing table keyed by a 64-bit
// hash of their sequence, and a case joins a slot only if its sequence equals
// that of the case that claimed it, element by element (the sequences are
// input, so nothing has to be published with the claim); different sequences
// with one hash take different slots.  Variant ids follow (count desc,
// representative asc) with the representative the smallest case id.
//
//   k_var_clear    the table and the per-case counters
//   k_var_group    per case: sum over positions of mix(position, activity), mixed
//                  with the length (wave-cooperative, coalesced); equal hashes
//                  of a wave's 64 cases meet in LDS, one lane of each enters
//                  the table: claiming case, further members, smallest member
//   k_var_reps     representatives and their counts, in case order; histogram
//                  of the count digit (255 - min(count, 255)) per tile
//   scan           of the digit rows (more than 64 tiles)
//   k_var_order    representatives to their place by (digit, case): the final
//                  order, except among the variants of 255 cases or more
//   k_var_top      those by descending count
//   k_var_ids      counts, lengths, representatives in final order
//   k_var_emit     CSR sequences, ids of the cases
// 8 launches (sorting the cases by hash, then the variants by count, took 46,
// which was most of a call on a small log).  All sizes (cases, variants) stay
// on the device; nothing synchronises.
#include "common.hpp"
#include "devsort.hpp"
#include "internal.hpp"
#include "prof.hpp"
#include "../../include/pm4g.h"

namespace pm4g {

VarWs var_ws_layout(Bump& b, int64_t n) {
    VarWs w{};
    const size_t m = (size_t)(n > 0 ? n : 1);
    w.hash = b.take<uint64_t>(m);
    w.hash2 = b.take<uint64_t>(m);
    w.idx = b.take<uint32_t>(m);
    w.idx2 = b.take<uint32_t>(m);
    w.hist = b.take<uint32_t>(256 * (size_t)(dev::tiles(n) + 1));
    w.rowsum = b.take<uint32_t>(256);
    w.flag = b.take<uint32_t>(m);
    w.sid = b.take<uint32_t>(m);
    w.sstart = b.take<uint32_t>(m + 1);
    w.repflag = b.take<uint32_t>(m);
    w.rrank = b.take<uint32_t>(m);
    w.vcr = b.take<uint2>(m);
    w.cvar = b.take<uint32_t>(m);
    w.vkey = b.take<uint32_t>(m);
    w.vkey2 = b.take<uint32_t>(m);
    w.vidx = b.take<uint32_t>(m);
    w.vidx2 = b.take<uint32_t>(m);
    w.fid = b.take<uint32_t>(m);
    w.lens = b.take<uint32_t>(m);
    w.part32 = b.take<uint32_t>(dev::kScanGrid);
    w.part64 = b.take<int64_t>(dev::kScanGrid);
    w.scal = b.take<int64_t>(8);
    w.u32scal = b.take<uint32_t>(8);
    return w;
}

namespace {

constexpr int kGrid = 2048;
constexpr int kBlk = 256;

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Equal sequences?  By one lane; a step's loads are in flight together (at the
// end clamped to the last event).
__device__ bool same_seq(const int32_t* act_s, const int64_t* case_off, uint32_t a, uint32_t b) {
    const int64_t a0 = case_off[a], n = case_off[a + 1] - a0;
    const int64_t b0 = case_off[b];
    if (n != case_off[b + 1] - b0) return false;
    const int32_t *pa = act_s + a0, *pb = act_s + b0;
    constexpr int kU = 6, kT = 4;
    int64_t k = 0;
    for (; k + kU <= n; k += kU) {
        int32_t x[kU], y[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            x[u] = pa[k + u];
            y[u] = pb[k + u];
        }
        int32_t diff = 0;
#pragma unroll
        for (int u = 0; u < kU; ++u) diff |= x[u] ^ y[u];
        if (diff) return false;
    }
    for (; k < n; k += kT) {
        int32_t x[kT], y[kT], diff = 0;
#pragma unroll
        for (int u = 0; u < kT; ++u) {
            const int64_t i = k + u < n ? k + u : n - 1;
            x[u] = pa[i];
            y[u] = pb[i];
        }
#pragma unroll
        for (int u = 0; u < kT; ++u) diff |= x[u] ^ y[u];
        if (diff) return false;
    }
    return true;
}

// By a wave (a and b the same in every lane), for sequences of kLongSeq events
// or more: one lane's steps would follow each other.
constexpr int64_t kLongSeq = 128;
__device__ bool same_long_seq(const int32_t* act_s, const int64_t* case_off, uint32_t a, uint32_t b) {
    const int64_t a0 = case_off[a], n = case_off[a + 1] - a0;
    const int64_t b0 = case_off[b];
    if (n != case_off[b + 1] - b0) return false;
    constexpr int kU = 4;
    for (int64_t k = 0; k < n; k += kU * kWave) {
        int32_t x[kU], y[kU], diff = 0;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t i = k + u * kWave + lane();
            const int64_t ic = i < n ? i : n - 1;
            x[u] = act_s[a0 + ic];
            y[u] = act_s[b0 + ic];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) diff |= x[u] ^ y[u];
        if (__ballot(diff != 0) != 0) return false;
    }
    return true;
}

// Scalars: scal[0] C, [1] V, [2] variants of 255 cases or more.
// Counters per claiming case (more: members besides it, low: its smallest
// member if smaller); claim words: hash's low half << 32 | case + 1, 0 empty.
__device__ __forceinline__ int64_t var_slots(int64_t C) { return 2 * C; }

__global__ __launch_bounds__(kBlk) void k_var_clear(VarWs w, const int64_t* n_cases) {
    const int64_t C = *n_cases, stride = (int64_t)gridDim.x * kBlk;
    uint64_t* claim = w.hash;   // runs on into hash2
    for (int64_t i = (int64_t)blockIdx.x * kBlk + threadIdx.x; i < C; i += stride) {
        *reinterpret_cast<ulonglong2*>(claim + 2 * i) = make_ulonglong2(0, 0);
        w.repflag[i] = 0;
        w.rrank[i] = 0xFFFFFFFFu;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) w.scal[0] = C;
}

// Wave-cooperative walk over 64 consecutive segments: lane m holds the
// virtual start of segment m (INT64_MAX if absent); returns the segment that
// contains virtual position p (the last m with start_m <= p).  Starts are
// strictly increasing (segments are non-empty) and p >= start_0.  Must be
// called with all 64 lanes active (the shuffles read every lane).
__device__ __forceinline__ int seg_of(int64_t vstart, int64_t p) {
    int lo = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        const int cand = lo + step;
        if (__shfl(vstart, cand) <= p) lo = cand;
    }
    return lo;
}

// The table slot of each entering lane's case c (hash h, len events): the case
// that claimed it, c itself if it is the first.  A slot is read without a
// device-scope access first: a claim never changes, so a stale read can only
// show it empty, and the compare-and-swap then tells.  Every lane of the wave
// must execute it.
__device__ __forceinline__ uint32_t enter(bool open, uint64_t* claim, int64_t slots, uint64_t h, uint32_t c, int64_t len,
                                          const int32_t* act_s, const int64_t* case_off) {
    const uint64_t mine = (h << 32) | (uint64_t)(c + 1u);
    uint64_t p = __umul64hi(h, (uint64_t)slots);
    uint32_t lead = c;
    while (__ballot(open) != 0) {   // ends: the table has twice as many slots as cases
        bool meets = false, same = false;
        if (open) {
            uint64_t cur = __hip_atomic_load(&claim[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            if (cur == 0) {
                uint64_t want = 0;
                if (__hip_atomic_compare_exchange_strong(&claim[p], &want, mine, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT))
                    open = false;   // lead is c
                else
                    cur = want;
            }
            if (open) {
                lead = (uint32_t)cur - 1u;
                meets = (uint32_t)(cur >> 32) == (uint32_t)h;
            }
        }
        for (uint64_t m = __ballot(meets && len >= kLongSeq); m != 0; m &= m - 1) {   // wave-uniform
            const int l = __ffsll((unsigned long long)m) - 1;
            const bool eq = same_long_seq(act_s, case_off, wave_lane(c, l), wave_lane(lead, l));
            if (lane() == l) same = eq;
        }
        if (meets && len < kLongSeq) same = same_seq(act_s, case_off, c, lead);
        if (same) open = false;
        if (open) {
            lead = c;
            p = p + 1 == (uint64_t)slots ? 0 : p + 1;
        }
    }
    return lead;
}

// Sequence hash of every case, and its variant's slot.  The hash is a sum over
// positions of mix(position, activity) (order-sensitive, computable in any
// order), mixed with the length.  A wave takes 64 consecutive cases; their
// events are read in 1024-event windows with coalesced 16-byte loads into LDS,
// then each lane sums 16 consecutive events, adding a case's partial sum to
// its LDS total when it leaves the case (so a case costs one or two LDS
// additions, not one per event).
// Then the wave's equal hashes meet in a 128-slot LDS table, one lane of each
// enters the global table for all of them, and the further members of a
// variant and its smallest one are kept in a block-wide LDS cache by claiming
// case, written out at the end: a variant that holds a third of the cases costs
// two global atomics per block, not per case (they queue on one address at
// about 8 ns each: with an atomic for every case below its claiming one, a call
// on 200,000 equal cases of 50 events took 520 to 790 us, so 95).
// Bound by the latency of the scattered claims (a hash of a seventh of the
// multiplies made no difference): 0.39 ms on 5M cases of 99M events (0.45 with
// a part-filled last wave of blocks; sorting by hash and regrouping took 0.80
// ms after the hash).
constexpr int kHashWin = 1024;
constexpr int kMeet = 2 * kWave;   // LDS slots for a wave's hashes
constexpr int kMore = 512;         // claiming cases cached per block
constexpr int kGroupGrid = 1280;   // five blocks per CU, what its LDS holds: with 2048 the last 768 ran alone
__global__ __launch_bounds__(kBlk) void k_var_group(const int32_t* __restrict__ act_s,
                                                    const int64_t* __restrict__ case_off, VarWs w,
                                                    uint64_t mask, int64_t n) {
    __shared__ uint32_t meet[kBlk / kWave][kMeet];       // lane + 1 of a hash's first lane
    __shared__ unsigned long long members[kBlk / kWave][kWave];   // its lanes, a bit each
    __shared__ uint32_t lead_of[kBlk / kWave][kWave];    // its claiming case
    __shared__ uint32_t mtag[kMore], mcnt[kMore], mlow[kMore];   // claiming case + 1, further members, smallest member
    __shared__ unsigned long long hsum[kBlk / kWave][kWave];
    __shared__ int64_t sst[kBlk / kWave][kWave + 1];
    __shared__ int32_t sact[kBlk / kWave][kHashWin];
    const int64_t C = w.scal[0];
    const int wl = threadIdx.x / kWave;
    const int64_t wv = ((int64_t)blockIdx.x * kBlk + threadIdx.x) / kWave;
    const int64_t nw = (int64_t)gridDim.x * kBlk / kWave;
    const bool aligned = (reinterpret_cast<uintptr_t>(act_s) & 15) == 0;
    for (int i = threadIdx.x; i < kMore; i += kBlk) {
        mtag[i] = mcnt[i] = 0;
        mlow[i] = 0xFFFFFFFFu;
    }
    __syncthreads();
    auto more = [&](uint32_t lead, uint32_t k, uint32_t low) {
        const uint32_t at = (lead * 0x9E3779B1u) >> 23;   // 9 bits: kMore
        const uint32_t old = atomicCAS(&mtag[at], 0u, lead + 1u);
        if (old == 0u || old == lead + 1u) {
            atomicAdd(&mcnt[at], k);
            atomicMin(&mlow[at], low);
        } else {
            if (k) atomicAdd(&w.repflag[lead], k);
            if (low < lead) atomicMin(&w.rrank[lead], low);
        }
    };
    constexpr int kPer = kHashWin / kWave;   // 16 events per lane and window
    for (int64_t c0 = wv * kWave; c0 < C; c0 += nw * kWave) {
        const int64_t c = c0 + lane();
        const bool has = c < C;
        const int64_t st = has ? case_off[c] : INT64_MAX;
        const int64_t en = has ? case_off[c + 1] : 0;
        hsum[wl][lane()] = 0;
        sst[wl][lane()] = st;
        if (lane() == 0) sst[wl][kWave] = INT64_MAX;
        const int last = (C - 1 - c0) < (kWave - 1) ? (int)(C - 1 - c0) : (kWave - 1);
        const int64_t base = __shfl(st, 0);
        const int64_t end = __shfl(en, last);
        for (int64_t w0 = base & ~(int64_t)3; w0 < end; w0 += kHashWin) {   // wave-uniform
            // stage the window's activities (positions outside [base, end) are not used);
            // the 16-byte loads take in-bounds positions with no branch around them
            // and are all issued before the first store (a quad past n - 4 re-reads
            // the last aligned quad and is replaced below)
            constexpr int kQ = kHashWin / (4 * kWave);
            int4 v[kQ];
            const bool vec = aligned && n >= 4;
            const int64_t plast = (n - 4) & ~(int64_t)3;
#pragma unroll
            for (int k = 0; k < kQ; ++k) {
                const int64_t p = w0 + 4 * (k * kWave + lane());
                if (vec) v[k] = *reinterpret_cast<const int4*>(act_s + (p + 3 < n ? p : plast));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < kQ; ++k) {
                const int o = 4 * (k * kWave + lane());
                const int64_t p = w0 + o;
                if (vec && p + 3 < n) {
                    sact[wl][o] = v[k].x;
                    sact[wl][o + 1] = v[k].y;
                    sact[wl][o + 2] = v[k].z;
                    sact[wl][o + 3] = v[k].w;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) sact[wl][o + j] = p + j < n ? act_s[p + j] : 0;
                }
            }
            // lane-contiguous sums
            const int64_t q0 = w0 + (int64_t)kPer * lane();
            const int64_t lo = q0 > base ? q0 : base;
            const int64_t hi = (q0 + kPer) < end ? (q0 + kPer) : end;
            int m = seg_of(st, lo < end ? lo : end - 1);   // all lanes active
            int64_t s_m = sst[wl][m], nxt = sst[wl][m + 1];
            uint64_t acc = 0;
            for (int64_t p = lo; p < hi; ++p) {
                if (p >= nxt) {   // cases are non-empty: one step at a time
                    atomicAdd(&hsum[wl][m], (unsigned long long)acc);
                    acc = 0;
                    ++m;
                    s_m = nxt;
                    nxt = sst[wl][m + 1];
                }
                acc += mix64(((uint64_t)(p - s_m) << 13) + (uint64_t)(uint32_t)sact[wl][p - w0] +
                             0x632be59bd9b4e019ull);
            }
            if (lo < hi) atomicAdd(&hsum[wl][m], (unsigned long long)acc);
        }
        uint64_t h = mix64((uint64_t)hsum[wl][lane()] ^ mix64((uint64_t)(en - st) + 0x9e3779b97f4a7c15ull));
        if (mask) h &= mask;
        // meet: every lane finds the first lane with its hash (itself perhaps)
        meet[wl][lane()] = 0;
        meet[wl][lane() + kWave] = 0;
        members[wl][lane()] = 0;
        hsum[wl][lane()] = h;
        wave_sync();
        int first = lane();
        if (has) {
            for (uint32_t p = (uint32_t)h & (kMeet - 1);; p = (p + 1) & (kMeet - 1)) {   // 64 lanes, 128 slots
                const uint32_t old = atomicCAS(&meet[wl][p], 0u, (uint32_t)lane() + 1u);
                if (old == 0u) break;
                if ((uint64_t)hsum[wl][old - 1u] == h) {
                    first = (int)old - 1;
                    break;
                }
            }
            // one hash, another sequence: the lane enters the table by itself
            if (first != lane() && !same_seq(act_s, case_off, (uint32_t)c, (uint32_t)(c0 + first))) first = lane();
            atomicOr(&members[wl][first], 1ull << lane());
        }
        wave_sync();
        const bool enters = has && first == lane();
        const uint32_t lead = enter(enters, w.hash, var_slots(C), h, (uint32_t)c, en - st, act_s, case_off);
        if (enters) {
            lead_of[wl][lane()] = lead;
            const uint64_t m = members[wl][lane()];
            const uint32_t k = (uint32_t)__popcll(m) - (lead == (uint32_t)c ? 1u : 0u);
            const uint32_t low = (uint32_t)c0 + (uint32_t)__builtin_ctzll(m);
            if (k || low < lead) more(lead, k, low);
        }
        wave_sync();
        if (has) w.cvar[c] = lead_of[wl][first];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kMore; i += kBlk) {
        if (mcnt[i]) atomicAdd(&w.repflag[mtag[i] - 1u], mcnt[i]);
        if (mtag[i] && mlow[i] < mtag[i] - 1u) atomicMin(&w.rrank[mtag[i] - 1u], mlow[i]);
    }
}

// Representative of every case (w.idx), and the count of a representative's
// variant (w.idx2; 0 for the other cases); per tile the histogram of the
// representatives' count digits.
__device__ __forceinline__ uint32_t count_digit(uint32_t count) { return 255u - (count < 255u ? count : 255u); }

__global__ __launch_bounds__(dev::kB) void k_var_reps(VarWs w, int64_t nb) {
    __shared__ uint32_t h[256];
    const int64_t C = w.scal[0], tiles_n = (C + dev::kTile - 1) / dev::kTile;
    for (int64_t tile = blockIdx.x; tile < tiles_n; tile += gridDim.x) {
        if (threadIdx.x < 256) h[threadIdx.x] = 0;
        __syncthreads();
        uint32_t lead[dev::kI], low[dev::kI], cnt[dev::kI];
#pragma unroll
        for (int k = 0; k < dev::kI; ++k) {
            const int64_t c = tile * dev::kTile + k * dev::kB + threadIdx.x;
            lead[k] = w.cvar[c < C ? c : C - 1];
        }
#pragma unroll
        for (int k = 0; k < dev::kI; ++k) {
            low[k] = w.rrank[lead[k]];
            cnt[k] = w.repflag[lead[k]] + 1u;
        }
#pragma unroll
        for (int k = 0; k < dev::kI; ++k) {
            const int64_t c = tile * dev::kTile + k * dev::kB + threadIdx.x;
            if (c >= C) continue;
            const uint32_t rep = low[k] < lead[k] ? low[k] : lead[k];
            const bool is = rep == (uint32_t)c;
            w.idx[c] = rep;
            w.idx2[c] = is ? cnt[k] : 0u;
            if (is) atomicAdd(&h[count_digit(cnt[k])], 1u);
        }
        __syncthreads();
        if (threadIdx.x < 256) w.hist[(int64_t)threadIdx.x * nb + tile] = h[threadIdx.x];
        __syncthreads();
    }
}

// Representatives (count, case) to their place by (digit, case), in vcr: one
// stable digit pass over the cases, as dev::k_scatter, where only the
// representatives take part.
// Up to kFewTiles tiles the rows are not scanned: each block adds them up
// itself (64 words of a digit at most, against a launch of 4.5 us).
constexpr int64_t kFewTiles = 64;
__global__ __launch_bounds__(dev::kB) void k_var_order(VarWs w, int64_t nb) {
    using namespace dev;
    __shared__ uint32_t cnt[kW * 256];
    __shared__ uint32_t tstart[256];
    __shared__ int64_t gshift[256];
    __shared__ uint32_t scnt[kTile];
    __shared__ uint32_t scase[kTile];
    __shared__ uint32_t tmp[kB / kWave + 1];

    const int64_t C = w.scal[0], tiles_n = (C + kTile - 1) / kTile;
    const int wv = threadIdx.x / kWave;
    uint32_t all;
    const bool scanned = nb > kFewTiles;
    // elements of this thread's digit in the tiles before `tile`
    auto before = [&](int64_t tile) {
        uint32_t x = 0;
#pragma unroll 8
        for (int64_t t = 0; t < tile; ++t) x += w.hist[(int64_t)threadIdx.x * nb + t];
        return x;
    };
    const uint32_t rs = threadIdx.x >= 256 ? 0u : scanned ? w.rowsum[threadIdx.x] : before(tiles_n);
    const uint32_t digit_base = block_excl_sum<kB>(rs, tmp, &all);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        w.scal[1] = all;   // V
        w.scal[2] = rs;    // digit 0: 255 cases or more
    }
    const XcdSplit xs = xcd_split(tiles_n);
    for (int64_t tile = xs.first; tile < xs.end; tile += xs.stride) {
        const int64_t wbase = tile * kTile + (int64_t)wv * (kWave * kI);
        for (int i = threadIdx.x; i < kW * 256; i += kB) cnt[i] = 0;
        uint32_t key[kI], rk[kI];
#pragma unroll
        for (int k = 0; k < kI; ++k) {
            const int64_t i = wbase + k * kWave + lane();
            key[k] = i < C ? w.idx2[i] : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kI; ++k) {
            const bool valid = key[k] != 0u;
            const uint32_t d = count_digit(key[k]);
            const uint64_t peers = match_digit<8>(d, __ballot(valid));
            const uint32_t below = __popcll(peers & lanes_below());
            uint32_t c = 0;
            if (valid) c = cnt[wv * 256 + d];
            rk[k] = c + below;
            if (valid && below == 0) cnt[wv * 256 + d] = c + __popcll(peers);
        }
        __syncthreads();
        uint32_t tot = 0;
        if (threadIdx.x < 256) {
            uint32_t run = 0;
            for (int ww = 0; ww < kW; ++ww) {
                const uint32_t x = cnt[ww * 256 + threadIdx.x];
                cnt[ww * 256 + threadIdx.x] = run;
                run += x;
            }
            tot = run;
        }
        uint32_t reps;
        const uint32_t ex = block_excl_sum<kB>(tot, tmp, &reps);
        if (threadIdx.x < 256) {
            tstart[threadIdx.x] = ex;
            const uint32_t at = scanned ? w.hist[(int64_t)threadIdx.x * nb + tile] : before(tile);
            gshift[threadIdx.x] = (int64_t)digit_base + (int64_t)at - (int64_t)ex;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kI; ++k) {
            if (key[k] == 0u) continue;
            const uint32_t d = count_digit(key[k]);
            const uint32_t pos = tstart[d] + cnt[wv * 256 + d] + rk[k];
            scnt[pos] = key[k];
            scase[pos] = (uint32_t)(wbase + k * kWave + lane());
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < reps; i += kB)
            w.vcr[gshift[count_digit(scnt[i])] + i] = make_uint2(scnt[i], scase[i]);
        __syncthreads();
    }
}

// The variants of 255 cases or more (the first scal[2] of vcr, in case order)
// by descending count, case order kept among equals.  At most 16384 of them:
// an element's place is the number of elements before it, counted over all of
// them (64 elements per block, its waves sharing the others in 64-element
// chunks, lane by lane through a scalar register; hundreds in the logs seen),
// into vkey (case) and vkey2 (count).  More: one block, stable byte passes
// between (vkey, vkey2) and (vidx, vidx2); there are at most n / 255.  99M events
// in cases of two, 190,000 such variants: 1.6 ms of a 5.9 ms call (9.3 ms where
// all cases were sorted by hash, then the variants by count).
constexpr int kTopThreads = 1024;
constexpr int64_t kTopPairs = 16384;
__global__ __launch_bounds__(kTopThreads) void k_var_top(VarWs w) {
    __shared__ uint32_t cnt[kTopThreads / kWave * 256];
    __shared__ uint32_t base[256];
    __shared__ uint32_t tmp[kTopThreads / kWave + 1];
    const int64_t M = w.scal[2];
    if (M <= kTopPairs) {
        __shared__ uint32_t place[kWave];
        if ((int64_t)blockIdx.x * kWave >= M) return;
        if (threadIdx.x < kWave) place[threadIdx.x] = 0;
        __syncthreads();
        const int64_t i = (int64_t)blockIdx.x * kWave + lane();
        const uint2 me = i < M ? w.vcr[i] : make_uint2(0, 0);
        uint32_t before = 0;
        for (int64_t ch = threadIdx.x / kWave; ch * kWave < M; ch += kTopThreads / kWave) {   // wave-uniform
            const int64_t j0 = ch * kWave;
            const uint32_t o = j0 + lane() < M ? w.vcr[j0 + lane()].x : 0u;   // 0: before nobody
            // an equal count of an earlier element comes first: in earlier chunks
            // all of them do, in later ones none, in this one the lower lanes
            const uint32_t lim = ch < (int64_t)blockIdx.x ? me.x : me.x + 1u;
#pragma unroll 16
            for (int j = 0; j < kWave; ++j) {
                const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)o, j);
                before += v >= lim ? 1u : 0u;
                if (ch == (int64_t)blockIdx.x) before += (v == me.x && j < lane()) ? 1u : 0u;
            }
        }
        atomicAdd(&place[lane()], before);
        __syncthreads();
        if (threadIdx.x < kWave && i < M) {
            w.vkey[place[threadIdx.x]] = me.y;
            w.vkey2[place[threadIdx.x]] = me.x;
        }
        return;
    }
    if (blockIdx.x != 0) return;
    const int wv = threadIdx.x / kWave;
    uint32_t *ck = w.vidx, *cv = w.vidx2, *ok = w.vkey, *ov = w.vkey2;   // (case, count), 4 passes: ends in (vkey, vkey2)
    for (int64_t i = threadIdx.x; i < M; i += kTopThreads) {
        ok[i] = w.vcr[i].y;
        ov[i] = w.vcr[i].x;
    }
    for (int shift = 0; shift < 32; shift += 8) {
        uint32_t* t = ck; ck = ok; ok = t;
        t = cv; cv = ov; ov = t;
        __threadfence_block();
        __syncthreads();
        if (threadIdx.x < 256) base[threadIdx.x] = 0;
        __syncthreads();
        for (int64_t i = threadIdx.x; i < M; i += kTopThreads) atomicAdd(&base[(~cv[i] >> shift) & 255u], 1u);
        __syncthreads();
        uint32_t all;
        const uint32_t v = threadIdx.x < 256 ? base[threadIdx.x] : 0u;
        const uint32_t ex = block_excl_sum<kTopThreads>(v, tmp, &all);
        if (threadIdx.x < 256) base[threadIdx.x] = ex;
        for (int64_t t0 = 0; t0 < M; t0 += kTopThreads) {
            for (int i = threadIdx.x; i < kTopThreads / kWave * 256; i += kTopThreads) cnt[i] = 0;
            __syncthreads();
            const int64_t i = t0 + threadIdx.x;
            const bool valid = i < M;
            const uint32_t c = valid ? ck[i] : 0u, k = valid ? cv[i] : 0u;
            const uint32_t d = (~k >> shift) & 255u;
            const uint64_t peers = match_digit<8>(d, __ballot(valid));
            const uint32_t below = __popcll(peers & lanes_below());
            if (valid && below == 0) cnt[wv * 256 + d] = __popcll(peers);
            __syncthreads();
            if (threadIdx.x < 256) {
                uint32_t run = base[threadIdx.x];
                for (int ww = 0; ww < kTopThreads / kWave; ++ww) {
                    const uint32_t x = cnt[ww * 256 + threadIdx.x];
                    cnt[ww * 256 + threadIdx.x] = run;
                    run += x;
                }
                base[threadIdx.x] = run;
            }
            __syncthreads();
            if (valid) {
                const uint32_t g = cnt[wv * 256 + d] + below;
                ok[g] = c;
                ov[g] = k;
            }
            __syncthreads();
        }
    }
}

// The final order in ranges of variants, one per block (k_var_emit walks the
// same ranges): counts, representatives, lengths; the range's total length in
// part64, the variant of each representative in fid (by case).
constexpr int kEmitBlk = 512;
__device__ __forceinline__ int64_t emit_chunk(int64_t V) { return (V + gridDim.x - 1) / gridDim.x; }

__global__ __launch_bounds__(kEmitBlk) void k_var_ids(VarWs w, const int64_t* __restrict__ case_off,
                                                      const int32_t* __restrict__ case_code, VarOutDev out) {
    __shared__ int64_t red[kEmitBlk / kWave];
    const int64_t V = w.scal[1], M = w.scal[2], chunk = emit_chunk(V);
    const int64_t b0 = blockIdx.x * chunk, b1 = b0 + chunk < V ? b0 + chunk : V;
    int64_t sum = 0;
    for (int64_t k = b0 + threadIdx.x; k < b1; k += kEmitBlk) {
        const uint2 cr = k < M ? make_uint2(w.vkey2[k], w.vkey[k]) : w.vcr[k];
        const uint32_t r = cr.y;
        const uint32_t L = (uint32_t)(case_off[r + 1] - case_off[r]);
        w.fid[r] = (uint32_t)k;
        w.sstart[k] = r;
        out.var_count[k] = cr.x;
        out.var_rep[k] = case_code[r];
        out.var_len[k] = (int32_t)L;
        w.lens[k] = L;
        sum += L;
    }
    sum = wave_sum(sum);
    if (lane() == 0) red[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int k = 0; k < kEmitBlk / kWave; ++k) t += red[k];
        w.part64[blockIdx.x] = t;
    }
}

// Sequences in final order: a block takes its range in steps of 512 variants
// (offsets from the ranges' totals and a block scan), a wave 64 consecutive
// variants of a step, copying their representatives' activities, writes
// coalesced over the output range.  Bound by the vector instructions that find
// each position's variant: with one search per four positions 0.255 ms for the
// 99M activities of 5M cases, 0.306 with one per position.
__global__ __launch_bounds__(kEmitBlk) void k_var_emit(const int32_t* __restrict__ act_s,
                                                       const int64_t* __restrict__ case_off, VarWs w,
                                                       const int32_t* status_in, VarOutDev out) {
    __shared__ int64_t tmp[kEmitBlk / kWave + 1];
    __shared__ uint32_t sdst[kEmitBlk / kWave][kWave + 1];  // a wave's variants: output start after the wave's,
    __shared__ int32_t ssrc[kEmitBlk / kWave][kWave];       // source position minus output position
    const int wl = threadIdx.x / kWave;
    const int64_t C = w.scal[0];
    const int64_t V = w.scal[1], chunk = emit_chunk(V);
    const int64_t b0 = blockIdx.x * chunk, b1 = b0 + chunk < V ? b0 + chunk : V;
    int64_t run;
    {
        int64_t before = 0;
        for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += kEmitBlk) before += w.part64[i];
        block_excl_sum<kEmitBlk>(before, tmp, &run);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        out.var_off[V] = run + w.part64[blockIdx.x];
        *out.n_variants = V;
        *out.status = status_in ? *status_in : 0;
    }
    for (int64_t s0 = b0; s0 < b1; s0 += kEmitBlk) {   // block-uniform
        const int64_t k0 = s0 + threadIdx.x / kWave * kWave;
        const int64_t k = k0 + lane();
        const bool has = k < b1;
        int64_t src = 0, len = 0;
        if (has) {
            src = case_off[w.sstart[k]];
            len = w.lens[k];
        }
        int64_t total;
        const int64_t dst = run + block_excl_sum<kEmitBlk>(len, tmp, &total);
        run += total;
        if (has) out.var_off[k] = dst;
        if (k0 >= b1) continue;   // wave-uniform; the block scan above is every wave's
        const int last = (b1 - 1 - k0) < (kWave - 1) ? (int)(b1 - 1 - k0) : (kWave - 1);
        const int64_t base = __shfl(dst, 0);
        const int64_t end = __shfl(dst + len, last);
        // four consecutive output positions per lane, from an aligned one on: one
        // search per four, the variant's end tells when to step on.  Offsets from
        // that position fit 32 bits (a log has fewer than 2^31 events).
        const uint32_t skip = (uint32_t)((reinterpret_cast<uintptr_t>(out.var_acts + base) / 4) & 3);
        int32_t* to = out.var_acts + base - skip;
        const int32_t* from = act_s + base - skip;
        const uint32_t top = (uint32_t)(end - base) + skip;
        const uint32_t first = has ? (uint32_t)(dst - base) + skip : UINT32_MAX;
        sdst[wl][lane()] = first;
        ssrc[wl][lane()] = has ? (int32_t)(src - dst) : 0;
        if (lane() == 0) sdst[wl][kWave] = UINT32_MAX;
        wave_sync();
        for (uint32_t q0 = 0; q0 < top; q0 += 4 * kWave) {   // wave-uniform
            const uint32_t q = q0 + 4 * lane();
            int m = seg_of32(first, q < skip ? skip : q);
            uint32_t nxt = sdst[wl][m + 1];
            int32_t sh = ssrc[wl][m];
            int32_t av[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t p = q + j;
                if (p >= nxt) {   // variants are non-empty: one step at a time
                    ++m;
                    nxt = sdst[wl][m + 1];
                    sh = ssrc[wl][m];
                }
                av[j] = p >= skip && p < top ? from[(int64_t)p + sh] : 0;
            }
            if (q >= skip && q + 3 < top) {
                *reinterpret_cast<int4*>(to + q) = make_int4(av[0], av[1], av[2], av[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (q + j >= skip && q + j < top) to[q + j] = av[j];
            }
        }
        wave_sync();
    }
    if (out.case_variant) {
        for (int64_t c = (int64_t)blockIdx.x * kEmitBlk + threadIdx.x; c < C; c += (int64_t)gridDim.x * kEmitBlk)
            out.case_variant[c] = (int32_t)w.fid[w.idx[c]];
    }
}

}  // namespace

hipError_t launch_variants(const int32_t* act_s, const int64_t* case_off, const int32_t* case_code,
                           const int64_t* n_cases, const int32_t* status_in, int64_t n, VarWs w,
                           VarOutDev out, uint32_t debug_hash_bits, hipStream_t s) {
    const uint64_t mask = (debug_hash_bits == 0 || debug_hash_bits >= 64)
                              ? 0ull
                              : ((uint64_t(1) << debug_hash_bits) - 1);
    const int64_t nb = dev::tiles(n);
    // the case count is on the device; n bounds it, and with it every grid
    const auto grid = [](int64_t want, int64_t most) { return (unsigned)(want < 1 ? 1 : (want < most ? want : most)); };
    {
        ProfScope p(P_VAR_HASH, s);
        k_var_clear<<<grid((n + kBlk - 1) / kBlk, kGrid), kBlk, 0, s>>>(w, n_cases);
        k_var_group<<<grid((n + kBlk - 1) / kBlk, kGroupGrid), kBlk, 0, s>>>(act_s, case_off, w, mask, n);
    }
    {
        ProfScope p(P_VAR_ORDER, s);
        k_var_reps<<<dev::grid_for(nb), dev::kB, 0, s>>>(w, nb);
        if (nb > kFewTiles) dev::k_hist_scan<<<256, 256, 0, s>>>(w.hist, &w.scal[0], nb, w.rowsum);
        k_var_order<<<dev::grid_for(nb), dev::kB, 0, s>>>(w, nb);
        // at most n / 255 variants have 255 cases
        k_var_top<<<grid((n / 255 + kWave - 1) / kWave, kTopPairs / kWave), kTopThreads, 0, s>>>(w);
    }
    ProfScope p(P_VAR_EMIT, s);
    const unsigned ge = grid((n + kEmitBlk - 1) / kEmitBlk, dev::kScanGrid);
    k_var_ids<<<ge, kEmitBlk, 0, s>>>(w, case_off, case_code, out);
    k_var_emit<<<ge, kEmitBlk, 0, s>>>(act_s, case_off, w, status_in, out);
    return hipGetLastError();
}

}  // namespace pm4g
