// Stable LSD radix passes over (key u32, ts i64, act u32) elements, digits of 8
// bits (9 or 10 where that saves a pass), reduce-then-scan:
//   k_radix_hist     per-tile digit histograms, digit-major [digits][tiles]
//   k_radix_scan     exclusive scan of each digit row, row totals (up to
//                    kRadixFewTiles tiles: by each scatter block itself; a
//                    single tile needs neither histogram nor scan)
//   k_radix_scatter  wave64 ballot ranking (stable: wave, item, lane order),
//                    LDS staging in digit order, coalesced-run writes; tiles
//                    laid out XCD-contiguously over the grid
// The first pass reads the raw log columns directly (case id biased by the
// case minimum), so the caller's arrays are never copied.
//
// This is the grouping step of Sec. 3's first formatting step: events of a
// case become adjacent while keeping their row order (stability); the
// per-case timestamp order is applied afterwards in LDS (segsort.hip).
// Packed layout (PACKED): when the case bits and the activity bits fit in 32,
// the activity rides in the key above the case bits (key_mask selects the
// case bits) and no activity column moves: 12 bytes per element.
// Bytes per event per pass: 4 (hist) + 16 read + 16 write (12 + 12 packed).
// Row order (ROW): when the caller asks for the permutation, each element
// also carries its original row (the first pass takes it from its position),
// 4 more bytes read and written per element; otherwise nothing moves for it.
#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"

namespace pm4g {

constexpr int kRB = 512;               // threads per block
constexpr int kRI = kRadixTile / kRB;  // items per thread (8)
constexpr int kRW = kRB / kWave;       // waves per block (8)

template <int SRC, int BITS>
__device__ __forceinline__ uint32_t digit_of(uint32_t key, int64_t ts, int shift, int64_t ts_min,
                                             uint32_t key_mask) {
    constexpr uint32_t kMask = (1u << BITS) - 1u;
    if (SRC == 0) return ((key & key_mask) >> shift) & kMask;
    return (uint32_t)(((uint64_t)ts - (uint64_t)ts_min) >> shift) & kMask;
}

// The first pass reads the raw columns: key = case - case_min (| act << act_shift when packed).
template <bool FIRST, bool PACKED>
__device__ __forceinline__ uint32_t load_key(const SortBufs& in, int64_t i, int32_t case_min, int act_shift) {
    if (FIRST) {
        uint32_t k = (uint32_t)reinterpret_cast<const int32_t*>(in.key)[i] - (uint32_t)case_min;
        if (PACKED) k |= (uint32_t)reinterpret_cast<const int32_t*>(in.act)[i] << act_shift;
        return k;
    }
    return in.key[i];
}

template <int SRC, bool FIRST, int BITS>
__global__ __launch_bounds__(kRB) void k_radix_hist(SortBufs in, int64_t n, int shift,
                                                    const RangeInfo* info, uint32_t* hist,
                                                    int64_t nb, uint32_t key_mask) {
    constexpr int D = 1 << BITS;
    __shared__ uint32_t h[D];
    for (int k = threadIdx.x; k < D; k += kRB) h[k] = 0;
    __syncthreads();
    const int32_t case_min = info->case_min;
    const int64_t ts_min = info->ts_min;
    const int64_t base = (int64_t)blockIdx.x * kRadixTile;
    const bool vec = SRC == 0 && base + kRadixTile <= n && (reinterpret_cast<uintptr_t>(in.key) & 15) == 0;
    if (vec) {
        // full tile: 16-byte loads of four keys
        const uint4* k4 = reinterpret_cast<const uint4*>(in.key + base);
#pragma unroll
        for (int q = 0; q < kRI / 4; ++q) {
            const uint4 v = k4[q * kRB + threadIdx.x];
            const uint32_t bias = FIRST ? (uint32_t)case_min : 0u;
            atomicAdd(&h[digit_of<0, BITS>(v.x - bias, 0, shift, 0, key_mask)], 1u);
            atomicAdd(&h[digit_of<0, BITS>(v.y - bias, 0, shift, 0, key_mask)], 1u);
            atomicAdd(&h[digit_of<0, BITS>(v.z - bias, 0, shift, 0, key_mask)], 1u);
            atomicAdd(&h[digit_of<0, BITS>(v.w - bias, 0, shift, 0, key_mask)], 1u);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kRI; ++k) {
            const int64_t i = base + k * kRB + threadIdx.x;
            if (i < n) {
                uint32_t d;
                if (SRC == 0) d = digit_of<0, BITS>(load_key<FIRST, false>(in, i, case_min, 0), 0, shift, 0, key_mask);
                else d = digit_of<1, BITS>(0, in.ts[i], shift, ts_min, key_mask);
                atomicAdd(&h[d], 1u);
            }
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < D; k += kRB) hist[(int64_t)k * nb + blockIdx.x] = h[k];
}

// One block per digit: exclusive scan of hist[d][0..nb) in place, row total.
__global__ __launch_bounds__(256) void k_radix_scan(uint32_t* hist, int64_t nb, uint32_t* rowsum) {
    __shared__ uint32_t tmp[256 / kWave + 1];
    uint32_t* row = hist + (int64_t)blockIdx.x * nb;
    uint32_t run = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += 256 * 4) {
        uint32_t v[4];
        uint32_t s = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = c0 + threadIdx.x * 4 + q;
            v[q] = i < nb ? row[i] : 0u;
            s += v[q];
        }
        uint32_t total;
        uint32_t ex = block_excl_sum<256>(s, tmp, &total);
        uint32_t r = run + ex;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = c0 + threadIdx.x * 4 + q;
            if (i < nb) row[i] = r;
            r += v[q];
        }
        run += total;
    }
    if (threadIdx.x == 0) rowsum[blockIdx.x] = run;
}

// First case pass with the range scan's histograms of the raw low byte u:
// digit d of case - case_min is u = (d + case_min) & 255, so row d is the
// scan of raw row (d + case_min) & 255.
__global__ __launch_bounds__(256) void k_radix_scan_rot(const uint32_t* hist_raw, uint32_t* hist, int64_t nb,
                                                        uint32_t* rowsum, const RangeInfo* info) {
    __shared__ uint32_t tmp[256 / kWave + 1];
    const uint32_t u = (blockIdx.x + (uint32_t)info->case_min) & 255u;
    const uint32_t* in = hist_raw + (int64_t)u * nb;
    uint32_t* row = hist + (int64_t)blockIdx.x * nb;
    uint32_t run = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += 256 * 4) {
        uint32_t v[4];
        uint32_t s = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = c0 + threadIdx.x * 4 + q;
            v[q] = i < nb ? in[i] : 0u;
            s += v[q];
        }
        uint32_t total;
        uint32_t r = run + block_excl_sum<256>(s, tmp, &total);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = c0 + threadIdx.x * 4 + q;
            if (i < nb) row[i] = r;
            r += v[q];
        }
        run += total;
    }
    if (threadIdx.x == 0) rowsum[blockIdx.x] = run;
}

// Where a scatter block finds its tile's place in each digit: in the scanned
// rows and the row totals; in the rows as counted (few tiles: each block adds
// up the entries before its own and all, 64 words of a digit from the L2
// against a launch of 4.5 us), turned by the case minimum when they are the
// range scan's raw rows; or nowhere (the only tile starts every digit).
enum RadixRows { ROWS_SCANNED, ROWS_COUNTED, ROWS_RAW, ROWS_NONE };

// What bounds a pass: the loads and the scattered stores (12 bytes read and
// written per packed element; at 8 bits a tile's runs average 16 elements).
// Wider digits make more and shorter runs and take more ranking steps, so
// they pay where they save a pass, 10 bits only among few tiles: two passes of
// 10 bits over 10M events took 231 us where three of 8 take 215 (histograms of
// 1024 rows, 30 us each).  Formatting 1.2M events of 17 bits went from 132 to 105
// us, 25M of 18 bits from 950 to 868, and without histograms or scans 4000 events
// of 9 bits from 73 to 54 us, 200,000 of 15 bits from 80 to 73.
template <int SRC, bool FIRST, bool PACKED, bool ROW, int BITS>
__global__ __launch_bounds__(kRB) void k_radix_scatter(SortBufs in, SortBufs out, int64_t n, int shift,
                                                       const RangeInfo* info, const uint32_t* hist,
                                                       const uint32_t* rowsum, int64_t nb,
                                                       uint32_t key_mask, int act_shift, RadixRows rows) {
    constexpr int D = 1 << BITS;
    constexpr int kDPer = (D + kRB - 1) / kRB;   // digits per thread
    __shared__ alignas(4) uint16_t cnt[kRW * D];   // per-wave running digit counts (a tile has 4096 elements)
    __shared__ uint32_t tstart[D];            // tile-local start of each digit
    __shared__ int64_t gshift[D];             // global position - tile position
    __shared__ uint32_t skey[kRadixTile];
    __shared__ int64_t sts[kRadixTile];
    __shared__ uint32_t sact[PACKED ? 1 : kRadixTile];
    __shared__ uint32_t srow[ROW ? kRadixTile : 1];
    __shared__ uint32_t tmp[kRB / kWave + 1];

    const int32_t case_min = info->case_min;
    const int64_t ts_min = info->ts_min;
    const int w = threadIdx.x / kWave;
    // one tile per block, XCD-contiguous: the runs of neighbouring tiles meet
    // in the same L2, where their shared boundary lines are completed
    const int64_t tile = xcd_split(nb).first;
    const int64_t tile0 = tile * kRadixTile;
    const int64_t wbase = tile0 + (int64_t)w * (kWave * kRI);

    for (int i = threadIdx.x; i < kRW * D / 2; i += kRB) reinterpret_cast<uint32_t*>(cnt)[i] = 0;

    uint32_t key[kRI], act[kRI], dg[kRI], rk[kRI], rw[kRI];
    int64_t tv[kRI];
    if constexpr (FIRST) {
        // all loads of the tile first: forming each key from its two raw
        // columns right after their loads (as the compiler schedules it
        // otherwise) made every item's loads wait for the previous item's
        uint32_t rc[kRI], ra[kRI];
#pragma unroll
        for (int k = 0; k < kRI; ++k) {
            const int64_t i = wbase + k * kWave + lane();
            if (i < n) {
                rc[k] = reinterpret_cast<const uint32_t*>(in.key)[i];
                ra[k] = in.act[i];
                tv[k] = in.ts[i];
            } else {
                rc[k] = (uint32_t)case_min;
                ra[k] = 0;
                tv[k] = ts_min;
            }
            rw[k] = (uint32_t)i;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < kRI; ++k) {
            key[k] = rc[k] - (uint32_t)case_min;   // 0 past the end
            if (PACKED) key[k] |= ra[k] << act_shift;
            act[k] = PACKED ? 0u : ra[k];
            dg[k] = digit_of<SRC, BITS>(key[k], tv[k], shift, ts_min, key_mask);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kRI; ++k) {
            const int64_t i = wbase + k * kWave + lane();
            if (i < n) {
                key[k] = load_key<FIRST, PACKED>(in, i, case_min, act_shift);
                tv[k] = in.ts[i];
                act[k] = PACKED ? 0u : in.act[i];
                rw[k] = ROW ? in.row[i] : 0u;
            } else {
                key[k] = 0;
                tv[k] = ts_min;
                act[k] = 0;
                rw[k] = 0;
            }
            dg[k] = digit_of<SRC, BITS>(key[k], tv[k], shift, ts_min, key_mask);
        }
    }
    __syncthreads();

    // Stable ranks within the wave's contiguous chunk, in (item, lane) order.
#pragma unroll
    for (int k = 0; k < kRI; ++k) {
        const int64_t i = wbase + k * kWave + lane();
        const bool valid = i < n;
        const uint64_t active = __ballot(valid);
        const uint64_t peers = match_digit<BITS>(dg[k], active);
        const uint32_t below = __popcll(peers & lanes_below());
        uint32_t c = 0;
        if (valid) c = cnt[w * D + dg[k]];
        rk[k] = c + below;
        if (valid && below == 0) cnt[w * D + dg[k]] = (uint16_t)(c + __popcll(peers));
    }
    __syncthreads();

    // Per digit: exclusive offsets of the waves, the tile's digit totals.
    uint32_t tot[kDPer], own[kDPer], rs[kDPer];   // tile's elements, elements of tiles before, of all tiles
    uint32_t tsum = 0, rsum = 0;
#pragma unroll
    for (int q = 0; q < kDPer; ++q) {
        const int d = (int)threadIdx.x * kDPer + q;
        tot[q] = own[q] = rs[q] = 0;
        if (d < D) {
            uint32_t run = 0;
            for (int ww = 0; ww < kRW; ++ww) {
                const uint32_t x = cnt[ww * D + d];
                cnt[ww * D + d] = (uint16_t)run;
                run += x;
            }
            tot[q] = rs[q] = run;
            if (rows == ROWS_SCANNED) {
                own[q] = hist[(int64_t)d * nb + tile];
                rs[q] = rowsum[d];
            } else if (rows != ROWS_NONE) {
                const uint32_t u = rows == ROWS_RAW ? ((uint32_t)d + (uint32_t)case_min) & 255u : (uint32_t)d;
                const uint32_t* row = hist + (int64_t)u * nb;
                uint32_t before = 0, all = 0;
#pragma unroll 8
                for (int64_t k = 0; k < nb; ++k) {
                    const uint32_t x = row[k];
                    all += x;
                    before += k < tile ? x : 0u;
                }
                own[q] = before;
                rs[q] = all;
            }
        }
        tsum += tot[q];
        rsum += rs[q];
    }
    uint32_t all;
    uint32_t ts_excl = block_excl_sum<kRB>(tsum, tmp, &all);
    uint32_t digit_base = block_excl_sum<kRB>(rsum, tmp, &all);
#pragma unroll
    for (int q = 0; q < kDPer; ++q) {
        const int d = (int)threadIdx.x * kDPer + q;
        if (d < D) {
            tstart[d] = ts_excl;
            gshift[d] = (int64_t)digit_base + (int64_t)own[q] - (int64_t)ts_excl;
        }
        ts_excl += tot[q];
        digit_base += rs[q];
    }
    __syncthreads();

#pragma unroll
    for (int k = 0; k < kRI; ++k) {
        const int64_t i = wbase + k * kWave + lane();
        if (i < n) {
            const uint32_t pos = tstart[dg[k]] + cnt[w * D + dg[k]] + rk[k];
            skey[pos] = key[k];
            sts[pos] = tv[k];
            if (!PACKED) sact[pos] = act[k];
            if (ROW) srow[pos] = rw[k];
        }
    }
    __syncthreads();

    const int64_t valid_count = (n - tile0) < kRadixTile ? (n - tile0) : kRadixTile;
    for (int i = threadIdx.x; i < valid_count; i += kRB) {
        const uint32_t k = skey[i];
        const int64_t t = sts[i];
        const uint32_t d = digit_of<SRC, BITS>(k, t, shift, ts_min, key_mask);
        const int64_t g = gshift[d] + i;
        out.key[g] = k;
        out.ts[g] = t;
        if (!PACKED) out.act[g] = sact[i];
        if (ROW) out.row[g] = srow[i];
    }
}

template <int SRC, bool FIRST, bool PACKED, bool ROW, int BITS>
static void run_pass(SortBufs in, SortBufs out, int64_t n, int shift, const RangeInfo* info,
                     uint32_t* hist, uint32_t* rowsum, uint32_t key_mask, int act_shift,
                     const uint32_t* hist_raw, hipStream_t s) {
    const int64_t nb = radix_blocks(n);
    RadixRows rows = nb == 1 ? ROWS_NONE : nb > kRadixFewTiles ? ROWS_SCANNED : hist_raw ? ROWS_RAW : ROWS_COUNTED;
    if (rows == ROWS_SCANNED && hist_raw) {
        ProfScope p(P_RADIX_SCAN, s);
        k_radix_scan_rot<<<256, 256, 0, s>>>(hist_raw, hist, nb, rowsum, info);
    } else if (rows == ROWS_SCANNED || rows == ROWS_COUNTED) {
        {
            ProfScope p(P_RADIX_HIST, s);
            k_radix_hist<SRC, FIRST, BITS><<<(unsigned)nb, kRB, 0, s>>>(in, n, shift, info, hist, nb, key_mask);
        }
        if (rows == ROWS_SCANNED) {
            ProfScope p(P_RADIX_SCAN, s);
            k_radix_scan<<<1 << BITS, 256, 0, s>>>(hist, nb, rowsum);
        }
    }
    ProfScope p(P_RADIX_SCATTER, s);
    k_radix_scatter<SRC, FIRST, PACKED, ROW, BITS>
        <<<(unsigned)nb, kRB, 0, s>>>(in, out, n, shift, info, rows == ROWS_RAW ? hist_raw : hist, rowsum, nb, key_mask,
                                      act_shift, rows);
}

// Passes over `bits` case bits: as few as the widest digits need where that is
// fewer than 8-bit ones need, the first as narrow as the others allow (8 bits
// take the range scan's histograms); 8-bit digits otherwise.
int radix_plan(int bits, int64_t n, int width[4]) {
    const int widest = radix_blocks(n) <= kRadixFewTiles ? kRadixMaxBits : kRadixManyBits;
    int left = bits > 0 ? bits : 1;   // a single case: one pass still biases the keys
    const int p8 = (left + 7) / 8, pw = (left + widest - 1) / widest;
    const int passes = pw < p8 ? pw : p8;
    for (int p = 0; p < passes; ++p) {
        const int rest = left - widest * (passes - 1 - p);
        width[p] = pw < p8 && rest > 8 ? rest : 8;
        left -= width[p];
    }
    return passes;
}

hipError_t launch_radix_pass(SortBufs in, SortBufs out, int64_t n, int digit_src, int shift, int width,
                             bool first, const RangeInfo* info, uint32_t* hist, uint32_t* rowsum,
                             int act_shift, const uint32_t* hist_raw, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const bool packed = act_shift > 0;
    const uint32_t key_mask = packed ? ((act_shift >= 32) ? 0xFFFFFFFFu : ((1u << act_shift) - 1u)) : 0xFFFFFFFFu;
    // the raw-byte histograms describe the first case pass only
    if (!(digit_src == 0 && first && shift == 0 && width == 8)) hist_raw = nullptr;
    // the row order is carried iff the output has a row array
#define PM4G_PASS(SRC, FIRST, PACKED, BITS)                                                                  \
    do {                                                                                                    \
        if (out.row)                                                                                        \
            run_pass<SRC, FIRST, PACKED, true, BITS>(in, out, n, shift, info, hist, rowsum, key_mask,       \
                                                     act_shift, hist_raw, s);                               \
        else                                                                                                \
            run_pass<SRC, FIRST, PACKED, false, BITS>(in, out, n, shift, info, hist, rowsum, key_mask,      \
                                                      act_shift, hist_raw, s);                              \
    } while (0)
#define PM4G_CASE_PASS(BITS)                                                                                 \
    do {                                                                                                    \
        if (first) { if (packed) PM4G_PASS(0, true, true, BITS); else PM4G_PASS(0, true, false, BITS); }    \
        else { if (packed) PM4G_PASS(0, false, true, BITS); else PM4G_PASS(0, false, false, BITS); }        \
    } while (0)
    if (digit_src == 0) {
        if (width == 8) PM4G_CASE_PASS(8);
        else if (width == 9) PM4G_CASE_PASS(9);
        else PM4G_CASE_PASS(10);
    } else {
        if (first) { if (packed) PM4G_PASS(1, true, true, 8); else PM4G_PASS(1, true, false, 8); }
        else { if (packed) PM4G_PASS(1, false, true, 8); else PM4G_PASS(1, false, false, 8); }
    }
#undef PM4G_CASE_PASS
#undef PM4G_PASS
    return hipGetLastError();
}

}  // namespace pm4g
