// Range scan of a raw log: case-id and timestamp extremes (they fix the
// radix key widths), activity validation, and the order check for a log
// that claims to be presorted (Sec. 3: (case, timestamp, row) order).
//
// Streaming pass, HBM-bound: 8 bytes/event (case, activity), 16 with the
// timestamp.  Block reductions into per-block partials, folded by one block
// (no same-address atomics: across the 8 XCDs they serialise).
#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"
#include "../../include/pm4g.h"

namespace pm4g {

// A log that claims to be ordered: activities in range, and every event not
// before its predecessor.  Four events per thread and step (16-byte loads where
// the columns allow them), the event before them from its own cache lines.
__global__ __launch_bounds__(256) void k_range_scan(const int32_t* __restrict__ case_id,
                                                    const int32_t* __restrict__ act,
                                                    const int64_t* __restrict__ ts, int64_t n,
                                                    int32_t A, RangePart* part) {
    bool bad = false, unsorted = false;
    const bool aligned = ((reinterpret_cast<uintptr_t>(case_id) | reinterpret_cast<uintptr_t>(act) |
                           reinterpret_cast<uintptr_t>(ts)) & 15) == 0;
    const int64_t stride = 4 * (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x); i < n; i += stride) {
        const int32_t cp = i > 0 ? case_id[i - 1] : INT32_MIN;
        const int64_t tp = i > 0 ? ts[i - 1] : INT64_MIN;
        if (aligned && i + 3 < n) {
            const int4 c = *reinterpret_cast<const int4*>(case_id + i);
            const int4 a = *reinterpret_cast<const int4*>(act + i);
            const longlong2 t0 = *reinterpret_cast<const longlong2*>(ts + i);
            const longlong2 t1 = *reinterpret_cast<const longlong2*>(ts + i + 2);
            bad |= (uint32_t)a.x >= (uint32_t)A || (uint32_t)a.y >= (uint32_t)A || (uint32_t)a.z >= (uint32_t)A ||
                   (uint32_t)a.w >= (uint32_t)A;
            unsorted |= cp > c.x || (cp == c.x && tp > t0.x);
            unsorted |= c.x > c.y || (c.x == c.y && t0.x > t0.y);
            unsorted |= c.y > c.z || (c.y == c.z && t0.y > t1.x);
            unsorted |= c.z > c.w || (c.z == c.w && t1.x > t1.y);
        } else {
            int32_t c0 = cp;
            int64_t t0 = tp;
            for (int64_t k = i; k < n && k < i + 4; ++k) {
                const int32_t c = case_id[k];
                const int64_t t = ts[k];
                bad |= (uint32_t)act[k] >= (uint32_t)A;
                unsorted |= c0 > c || (c0 == c && t0 > t);
                c0 = c;
                t0 = t;
            }
        }
    }
    const int any_bad = __syncthreads_or(bad);
    const int any_unsorted = __syncthreads_or(unsorted);
    if (threadIdx.x == 0)
        part[blockIdx.x] = RangePart{INT32_MAX, INT32_MIN, any_bad ? 1 : 0, any_unsorted ? 1 : 0, INT64_MAX, INT64_MIN};
}

// Folds a block's partials (one per thread) into the RangeInfo and starts the
// call's status word.
template <int THREADS>
__device__ __forceinline__ void store_range(RangePart r, RangePart* red, RangeInfo* info, int32_t* status,
                                            const BackDst& back) {
    r.cmin = wave_min(r.cmin);
    r.cmax = wave_max(r.cmax);
    r.tmin = wave_min(r.tmin);
    r.tmax = wave_max(r.tmax);
    r.bad = __ballot(r.bad != 0) != 0;
    r.unsorted = __ballot(r.unsorted != 0) != 0;
    if (lane() == 0) red[threadIdx.x / kWave] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < THREADS / kWave; ++k) {
            const RangePart& o = red[k];
            r.cmin = o.cmin < r.cmin ? o.cmin : r.cmin;
            r.cmax = o.cmax > r.cmax ? o.cmax : r.cmax;
            r.tmin = o.tmin < r.tmin ? o.tmin : r.tmin;
            r.tmax = o.tmax > r.tmax ? o.tmax : r.tmax;
            r.bad |= o.bad;
            r.unsorted |= o.unsorted;
        }
        info->case_min = r.cmin;
        info->case_max = r.cmax;
        info->ts_min = r.tmin;
        info->ts_max = r.tmax;
        info->status = r.bad ? PM4G_E_RANGE : (r.unsorted ? PM4G_E_NOT_SORTED : 0);
        info->long_case = 0;
        *status = info->status;
        publish(back, info, kInfoWords);
    }
}

// The formatting step's range scan over radix tiles (kRadixTile events per
// block, no timestamps): besides the partials, each tile's histogram of the
// low 8 bits of the raw case id.  The first radix pass digit is the low byte
// of case - case_min, a rotation of that byte by case_min, so this histogram
// replaces the first pass's histogram kernel (k_radix_scan_rot rotates it).
// WHOLE: one block takes all tiles and stores the result itself; with few
// tiles they take less than the folding launch (kRangeWhole).
constexpr int64_t kRangeWhole = 4;
template <bool WHOLE>
__global__ __launch_bounds__(kRangeTileThreads) void k_range_tiles(const int32_t* __restrict__ case_id,
                                                                   const int32_t* __restrict__ act, int64_t n,
                                                                   int32_t A, RangePart* part,
                                                                   uint32_t* hist_raw, int64_t nb, RangeInfo* info,
                                                                   int32_t* status, BackDst back) {
    __shared__ uint32_t h[256];
    __shared__ RangePart red[kRangeTileThreads / kWave];
    constexpr int kT = kRangeTileThreads;
    int32_t cmin = INT32_MAX, cmax = INT32_MIN;
    bool bad = false;
    auto visit = [&](int32_t c, int32_t a) {
        bad |= (uint32_t)a >= (uint32_t)A;
        cmin = c < cmin ? c : cmin;
        cmax = c > cmax ? c : cmax;
        atomicAdd(&h[(uint32_t)c & 255u], 1u);
    };
    for (int64_t t = WHOLE ? 0 : blockIdx.x; t < (WHOLE ? nb : (int64_t)blockIdx.x + 1); ++t) {
        if (threadIdx.x < 256) h[threadIdx.x] = 0;
        __syncthreads();
        const int64_t base = t * kRadixTile;
        const bool vec = base + kRadixTile <= n &&
                         ((reinterpret_cast<uintptr_t>(case_id) | reinterpret_cast<uintptr_t>(act)) & 15) == 0;
        if (vec) {
            const int4* c4 = reinterpret_cast<const int4*>(case_id + base);
            const int4* a4 = reinterpret_cast<const int4*>(act + base);
#pragma unroll
            for (int q = 0; q < kRadixTile / (4 * kT); ++q) {
                const int4 c = c4[q * kT + threadIdx.x];
                const int4 a = a4[q * kT + threadIdx.x];
                visit(c.x, a.x);
                visit(c.y, a.y);
                visit(c.z, a.z);
                visit(c.w, a.w);
            }
        } else {
            for (int64_t i = base + threadIdx.x; i < n && i < base + kRadixTile; i += kT) visit(case_id[i], act[i]);
        }
        __syncthreads();
        if (threadIdx.x < 256) hist_raw[(int64_t)threadIdx.x * nb + t] = h[threadIdx.x];
    }
    RangePart r{cmin, cmax, bad, 0, INT64_MAX, INT64_MIN};
    if (WHOLE) {
        store_range<kT>(r, red, info, status, back);
        return;
    }
    r.cmin = wave_min(cmin);
    r.cmax = wave_max(cmax);
    r.bad = __ballot(bad) != 0;
    if (lane() == 0) red[threadIdx.x / kWave] = r;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kT / kWave; ++k) {
            r.cmin = red[k].cmin < r.cmin ? red[k].cmin : r.cmin;
            r.cmax = red[k].cmax > r.cmax ? red[k].cmax : r.cmax;
            r.bad |= red[k].bad;
        }
        part[blockIdx.x] = r;
    }
}

// One block folds the per-block partials (none: an empty log).
__global__ __launch_bounds__(1024) void k_range_final(const RangePart* part, int nparts, RangeInfo* info,
                                                      int32_t* status, BackDst back) {
    __shared__ RangePart red[1024 / kWave];
    RangePart r{INT32_MAX, INT32_MIN, 0, 0, INT64_MAX, INT64_MIN};
    for (int k = threadIdx.x; k < nparts; k += 1024) {
        const RangePart o = part[k];
        r.cmin = o.cmin < r.cmin ? o.cmin : r.cmin;
        r.cmax = o.cmax > r.cmax ? o.cmax : r.cmax;
        r.tmin = o.tmin < r.tmin ? o.tmin : r.tmin;
        r.tmax = o.tmax > r.tmax ? o.tmax : r.tmax;
        r.bad |= o.bad;
        r.unsorted |= o.unsorted;
    }
    store_range<1024>(r, red, info, status, back);
}

__global__ __launch_bounds__(256) void k_ts_range(const int64_t* __restrict__ ts, int64_t n,
                                                  RangeInfo* info) {
    int64_t tmin = INT64_MAX, tmax = INT64_MIN;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const int64_t t = ts[i];
        tmin = t < tmin ? t : tmin;
        tmax = t > tmax ? t : tmax;
    }
    tmin = wave_min(tmin);
    tmax = wave_max(tmax);
    if (lane() == 0) {
        __hip_atomic_fetch_min(&info->ts_min, tmin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_max(&info->ts_max, tmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void k_publish(const RangeInfo* info, BackDst back, int64_t* skip) {
    *skip = info->long_case;
    publish(back, info, kInfoWords);
}

hipError_t launch_publish(const RangeInfo* info, BackDst back, int64_t* skip, hipStream_t s) {
    k_publish<<<1, 1, 0, s>>>(info, back, skip);
    return hipGetLastError();
}

__global__ void k_put_info(RangeInfo h, RangeInfo* info) { *info = h; }

hipError_t launch_put_info(const RangeInfo& h, RangeInfo* info, hipStream_t s) {
    k_put_info<<<1, 1, 0, s>>>(h, info);
    return hipGetLastError();
}

static int range_grid(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > kRangeParts) g = kRangeParts;
    return g < 1 ? 1 : (int)g;
}

hipError_t launch_range_scan(const int32_t* case_id, const int32_t* act, const int64_t* ts, int64_t n,
                             int32_t A, bool presorted, RangeInfo* info, RangePart* part,
                             uint32_t* hist_raw, int32_t* status, BackDst back, hipStream_t s) {
    ProfScope p(P_RANGE, s);
    int parts = 0;
    if (n > 0 && presorted) {
        parts = range_grid(n);
        k_range_scan<<<parts, 256, 0, s>>>(case_id, act, ts, n, A, part);
    } else if (n > 0) {
        parts = (int)radix_blocks(n);
        if (parts <= kRangeWhole) {
            k_range_tiles<true><<<1, kRangeTileThreads, 0, s>>>(case_id, act, n, A, part, hist_raw, parts, info, status,
                                                                back);
            return hipGetLastError();
        }
        k_range_tiles<false><<<parts, kRangeTileThreads, 0, s>>>(case_id, act, n, A, part, hist_raw, parts, info, status,
                                                                 back);
    }
    k_range_final<<<1, 1024, 0, s>>>(part, parts, info, status, back);
    return hipGetLastError();
}

hipError_t launch_ts_range(const int64_t* ts, int64_t n, RangeInfo* info, hipStream_t s) {
    if (n > 0) k_ts_range<<<range_grid(n), 256, 0, s>>>(ts, n, info);
    return hipGetLastError();
}

}  // namespace pm4g
