// Case table of a prepared log (Sec. 3, third formatting step, "cases
// dataframe"; Sec. 2.1 group identification): case_code[j] is the j-th
// distinct case id in order and case_off[j] the position of its first event.
// Reduce-then-scan compaction of the boundary flags
// flag(i) = (i == 0) || case_s[i] != case_s[i-1]:
//   k_case_count  per-tile flag counts (not needed where the per-case sort
//                 already counted the cases of each of its windows)
//   k_case_scan   exclusive scan of the tile counts, n_cases, case_off[C] = N
//                 (not needed up to kCaseDirect tiles: each tile of k_case_emit
//                 sums the counts before it itself, a few loads per thread)
//   k_case_emit   per-tile ranks -> case_off / case_code
// Bytes per event: 4 read after the per-case sort, else 4 + 4.
#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"

namespace pm4g {

constexpr int kCB = 256;
constexpr int kCI = kCaseTile / kCB;   // 16

__global__ __launch_bounds__(kCB) void k_case_count(const int32_t* __restrict__ case_s, int64_t n,
                                                    uint32_t* blockcnt) {
    __shared__ uint32_t tmp[kCB / kWave + 1];
    const int64_t base = (int64_t)blockIdx.x * kCaseTile;
    // loads at clamped positions (n >= 1), all issued before any is used
    int32_t cv[kCI], pv[kCI];
#pragma unroll
    for (int k = 0; k < kCI; ++k) {
        const int64_t i = base + k * kCB + threadIdx.x;
        const int64_t ic = i < n ? i : n - 1;
        cv[k] = case_s[ic];
        pv[k] = case_s[ic > 0 ? ic - 1 : 0];
    }
    __builtin_amdgcn_sched_barrier(0);
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kCI; ++k) {
        const int64_t i = base + k * kCB + threadIdx.x;
        if (i < n && (i == 0 || cv[k] != pv[k])) ++c;
    }
    uint32_t total;
    block_excl_sum<kCB>(c, tmp, &total);
    if (threadIdx.x == 0) blockcnt[blockIdx.x] = total;
}

// Counts of tile t: per_tile counts [t * per_tile, ...) of the nc given (1: one
// count per tile; 4: one per sort window).
constexpr int kPerTile = kCaseTile / kSegWindow;
static_assert(kCaseTile % kSegWindow == 0 && kPerTile == 4, "a case tile holds four sort windows (one 16-byte load)");
__device__ __forceinline__ uint32_t tile_count(const uint32_t* cnt, int64_t nc, int per_tile, int64_t t) {
    if (per_tile == 1) return t < nc ? cnt[t] : 0u;
    if (4 * t + 3 < nc) {
        const uint4 v = *reinterpret_cast<const uint4*>(cnt + 4 * t);
        return v.x + v.y + v.z + v.w;
    }
    uint32_t c = 0;
    for (int64_t k = 4 * t; k < nc; ++k) c += cnt[k];   // the last tile's windows, or none
    return c;
}

// The formatting step's header to the host (one thread), where the call waits for it.
__device__ __forceinline__ void publish_info(const BackDst& back, const RangeInfo* info) {
    if (info) publish(back, info, kInfoWords);
}

__global__ __launch_bounds__(1024) void k_case_scan(const uint32_t* cnt, int64_t nc, int per_tile, uint32_t* blockoff,
                                                    int64_t nb, int64_t n, int64_t* case_off, int64_t* n_cases,
                                                    const RangeInfo* info, BackDst back) {
    if (threadIdx.x == 0) publish_info(back, info);
    if (info && info->long_case) {   // uncounted windows
        if (threadIdx.x == 0) *n_cases = case_off[0] = 0;
        return;
    }
    __shared__ uint32_t tmp[1024 / kWave + 1];
    constexpr int kT = 4;   // tiles per thread and step
    uint32_t run = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += 1024 * kT) {
        const int64_t t0 = c0 + (int64_t)threadIdx.x * kT;
        uint32_t v[kT], sum = 0;
#pragma unroll
        for (int q = 0; q < kT; ++q) {
            v[q] = tile_count(cnt, nc, per_tile, t0 + q);
            sum += v[q];
        }
        uint32_t total;
        uint32_t r = run + block_excl_sum<1024>(sum, tmp, &total);
#pragma unroll
        for (int q = 0; q < kT; ++q) {
            if (t0 + q < nb) blockoff[t0 + q] = r;
            r += v[q];
        }
        run += total;
    }
    if (threadIdx.x == 0) {
        *n_cases = run;
        case_off[run] = n;
    }
}

__global__ __launch_bounds__(kCB) void k_case_emit(const int32_t* __restrict__ case_s, int64_t n,
                                                   const uint32_t* blockoff, const uint32_t* cnt, int64_t nc,
                                                   int per_tile, int64_t* case_off, int32_t* case_code,
                                                   int64_t* n_cases, const RangeInfo* info, BackDst back) {
    if (blockIdx.x == 0 && threadIdx.x == 0) publish_info(back, info);
    if (info && info->long_case) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *n_cases = case_off[0] = 0;
        return;
    }
    // striped layout (coalesced loads): item k of thread t is position base + k*256 + t,
    // so position order is (k, wave, lane) order; ranks from ballots + one small scan
    constexpr int kNW = kCB / kWave;
    __shared__ uint32_t wcnt[kCI * kNW];
    __shared__ uint32_t tmp[kCB / kWave + 1];
    const int64_t base = (int64_t)blockIdx.x * kCaseTile;
    const int w = threadIdx.x / kWave;
    uint64_t masks[kCI];
    // loads at clamped positions (n >= 1), all issued before any is used
    int32_t cv[kCI], pv[kCI];
#pragma unroll
    for (int k = 0; k < kCI; ++k) {
        const int64_t i = base + k * kCB + threadIdx.x;
        const int64_t ic = i < n ? i : n - 1;
        cv[k] = case_s[ic];
        pv[k] = case_s[ic > 0 ? ic - 1 : 0];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kCI; ++k) {
        const int64_t i = base + k * kCB + threadIdx.x;
        const bool f = i < n && (i == 0 || cv[k] != pv[k]);
        masks[k] = __ballot(f);
        if (lane() == 0) wcnt[k * kNW + w] = (uint32_t)__popcll(masks[k]);
    }
    __syncthreads();
    // exclusive scan of the kCI * kNW (k-major) wave counts; kCI * kNW = 64 <= kCB
    uint32_t total;
    const uint32_t v = threadIdx.x < kCI * kNW ? wcnt[threadIdx.x] : 0u;
    const uint32_t ex = block_excl_sum<kCB>(v, tmp, &total);
    if (threadIdx.x < kCI * kNW) wcnt[threadIdx.x] = ex;
    __syncthreads();
    uint32_t b0;
    if (blockoff) {
        b0 = blockoff[blockIdx.x];
    } else {   // no scan: the cases of the tiles before this one
        uint32_t before = 0;
        for (int64_t t = threadIdx.x; t < (int64_t)blockIdx.x; t += kCB) before += tile_count(cnt, nc, per_tile, t);
        block_excl_sum<kCB>(before, tmp, &b0);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
            *n_cases = b0 + total;
            case_off[b0 + total] = n;
        }
    }
#pragma unroll
    for (int k = 0; k < kCI; ++k) {
        if ((masks[k] >> lane()) & 1ull) {
            const uint32_t r = b0 + wcnt[k * kNW + w] + (uint32_t)__popcll(masks[k] & lanes_below());
            case_off[r] = base + k * kCB + threadIdx.x;
            case_code[r] = cv[k];
        }
    }
}

hipError_t launch_case_table(const int32_t* case_s, int64_t n, uint32_t* blockcnt, int64_t* case_off,
                             int32_t* case_code, int64_t* n_cases, const uint32_t* wincnt, const RangeInfo* info,
                             BackDst back, hipStream_t s) {
    ProfScope p(P_CASE_TABLE, s);
    const int64_t nb = case_blocks(n);
    // nb partial sums of the tiles before: nb^2 / 2 cached loads against a launch
    // of 4.5 us and a one-block scan (22 us for 24k tiles)
    constexpr int64_t kCaseDirect = 1024;
    const uint32_t* cnt = wincnt;
    int64_t nc = segsort_blocks(n);
    int per_tile = kPerTile;
    if (!wincnt) {
        info = nullptr;
        if (nb > 0) k_case_count<<<(unsigned)nb, kCB, 0, s>>>(case_s, n, blockcnt);
        cnt = blockcnt;
        nc = nb;
        per_tile = 1;
    }
    const bool scan = nb == 0 || nb > kCaseDirect;
    if (scan) {
        k_case_scan<<<1, 1024, 0, s>>>(cnt, nc, per_tile, blockcnt, nb, n, case_off, n_cases, info, back);
        back.words = nullptr;   // the first kernel writes the header
    }
    if (nb > 0)
        k_case_emit<<<(unsigned)nb, kCB, 0, s>>>(case_s, n, scan ? blockcnt : nullptr, cnt, nc, per_tile, case_off,
                                                 case_code, n_cases, info, back);
    return hipGetLastError();
}

}  // namespace pm4g
