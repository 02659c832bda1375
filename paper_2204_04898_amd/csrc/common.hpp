// Device helpers shared by the pm4g kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pm4g {

constexpr int kWave = 64;

__device__ __forceinline__ int lane() { return __lane_id(); }

// XCD-contiguous work split.  The dispatcher deals a grid's blocks
// round-robin to the 8 XCDs (block b runs on XCD b % 8), and each XCD has its
// own L2.  Items [0, n) are cut into 8 contiguous ranges, one per XCD; the
// blocks of an XCD stride over its range.  Neighbouring items (whose outputs
// share cache lines at run boundaries) then meet in the same L2.  A bijection
// for any grid; grids below 8 blocks keep the plain split.
struct XcdSplit {
    int64_t first, end, stride;
};
__device__ __forceinline__ XcdSplit xcd_split(int64_t n) {
    const int64_t G = gridDim.x, b = blockIdx.x;
    if (G < 8) return XcdSplit{b, n, G};
    const int64_t x = b % 8, j = b / 8;
    const int64_t blocks = G / 8 + (x < G % 8 ? 1 : 0);   // blocks on XCD x
    const int64_t q = n / 8, r = n % 8;
    const int64_t begin = x * q + (x < r ? x : r);
    return XcdSplit{begin + j, begin + q + (x < r ? 1 : 0), blocks};
}

// Order of the batched views' walks over tiles (or parts of tiles): the i-th of
// n items for block b of G, or -1 past the end (increasing in i).  With no more
// items than blocks, one each.  Otherwise chunks of kXcdChunk consecutive items
// are dealt round-robin to the 8 XCDs (block b runs on XCD b % 8) and an XCD's
// blocks stride over its chunks, so neighbouring tiles, whose runs of records
// sit side by side in the record segments, are written through the same L2,
// while the chunks keep the XCDs' loads even along the log.  (Few items dealt in
// chunks leave XCDs without any: 48 views of a 65,536-event log, 48 items, took
// 388 us, 142 one per block; a contiguous range of few items per XCD was no
// faster than the round-robin and up to 20 % slower.)
constexpr int64_t kXcdChunk = 64;
__host__ __device__ __forceinline__ int64_t walk_item(int64_t b, int64_t G, int64_t i, int64_t n) {
    int64_t t;
    if (G % 8 != 0 || n <= G) {
        t = b + i * G;
    } else {
        const int64_t x = b % 8, s = b / 8 + i * (G / 8);
        t = ((s / kXcdChunk) * 8 + x) * kXcdChunk + s % kXcdChunk;
    }
    return t < n ? t : -1;
}

// Mask of the lanes below this one.
__device__ __forceinline__ uint64_t lanes_below() {
    return (uint64_t(1) << lane()) - uint64_t(1);
}

// Lanes of this wave whose BITS-bit digit equals this lane's, among `active`.
// Per bit: the lanes agreeing with this lane are ~(ballot ^ s), s this lane's
// bit spread over the word (0 or all ones), which gfx950 folds with the and
// into one three-input bit operation per 32-bit half.
template <int BITS>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, uint64_t active) {
    uint32_t lo = (uint32_t)active, hi = (uint32_t)(active >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint32_t s = 0u - ((d >> b) & 1u);
        const uint64_t m = __ballot(s != 0u);
        lo &= ~((uint32_t)m ^ s);
        hi &= ~((uint32_t)(m >> 32) ^ s);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Lanes of this wave whose value agrees with this lane's in the low `bits`
// bits, among `active`.  Every lane of the wave must execute it (`bits` is
// wave-uniform).
__device__ __forceinline__ uint64_t match_bits(uint32_t v, int bits, uint64_t active) {
    uint32_t lo = (uint32_t)active, hi = (uint32_t)(active >> 32);
    for (int b = 0; b < bits; ++b) {
        const uint32_t s = 0u - ((v >> b) & 1u);   // as in match_digit
        const uint64_t m = __ballot(s != 0u);
        lo &= ~((uint32_t)m ^ s);
        hi &= ~((uint32_t)(m >> 32) ^ s);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Wave-aggregated LDS counter increment: the lanes with `has` set add one to
// counter[key]; each gets the counter's value before its own increment (one
// atomic per distinct key).  Every lane of the wave must execute it.
__device__ __forceinline__ uint32_t wave_bump(uint32_t* counter, uint32_t key, int key_bits, bool has) {
    const uint64_t active = __ballot(has);
    const uint64_t peers = match_bits(has ? key : 0u, key_bits, active);
    const uint32_t rank = (uint32_t)__popcll(peers & lanes_below());
    const int leader = has ? (int)__ffsll((unsigned long long)peers) - 1 : 0;
    uint32_t base = 0;
    if (has && rank == 0) base = atomicAdd(&counter[key], (uint32_t)__popcll(peers));
    base = (uint32_t)__shfl((int)base, leader);
    return base + rank;
}

// SplitMix64 (Steele, Lea and Flood, 2014): the x-th output (x = 0, 1, ...)
// of the generator started from state `seed`.  A bijection of x for a fixed
// seed, so distinct inputs never share a key.
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t x) {
    uint64_t z = seed + (x + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Segment of position p among 64 consecutive segments (lane m holds the start
// of segment m, INT64_MAX if absent; p >= start of segment 0): the last m
// whose start is <= p.  Every lane of the wave must execute it.
__device__ __forceinline__ int seg_at(int64_t vstart, int64_t p) {
    int lo = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        const int cand = lo + step;
        if (__shfl(vstart, cand) <= p) lo = cand;
    }
    return lo;
}

// Orders this wave's LDS accesses before it and after it (the lanes run
// together; only the compiler has to keep the order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sums over a wave run on DPP moves: six steps of a few cycles each, where a
// shuffle goes through LDS (a dependent step of 60 cycles and more).  Every
// lane of the wave must execute them.  wave_add_dpp: v plus the value that the
// DPP control CTRL brings from another lane (nothing where it has no source,
// or in the rows outside ROWS).
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T wave_add_dpp(T v) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "integers of 4 or 8 bytes");
    if constexpr (sizeof(T) == 4) {
        return v + (T)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
        const uint32_t hi =
            (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)v >> 32), CTRL, ROWS, 0xF, false);
        return (T)((uint64_t)v + (((uint64_t)hi << 32) | lo));
    }
}
// Lane l's value (l the same in every lane).
template <typename T>
__device__ __forceinline__ T wave_lane(T v, int l) {
    if constexpr (sizeof(T) == 4) {
        return (T)__builtin_amdgcn_readlane((int)v, l);
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), l);
        return (T)(((uint64_t)hi << 32) | lo);
    }
}
// Inclusive sums within each row of 16 lanes.
template <typename T>
__device__ __forceinline__ T row_incl_sum(T v) {
    v = wave_add_dpp<0x111, 0xF>(v);   // row_shr 1, 2, 4, 8
    v = wave_add_dpp<0x112, 0xF>(v);
    v = wave_add_dpp<0x114, 0xF>(v);
    return wave_add_dpp<0x118, 0xF>(v);
}
template <typename T>
__device__ __forceinline__ T wave_incl_sum(T v) {
    v = row_incl_sum(v);
    v = wave_add_dpp<0x142, 0xA>(v);      // row_bcast 15: row 0's sum to row 1, row 2's to row 3
    return wave_add_dpp<0x143, 0xC>(v);   // row_bcast 31: rows 0 and 1's sum to rows 2 and 3
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
    return wave_lane(wave_incl_sum(v), kWave - 1);
}

// A bit set of `bits` bits (64-bit words in memory) as 32-bit words in LDS, by a
// block; bits_bytes: their room.
inline size_t bits_bytes(int64_t bits) { return (size_t)((bits + 63) / 64) * 8; }
template <int BLOCK>
__device__ __forceinline__ void stage_bits(const uint64_t* __restrict__ words, int64_t bits, uint32_t* lds) {
    const uint32_t* w = reinterpret_cast<const uint32_t*>(words);
    const int n = 2 * (int)((bits + 63) / 64);
    for (int i = threadIdx.x; i < n; i += BLOCK) lds[i] = w[i];
}

// The same search over 32-bit starts (one lane exchange per step instead of
// two; UINT32_MAX if absent).
__device__ __forceinline__ int seg_of32(uint32_t vstart, uint32_t p) {
    int lo = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
        const int cand = lo + step;
        if (__shfl(vstart, cand) <= p) lo = cand;
    }
    return lo;
}

// First position of the ascending a[0, n) not below x; a wave together, 64
// probes a step (4 dependent loads over 16M entries, not 24).
__device__ __forceinline__ int64_t lb_i32(const int32_t* a, int64_t n, int32_t x) {
    int64_t lo = 0, hi = n;   // the answer lies in [lo, hi]
    while (lo < hi) {
        const int64_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t p = lo + (int64_t)lane() * step;
        const uint64_t below = __ballot(p < hi && a[p < hi ? p : lo] < x);   // the first lanes, or none
        if (below == 0) return lo;
        const int64_t last = lo + (63 - (int64_t)__clzll((long long)below)) * step;   // a[last] < x
        hi = last + step < hi ? last + step : hi;
        lo = last + 1;
    }
    return lo;
}

template <typename T>
__device__ __forceinline__ T wave_min(T v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        T u = __shfl_xor(v, o);
        v = u < v ? u : v;
    }
    return v;
}

template <typename T>
__device__ __forceinline__ T wave_max(T v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        T u = __shfl_xor(v, o);
        v = u > v ? u : v;
    }
    return v;
}

// Exclusive prefix sum over a block of BLOCK threads (one value per thread).
// `tmp` must hold BLOCK/64 + 1 entries of T in LDS.  Returns the exclusive
// sum; *total receives the block total.  Contains __syncthreads().  Each wave
// adds up the waves' sums itself (one LDS read and four DPP steps, instead of
// one thread's chain over LDS and a barrier; with the wave sums on DPP, three
// case filters of 20M events went from 699 to 642 us).
template <int BLOCK, typename T>
__device__ __forceinline__ T block_excl_sum(T v, T* tmp, T* total) {
    constexpr int NW = BLOCK / kWave;
    static_assert(BLOCK % kWave == 0 && NW >= 1 && NW <= 16, "the waves' sums fill one row of lanes");
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const T inc = wave_incl_sum(v);
    if (lane() == kWave - 1) tmp[w] = inc;
    __syncthreads();
    const T sums = row_incl_sum(lane() < NW ? tmp[lane()] : (T)0);
    __syncthreads();
    *total = wave_lane(sums, NW - 1);
    return (w > 0 ? wave_lane(sums, w - 1) : (T)0) + inc - v;
}

// Saturating add of non-negative 64-bit amounts, capped at 2^63 (any value
// >= 2^63 means "exceeds INT64_MAX").  Inputs must already be <= 2^63.
__device__ __forceinline__ uint64_t sat_add63(uint64_t a, uint64_t b) {
    constexpr uint64_t cap = uint64_t(1) << 63;
    return (a > cap - b) ? cap : a + b;
}
__device__ __forceinline__ uint64_t cap63(uint64_t a) {
    constexpr uint64_t cap = uint64_t(1) << 63;
    return a > cap ? cap : a;
}

// Record a data-dependent error; the first one wins.
__device__ __forceinline__ void set_status(int32_t* status, int32_t code) {
    atomicCAS(status, 0, code);
}

}  // namespace pm4g
