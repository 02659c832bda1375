// Sampling of a prepared log (Sec. 3: the sampling module, a sample by a
// number of cases or of events).  The k units (cases by id, or events by their
// position in the formatted log) with the smallest SplitMix64 keys are kept;
// the keys are distinct, so the sample is unique and nested in k.
//
// The k-th smallest key is found by three MSD digit passes over recomputed keys
// (no memory traffic for events; 4 B per case code), each a histogram of the
// next 8 bits of the keys that match the prefix found so far; every block finds
// the prefix itself from the histograms before.  The candidates left (keys are
// a bijection's images: about one in 2^24 units, a few hundred of all 2^32 case
// ids) are listed, and one block ranks them.  More candidates than the list
// holds are not expected of any ids; should they come, that block selects among
// all units, 8 bits a pass, so the answer never depends on it.
// Six launches; eight passes with a picking launch each were 17.
#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"
#include "../../include/pm4g.h"

namespace pm4g {
namespace {

constexpr int kSB = 1024;

__global__ __launch_bounds__(256) void k_sel_init(SelState* sel, int64_t k, const int64_t* count_dev,
                                                  int64_t count_host) {
    const int64_t count = count_dev ? *count_dev : count_host;
    for (int p = 0; p < kSelPasses; ++p) sel->hist[p][threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        sel->T = ~0ull;
        sel->none = k <= 0 ? 1 : 0;
        sel->all = (k > 0 && k >= count) ? 1 : 0;
        sel->n_list = 0;
    }
}

struct Units {
    const int32_t* case_code;    // NULL: units are positions
    const int64_t* count_dev;
    int64_t count_host;
    uint64_t seed;
    __device__ __forceinline__ int64_t count() const { return count_dev ? *count_dev : count_host; }
    __device__ __forceinline__ uint64_t key(int64_t u) const {
        return splitmix64(seed, case_code ? (uint64_t)(uint32_t)case_code[u] : (uint64_t)u);
    }
};

// The digit whose bin holds the krem-th smallest of the keys counted in hist;
// krem becomes its rank in the bin.  A block of 256 or more threads together.
template <int BLOCK>
__device__ __forceinline__ uint32_t pick(const uint32_t* hist, int64_t* krem, uint32_t* tmp, int64_t* found) {
    const uint32_t v = threadIdx.x < 256 ? hist[threadIdx.x] : 0u;
    uint32_t total;
    const uint32_t ex = block_excl_sum<BLOCK>(v, tmp, &total);
    const int64_t k = *krem;
    if (threadIdx.x < 256 && (int64_t)ex < k && k <= (int64_t)ex + (int64_t)v) {   // exactly one thread
        found[0] = threadIdx.x;
        found[1] = k - (int64_t)ex;
    }
    __syncthreads();
    const uint32_t d = (uint32_t)found[0];
    *krem = found[1];
    __syncthreads();
    return d;
}

// Histogram of digit `pass` (most significant first) of the keys whose higher
// digits equal the prefix; pass `last` lists those keys instead, `cap` at most.
__global__ __launch_bounds__(kSB) void k_sel_pass(Units units, int64_t k, int pass, int last, uint32_t cap,
                                                  SelState* sel) {
    __shared__ uint32_t h[256];
    __shared__ uint32_t tmp[kSB / kWave + 1];
    __shared__ int64_t found[2];
    if (sel->none || sel->all) return;   // uniform: nothing to select
    uint64_t prefix = 0;
    int64_t krem = k;
    for (int p = 0; p < pass; ++p) prefix = prefix << 8 | pick<kSB>(sel->hist[p], &krem, tmp, found);
    const int64_t count = units.count();
    const int shift = 64 - 8 * pass;   // bits below the prefix (64: no prefix yet)
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t u = (int64_t)blockIdx.x * kSB + threadIdx.x; u < count; u += (int64_t)gridDim.x * kSB) {
        const uint64_t key = units.key(u);
        if (pass > 0 && (key >> shift) != prefix) continue;
        if (pass < last) {
            atomicAdd(&h[(key >> (shift - 8)) & 255u], 1u);
        } else {
            const uint32_t at = atomicAdd(&sel->n_list, 1u);
            if (at < cap) sel->list[at] = key;
        }
    }
    if (pass == last) return;
    __syncthreads();
    if (threadIdx.x < 256 && h[threadIdx.x]) atomicAdd(&sel->hist[pass][threadIdx.x], h[threadIdx.x]);
}

// One block: the krem-th smallest of the keys listed after `last` passes.
__global__ __launch_bounds__(kSB) void k_sel_final(Units units, int64_t k, int last, uint32_t cap, SelState* sel) {
    __shared__ uint32_t tmp[kSB / kWave + 1];
    __shared__ int64_t found[2];
    __shared__ uint32_t h[256];
    if (sel->none || sel->all) return;
    uint64_t prefix = 0;
    int64_t krem = k;
    for (int p = 0; p < last; ++p) prefix = prefix << 8 | pick<kSB>(sel->hist[p], &krem, tmp, found);
    const uint32_t m = sel->n_list;
    if (m <= cap) {
        for (uint32_t i = threadIdx.x; i < m; i += kSB) {
            const uint64_t key = sel->list[i];
            int64_t rank = 1;
            for (uint32_t j = 0; j < m; ++j) rank += sel->list[j] < key ? 1 : 0;
            if (rank == krem) sel->T = key;   // keys are distinct: one thread
        }
        return;
    }
    const int64_t count = units.count();
    for (int pass = last; pass < 8; ++pass) {
        if (threadIdx.x < 256) h[threadIdx.x] = 0;
        __syncthreads();
        const int shift = 64 - 8 * pass;
        for (int64_t u = threadIdx.x; u < count; u += kSB) {
            const uint64_t key = units.key(u);
            if ((key >> shift) == prefix) atomicAdd(&h[(key >> (shift - 8)) & 255u], 1u);
        }
        __syncthreads();
        prefix = prefix << 8 | pick<kSB>(h, &krem, tmp, found);
    }
    if (threadIdx.x == 0) sel->T = prefix;
}

}  // namespace

hipError_t launch_sample_select(const pm4g_prepared* p, int64_t k, uint64_t seed, bool by_events, SelState* sel,
                                int passes, int list, hipStream_t s) {
    const int last = passes > 0 && passes < kSelPasses ? passes : kSelPasses;
    const uint32_t cap = list >= 0 && list < kSelList ? (uint32_t)list : (uint32_t)kSelList;
    // events, or an upper bound of the cases
    const Units units{by_events ? nullptr : p->case_code, by_events ? nullptr : p->n_cases, p->n_events, seed};
    const int64_t g = (p->n_events + kSB - 1) / kSB;
    // 512 blocks: each adds its 256 counts to the same words
    const unsigned grid = (unsigned)(g < 512 ? (g < 1 ? 1 : g) : 512);
    k_sel_init<<<1, 256, 0, s>>>(sel, k, units.count_dev, units.count_host);
    for (int pass = 0; pass <= last; ++pass) k_sel_pass<<<grid, kSB, 0, s>>>(units, k, pass, last, cap, sel);
    k_sel_final<<<1, kSB, 0, s>>>(units, k, last, cap, sel);
    return hipGetLastError();
}

}  // namespace pm4g
