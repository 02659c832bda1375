// A few words from a kernel to the host code that waits for them: written into
// pinned host memory with system-scope stores, a sequence number last.  The
// waiting thread sees them some microseconds after the kernel wrote them, with
// later kernels already queued; a copy to pageable memory and a stream
// synchronisation took about 40 us, the GPU idle meanwhile.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pm4g {

constexpr int kBackWords = 16;

// Where a kernel writes; words == nullptr: nowhere (the caller copies instead).
struct BackDst {
    int64_t* words;
    uint64_t* flag;
    uint64_t seq;
};

// One thread writes the words, then the sequence number.  The words are read as
// bytes: `src` may be a struct of narrower fields that the thread has just stored.
__device__ __forceinline__ void publish(const BackDst& d, const void* src, int n) {
    if (!d.words) return;
    for (int k = 0; k < n; ++k) {
        int64_t w;
        __builtin_memcpy(&w, static_cast<const char*>(src) + k * sizeof(w), sizeof(w));
        __hip_atomic_store(&d.words[k], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __hip_atomic_store(d.flag, d.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Host side: one slot of the process's pinned page (64 slots, allocated once,
// kept; taken under a mutex, so calls of several threads hold different ones).
// Without a free slot, or without the page, dst() is empty and wait() copies.
class HostBack {
public:
    HostBack();
    ~HostBack();
    HostBack(const HostBack&) = delete;
    HostBack& operator=(const HostBack&) = delete;
    bool live() const { return slot_ >= 0; }   // false: wait() copies, so before the words are overwritten
    BackDst dst();   // for the next kernel that publishes; a call may publish several times
    // The n words that the kernel given dst() published, or (no slot) a copy of
    // the device words `dev`, which hold the same.
    hipError_t wait(const void* dev, int64_t* out, int n, hipStream_t s);

private:
    int slot_ = -1;
    bool pending_ = false;   // a kernel may still write into the slot
    uint64_t seq_ = 0;
};

}  // namespace pm4g
