// Pinned slots of HostBack (hostback.hpp).  Host code only.
#include "hostback.hpp"

#include <sched.h>

#include <chrono>
#include <mutex>

namespace pm4g {
namespace {

struct Slot {
    int64_t words[kBackWords];
    uint64_t flag;
    uint64_t pad[15];
};
static_assert(sizeof(Slot) == 256, "slots on lines of their own");
constexpr int kSlots = 64;

std::mutex g_mu;
Slot* g_page = nullptr;
uint64_t g_used = 0;   // bit per slot
uint64_t g_seq = 0;

}  // namespace

HostBack::HostBack() {
    std::lock_guard<std::mutex> l(g_mu);
    if (!g_page) {
        void* p = nullptr;
        if (hipHostMalloc(&p, kSlots * sizeof(Slot),
                          hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) {
            g_page = static_cast<Slot*>(p);
            for (int k = 0; k < kSlots; ++k) g_page[k].flag = 0;
        } else {
            // the copying way works without it; the next call asks again (another
            // thread's graph capture refuses allocations while it lasts)
            (void)hipGetLastError();
        }
    }
    if (!g_page || g_used == ~0ull) return;
    slot_ = __builtin_ctzll(~g_used);
    g_used |= 1ull << slot_;
}

HostBack::~HostBack() {
    // a slot that a kernel may still write into is never handed out again
    if (slot_ < 0 || pending_) return;
    std::lock_guard<std::mutex> l(g_mu);
    g_used &= ~(1ull << slot_);
}

BackDst HostBack::dst() {
    if (slot_ < 0) return BackDst{nullptr, nullptr, 0};
    {
        std::lock_guard<std::mutex> l(g_mu);
        seq_ = ++g_seq;
    }
    pending_ = true;
    Slot& s = g_page[slot_];
    return BackDst{s.words, &s.flag, seq_};
}

hipError_t HostBack::wait(const void* dev, int64_t* out, int n, hipStream_t s) {
    if (slot_ < 0) {
        hipError_t e = hipMemcpyAsync(out, dev, (size_t)n * sizeof(int64_t), hipMemcpyDeviceToHost, s);
        return e != hipSuccess ? e : hipStreamSynchronize(s);
    }
    Slot& slot = g_page[slot_];
    const auto there = [&] { return __atomic_load_n(&slot.flag, __ATOMIC_ACQUIRE) == seq_; };
    // poll for 2 ms (a call on a few million events), yielding; then let the
    // runtime wait.  Both end: the stream's work ends or reports an error.
    const auto t0 = std::chrono::steady_clock::now();
    bool ok = there();
    for (int k = 1; !ok; ++k) {
        __builtin_ia32_pause();
        ok = there();
        if (ok || k % 64) continue;
        sched_yield();
        if (std::chrono::steady_clock::now() - t0 < std::chrono::milliseconds(2)) continue;
        const hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        ok = there();
        if (!ok) {
            pending_ = false;   // the stream is done: nothing writes any more
            return hipErrorUnknown;
        }
    }
    pending_ = false;
    for (int k = 0; k < n; ++k) out[k] = slot.words[k];
    return hipSuccess;
}

}  // namespace pm4g
