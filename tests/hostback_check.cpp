// The pinned slots of HostBack on the CPU: the HIP calls it makes are this
// program's own (nothing touches a GPU).  Prints one line per failure and exits
// with their number.  Built and run by tests/test_hostback_cpu.py.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <vector>

#include "hostback.hip"

namespace {
int g_refuse = 0;    // hipHostMalloc calls still to refuse
int g_mallocs = 0, g_copies = 0, g_syncs = 0;
int g_fail = 0;

void expect(bool ok, const char* what) {
    if (!ok) {
        std::printf("FAIL %s\n", what);
        ++g_fail;
    }
}
}  // namespace

extern "C" {
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    ++g_mallocs;
    if (g_refuse > 0) {
        --g_refuse;
        return hipErrorStreamCaptureUnsupported;
    }
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    ++g_copies;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    ++g_syncs;
    return hipSuccess;
}
}

using pm4g::BackDst;
using pm4g::HostBack;

// What the kernel does with a destination.
static void publish_now(const BackDst& d, int64_t a, int64_t b) {
    d.words[0] = a;
    d.words[1] = b;
    __atomic_store_n(d.flag, d.seq, __ATOMIC_RELEASE);
}

int main() {
    const int64_t dev[2] = {41, 42};
    int64_t got[2] = {0, 0};

    g_refuse = 2;   // no page twice (as during another thread's capture), then one
    for (int k = 0; k < 2; ++k) {
        HostBack h;
        expect(!h.live() && h.dst().words == nullptr, "without a page there is no slot");
        expect(h.wait(dev, got, 2, nullptr) == hipSuccess && got[0] == 41 && got[1] == 42, "without a page the words are copied");
    }
    expect(g_copies == 2 && g_syncs == 2, "one copy and one wait each");
    {
        HostBack h;
        expect(h.live(), "a page refused once is asked for again");
        if (h.live()) {
            for (int64_t k = 0; k < 3; ++k) {   // several times per call
                publish_now(h.dst(), 7 + k, 8);
                expect(h.wait(nullptr, got, 2, nullptr) == hipSuccess && got[0] == 7 + k && got[1] == 8, "published words");
            }
        }
    }
    const int mallocs = g_mallocs, copies = g_copies;
    {
        std::vector<std::unique_ptr<HostBack>> all;
        for (int k = 0; k < 64; ++k) {
            all.push_back(std::make_unique<HostBack>());
            expect(all.back()->live(), "64 calls at once hold a slot each");
        }
        HostBack h;
        expect(!h.live() && h.wait(dev, got, 2, nullptr) == hipSuccess && got[1] == 42, "the next one copies");
    }
    expect(g_copies == copies + 1, "one copy");
    {
        HostBack h;
        expect(h.live(), "slots come back");
        (void)h.dst();   // never waited for: a kernel may still write
    }
    {
        std::vector<std::unique_ptr<HostBack>> all;
        int live = 0;
        for (int k = 0; k < 64; ++k) {
            all.push_back(std::make_unique<HostBack>());
            live += all.back()->live();
        }
        expect(live == 63, "a slot that a kernel may still write into is not handed out again");
    }
    expect(g_mallocs == mallocs, "one page for the process");
    std::printf("%d failures\n", g_fail);
    return g_fail;
}
