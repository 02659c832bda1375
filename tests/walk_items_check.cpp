// The order in which the batched views' walks take their work (walk_item), on
// the CPU: every item once, a block's items increasing, and with no more items
// than blocks none has two.  Prints a line per failure and exits with their
// number.  Built and run by tests/test_walk_items_cpu.py.
#include <cstdio>
#include <vector>

#include "common.hpp"

int main() {
    int fail = 0, checked = 0;
    for (int64_t G : {1, 2, 7, 8, 9, 16, 48, 64, 128, 208, 255, 256, 312, 512, 1000, 2048})
        for (int64_t n : {0, 1, 6, 8, 13, 48, 63, 64, 65, 104, 105, 128, 195, 208, 255, 256, 257, 312, 511, 512, 513, 1024, 2047, 2048,
                          2049, 5000, 24163}) {
            std::vector<int> seen(n, 0);
            int64_t most = 0;
            for (int64_t b = 0; b < G; ++b) {
                int64_t last = -1, k = 0;
                for (int64_t i = 0, t; (t = pm4g::walk_item(b, G, i, n)) >= 0; ++i, ++k) {
                    if (t >= n || t <= last) ++fail;
                    else ++seen[t];
                    last = t;
                }
                most = k > most ? k : most;
            }
            int64_t once = 0;
            for (int c : seen) once += c == 1;
            const bool ok = once == n && (n > G || most <= 1);
            if (!ok) {
                std::printf("FAIL %lld items on %lld blocks: %lld once, at most %lld per block\n", (long long)n, (long long)G,
                            (long long)once, (long long)most);
                ++fail;
            }
            ++checked;
        }
    std::printf("%d checked, %d failures\n", checked, fail);
    return fail;
}
