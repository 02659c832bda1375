// Workspace slices whose sizes follow the present kernels of formatting,
// variants, batched views, filters, the eventually-follows graph and CSV: each
// layout is laid out over a fake base address (nothing is dereferenced) and the
// room of every slice up to the next one held against what its kernels index,
// restated here from their loops and grids.  ws_layout_check.cpp does the same
// for the sizes that did not change with them.  Prints a line per failure and
// exits with their number.  Built and run by tests/test_ws_slices.py.
#include <algorithm>
#include <cstdio>
#include <string>
#include <vector>

#include "common.hpp"
#include "devsort.hpp"
#include "internal.hpp"

using namespace pm4g;

namespace {

struct Need {
    const char* name;
    const void* p;
    size_t bytes;
};
#define NEED(field, count) Need{#field, (const void*)w.field, (size_t)(count) * sizeof(*w.field)}

char* const kBase = reinterpret_cast<char*>(uintptr_t(1) << 40);
int g_checked = 0;

// Slices without room (and whether they start at 256 bytes).
int short_slices(const std::string& what, size_t total, std::vector<Need> v, bool print = true) {
    std::sort(v.begin(), v.end(), [](const Need& a, const Need& b) { return a.p < b.p; });
    int bad = 0;
    for (size_t i = 0; i < v.size(); ++i) {
        const char* p = static_cast<const char*>(v[i].p);
        const char* end = i + 1 < v.size() ? static_cast<const char*>(v[i + 1].p) : kBase + total;
        const bool ok = p >= kBase && p <= kBase + total && (size_t)(end - p) >= v[i].bytes &&
                        reinterpret_cast<uintptr_t>(p) % 256 == 0;
        if (ok) continue;
        if (print) std::printf("FAIL %s: %s needs %zu B, has %td\n", what.c_str(), v[i].name, v[i].bytes, end - p);
        ++bad;
    }
    ++g_checked;
    return bad;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t at_least1(int64_t x) { return x > 0 ? x : 1; }
std::string tag(const char* s, int64_t a, int64_t b = -1, int64_t c = -1) {
    return std::string(s) + "(" + std::to_string(a) + ", " + std::to_string(b) + ", " + std::to_string(c) + ")";
}

// Formatting: digit rows of every width that radix_plan hands out for this many
// tiles, a row total per digit; the rows are counted for one tile too many by no
// kernel.  The case table reads four windows' counts at once (in bounds only).
int prep(int64_t n, bool rows) {
    Bump b(kBase);
    const PrepWs w = prep_ws_layout(b, n, rows);
    const int64_t m = at_least1(n), nb = radix_blocks(n);
    int64_t digits = 256;
    for (int bits = 0; bits <= 32; ++bits) {
        int width[4];
        const int passes = radix_plan(bits, n, width);
        int covered = 0;
        for (int p = 0; p < passes; ++p) {
            digits = std::max(digits, int64_t(1) << width[p]);
            covered += width[p];
        }
        if (passes > 4 || covered < bits) std::printf("FAIL plan of %d bits\n", bits);
    }
    const int64_t parts = std::max(nb, std::min<int64_t>(ceil_div(n, 256), kRangeParts));
    std::vector<Need> v = {NEED(info, 1), NEED(rpart, at_least1(parts)), NEED(a.key, m), NEED(a.ts, m), NEED(a.act, m), NEED(b.key, m),
                           NEED(b.ts, m), NEED(b.act, m), NEED(hist, digits * at_least1(nb)), NEED(hist_raw, 256 * at_least1(nb)),
                           NEED(rowsum, digits), NEED(caseblk, at_least1(case_blocks(n))), NEED(wincnt, at_least1(segsort_blocks(n)))};
    if (rows) {
        v.push_back(NEED(a.row, m));
        v.push_back(NEED(b.row, m));
    }
    return short_slices(tag("prep", n, rows), b.off, v);
}

// Variants: a claim table of two words per case from hash on (hash2 is inside
// it), counters and representatives per case, digit rows per tile of cases, the
// variants in order, one partial length per block of the emitting kernels.
int variants(int64_t n) {
    Bump b(kBase);
    const VarWs w = var_ws_layout(b, n);
    const int64_t C = at_least1(n);
    return short_slices(tag("variants", n), b.off,
                        {NEED(hash, 2 * C), NEED(idx, C), NEED(idx2, C), NEED(hist, 256 * at_least1(dev::tiles(n))), NEED(rowsum, 256),
                         NEED(sstart, C), NEED(repflag, C), NEED(rrank, C), NEED(vcr, C), NEED(cvar, C), NEED(vkey, C / 255 + 1),
                         NEED(vkey2, C / 255 + 1), NEED(vidx, C / 255 + 1), NEED(vidx2, C / 255 + 1), NEED(fid, C), NEED(lens, C),
                         NEED(part64, dev::kScanGrid), NEED(scal, 3)});
}

// Batched views: scal up to [14]; the placing kernels' block sums (at most
// kScanGrid blocks, kViewMaxBlocks in the persistent launch); parts of shared
// segments and their arrival counts; segment places per (view, bucket).
int views(int64_t n, int32_t A, int32_t V, int32_t tile, int64_t pair_cap, int64_t rec_cap, int64_t cell_cap) {
    Bump b(kBase);
    const ViewWs w = view_ws_layout(b, n, A, V, tile, pair_cap, rec_cap, cell_cap);
    const int64_t tiles = ceil_div(n, tile), nvb = at_least1((int64_t)V * view_buckets(A)), vm = at_least1(V);
    const int64_t pc = at_least1(pair_cap), rc = at_least1(rec_cap), cc = at_least1(cell_cap);
    const int64_t sums = std::max<int64_t>(dev::kScanGrid, kViewMaxBlocks);
    int bad = 0;
    if (w.parts < 1 || w.parts > 16 || (w.parts > 1 && (int64_t)w.parts * 16 > V)) {
        std::printf("FAIL %s: %d parts\n", tag("views", n, A, V).c_str(), w.parts);
        ++bad;
    }
    return bad + short_slices(tag("views", n, A, V), b.off,
                              {NEED(p0, vm), NEED(p1, vm), NEED(tcount, tiles + 1), NEED(toff, tiles + 1), NEED(tcursor, at_least1(tiles)),
                               NEED(list, pc), NEED(scal, 16), NEED(part32, sums), NEED(part64, sums), NEED(part64b, sums),
                               NEED(bar, kViewMaxBlocks + 1), NEED(rec_cell, rc), NEED(rec_gap, rc), NEED(pair_carry, pc),
                               NEED(pair_rel, pc * view_buckets(A)), NEED(vb_cnt, nvb), NEED(vb_base, nvb), NEED(vb_seg, nvb),
                               NEED(seg_key, nvb), NEED(seg_rec, nvb + 1), NEED(seg_cells, nvb), NEED(seg_tmp, nvb), NEED(seg_out, nvb),
                               NEED(view_cells, vm), NEED(t_cell, cc), NEED(t_count, cc), NEED(t_sum, cc), NEED(t_min, cc),
                               NEED(t_max, cc), NEED(agg_item, kViewAggItems), NEED(agg_done, kViewAggItems)});
}

// Event filters: a count per block of a grid of at most 2048 blocks and one per
// tile.  Case filters: flags and kept events per case, sums per block.
int filters(int64_t n) {
    Bump b(kBase);
    const FilterWs w = filter_ws_layout(b, n);
    const int64_t blocks = at_least1(std::min<int64_t>(ceil_div(n, kFilterTile), 2048));
    int bad = short_slices(tag("filter", n), b.off, {NEED(scal, 8), NEED(tile_cnt, blocks), NEED(caseblk, blocks)});
    Bump b2(kBase);
    {
        const CaseFilterWs w = case_filter_ws_layout(b2, n);
        const int64_t C = at_least1(n), g = at_least1(std::min<int64_t>(ceil_div(n, 512), dev::kScanGrid));
        bad += short_slices(tag("case_filter", n), b2.off, {NEED(flags, C), NEED(cnt, C), NEED(part32, g), NEED(part64, g)});
    }
    return bad;
}

// Eventually-follows graph: scal up to [5] ([5]: a long case).
int efg(int64_t n, int32_t A) {
    Bump b(kBase);
    const EfgWs w = efg_ws_layout(b, n, A);
    const int64_t nbk = efg_buckets(A), m = at_least1(n), entries = 512 + nbk;   // the plan's entries, at most
    static_assert(kEfgPlanBlocks >= 512, "two entries per aggregation block");
    return short_slices(tag("efg", n, A), b.off,
                        {NEED(tail, m), NEED(poff, m + 1), NEED(part64, dev::kScanGrid), NEED(scal, 6), NEED(bfirst, nbk), NEED(bnum, nbk),
                         NEED(plan, entries), NEED(part, entries * (int64_t)kSlotWords)});
}

// CSV: two fields and slots per row, written two at a time (aligned to 16 and 8
// bytes); the first rows' counts per 2048 rows.
int csv(int64_t n_bytes, int64_t max_rows) {
    Bump b(kBase);
    const CsvWs w = csv_ws_layout(b, n_bytes, max_rows);
    const int64_t rows = at_least1(max_rows);
    return short_slices(tag("csv", n_bytes, max_rows), b.off,
                        {NEED(line_end, rows + 2), NEED(foff, 2 * rows), NEED(flen, 2 * rows), NEED(slot, 2 * rows),
                         NEED(table, 2 * w.tsize), NEED(k0, ceil_div(rows, 2048)), NEED(scal, kBackWords)});
}

}  // namespace

int main() {
    int fail = 0;
    {   // the check itself: a slice of 10 words where 11 are needed
        Bump b(kBase);
        struct {
            uint32_t *x, *y;
        } w{b.take<uint32_t>(64), b.take<uint32_t>(10)};
        if (short_slices("self", b.off, {NEED(x, 64), NEED(y, 10)}, false) != 0) ++fail;
        if (short_slices("self", b.off, {NEED(x, 65), NEED(y, 10)}, false) != 1) ++fail;
        if (short_slices("self", b.off, {NEED(x, 64), NEED(y, 11)}, false) != 1) ++fail;
    }
    const int64_t ns[] = {0, 1, 2, 63, 254, 255, 256, 3072, 4095, 4096, 4097, 100000, 262144, 262145, 1 << 20, 16777217, 98969504, (1ll << 31) - 1};
    for (int64_t n : ns) {
        fail += prep(n, false) + prep(n, true) + variants(n) + filters(n);
        for (int32_t A : {1, 7, 64, 65, 100, 512, 1000, 4096}) fail += efg(n, A);
        for (int32_t V : {0, 1, 31, 32, 100, 255, 256, 4096})
            for (int32_t A : {1, 63, 64, 512, 513, 1024})
                for (int32_t tile : {2048, 4096}) {
                    const int64_t pairs = 4 * (ceil_div(n, tile) + V) + 1024, recs = std::max<int64_t>(n, 4096);
                    fail += views(n, A, V, tile, pairs, recs, std::max<int64_t>(recs / 2, 4096)) + views(n, A, V, tile, 1, 1, 1);
                }
    }
    for (int64_t nb : {0ll, 1ll, 4097ll, 508795914ll, 1ll << 34})
        for (int64_t r : {0ll, 1ll, 2ll, 1000ll, 2048ll, 2049ll, 9976391ll, 1ll << 27}) fail += csv(nb, r);
    std::printf("%d layouts checked, %d failures\n", g_checked, fail);
    return fail;
}
