// Checks of expert_items.h on the CPU: every (segment, column, K range) of a launch is done by exactly
// one workgroup, the XCDs get equal shares, and a group mixes experts only where no expert repeats;
// and of the pieces a launch is cut into.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "expert_items.h"

using namespace qmoe;

#define CHECK(c) do { if (!(c)) { std::printf("failed line %d: %s (n %d cols %u)\n", __LINE__, #c, n, cols); std::exit(1); } } while (0)

// Workgroups as launch1 starts them and map_block decodes them.
template <class Pos>
static void walk(int n, unsigned cols, Pos &&pos) {
    const unsigned items = n * cols;
    unsigned share[kXcds] = {};
    std::vector<int> seen(items, 0);
    for (unsigned w = 0; w < item_grid(items); ++w) {
        unsigned item;
        if (!item_of(w, items, item)) continue;
        CHECK(item < items);
        const ItemPos p = pos(item);
        CHECK(p.pos < (unsigned)n && p.cq < cols);
        ++seen[(size_t)p.pos * cols + p.cq];
        ++share[w % kXcds];
    }
    for (int v : seen) CHECK(v == 1);
    CHECK(*std::max_element(share, share + kXcds) - *std::min_element(share, share + kXcds) <= 1);
}

// The same for a launch that deals its segments to the XCDs: the shares differ by at most 10 % of the mean.
static void walk_dealt(int n, unsigned cols, const uint32_t (&xcd)[kXcds + 1], const std::vector<ItemSeg> &it) {
    std::vector<int> seen((size_t)n * cols, 0);
    long load[kXcds] = {}, total = 0;
    for (unsigned w = 0; w < dealt_grid(xcd, cols); ++w) {
        const unsigned x = w % kXcds, item = w / kXcds, first = xcd[x], m = xcd[x + 1] - first;
        if (item >= m * cols) continue;
        const ItemPos p = column_item_pos(item, m, cols);
        CHECK(p.pos < m && p.cq < cols);
        ++seen[(size_t)(first + p.pos) * cols + p.cq];
        const long cost = std::max((it[first + p.pos].rows + 31) / 32, 3);
        load[x] += cost;
        total += cost;
    }
    for (int v : seen) CHECK(v == 1);
    CHECK(kXcds * *std::max_element(load, load + kXcds) <= total * 1.1);
}

int main() {
    int n_dealt = 0;
    std::srand(5);
    for (int n : {1, 2, 3, 4, 5, 8, 9, 31, 32, 33, 64, 65, 383, 384})
        for (unsigned cols : {1u, 2u, 5u, 7u, 8u, 9u, 10u, 11u, 16u, 31u, 32u, 33u, 64u, 112u, 128u}) {
            for (int most : {1, 3, 40}) {                 // most segments of one expert
                std::vector<Seg> segs;
                for (int e = 0; (int)segs.size() < n && e < kMaxExperts; ++e)
                    for (int c = e == 255 ? 400 : 1 + std::rand() % most; c > 0 && (int)segs.size() < n; --c)
                        segs.push_back(Seg{(uint32_t)segs.size() * 256, (uint16_t)(1 + std::rand() % 256), (uint16_t)e});
                const bool stream = items_stream(segs.data(), n);
                std::vector<ItemSeg> it(n);
                uint32_t xcd[kXcds + 1];
                const bool dealt = plan_items(segs.data(), n, stream, cols, most == 1, it.data(), xcd);
                std::vector<int> taken(n, 0);
                for (int i = 0; i < n; ++i) {
                    const Seg &s = segs[it[i].row0 / 256];
                    CHECK(it[i].rows == s.rows && it[i].expert == s.expert);
                    ++taken[it[i].row0 / 256];
                    const int in = it[i].grp & 15, size = it[i].grp >> 4;
                    CHECK(size >= 1 && size <= kGroupSegs && in < size && i - in >= 0 && i - in + size <= n);
                    CHECK(it[i - in].grp == (size << 4));
                    CHECK(stream || it[i - in].expert == it[i].expert);
                }
                for (int t : taken) CHECK(t == 1);
                if (dealt) {
                    ++n_dealt;
                    CHECK(!stream && xcd[0] == 0 && xcd[kXcds] == n);
                    walk_dealt(n, cols, xcd, it);
                } else {
                    walk(n, cols, [&](unsigned item) {
                        return item_pos(item, cols, [&](unsigned q, unsigned &in, unsigned &size) { in = it[q].grp & 15; size = it[q].grp >> 4; });
                    });
                }
            }
            walk(n, cols, [&](unsigned item) { return column_item_pos(item, (unsigned)n, cols); });
        }
    {   // which launches deal their experts to the XCDs
        auto deals = [](const std::vector<int> &rows, unsigned cols, bool four_bit) {      // one entry per expert
            std::vector<Seg> segs;
            uint32_t row = 0;
            for (size_t e = 0; e < rows.size(); ++e) {
                const int parts = (rows[e] + 255) / 256, tiles = (rows[e] + 31) / 32;
                for (int p = 0, left = rows[e]; p < parts; ++p) {
                    const int take = std::min(left, (tiles / parts + (p < tiles % parts)) * 32);
                    segs.push_back(Seg{row, (uint16_t)take, (uint16_t)e});
                    row += take;
                    left -= take;
                }
            }
            std::vector<ItemSeg> it(segs.size());
            uint32_t xcd[kXcds + 1];
            const bool yes = plan_items(segs.data(), (int)segs.size(), items_stream(segs.data(), (int)segs.size()), cols, four_bit, it.data(), xcd);
            for (int x = 0; yes && x < kXcds; ++x)                                          // an expert is on one XCD
                for (int i = 0; i < (int)it.size(); ++i)
                    for (int j = xcd[x]; j < xcd[x + 1]; ++j)
                        if (it[i].expert == it[j].expert && (i < xcd[x] || i >= xcd[x + 1])) return -1;
            return yes ? 1 : 0;
        };
        const int n = n_dealt, cols = 0;
        CHECK(n_dealt > 50);
        const std::vector<int> two = {402, 380, 385, 370, 391, 384, 377, 373}, even(32, 500);
        const std::vector<int> three = {530, 520, 515, 500, 510, 505, 506, 510}, skewed = {1280, 300, 300, 300, 300, 300, 260, 258};
        CHECK(deals(two, 112, false) == 1 && deals(two, 112, true) == 0 && deals(two, 64, false) == 1);
        CHECK(deals(three, 112, false) == 0 && deals(three, 16, false) == 1 && deals(three, 64, false) == 0);
        CHECK(deals(even, 12, false) == 1 && deals(even, 12, true) == 1);
        CHECK(deals(skewed, 112, false) == 0 && deals(skewed, 16, false) == 0);
        CHECK(deals(std::vector<int>(8, 896), 112, false) == 0 && deals(std::vector<int>(8, 250), 112, false) == 0);
    }
    // pieces of an fp32 launch: never 2^32 threads, and never more pieces than that needs
    for (uint64_t wgs : {uint64_t(1), uint64_t(3), uint64_t(256), uint64_t(512), uint64_t(4096), uint64_t(65535), (uint64_t(1) << 24) - 8}) {
        const int n = 0;
        const unsigned cols = (unsigned)wgs;
        const uint64_t most = segs_per_launch(wgs);
        CHECK(most >= 1 && (most * wgs + 7) * 256 < uint64_t(1) << 32 && (most + 1) * wgs + 8 > uint64_t(1) << 24);
    }
    std::printf("all item checks passed\n");
    return 0;
}
