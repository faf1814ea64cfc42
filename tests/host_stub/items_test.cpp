// Checks of expert_items.h on the CPU: every (segment, column, K range) of a launch is done by exactly
// one workgroup, the XCDs get equal shares, and a group mixes experts only where no expert repeats;
// and of the pieces a launch is cut into.
#include <cstdio>
#include <cstdlib>
#include <string>
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

// The same for a launch that deals its segments to the XCDs: no share is more than 15 % above the mean.
static void walk_dealt(int n, unsigned cols, const uint32_t (&xcd)[kXcds + 1], const std::vector<ItemSeg> &it) {
    std::vector<int> seen((size_t)n * cols, 0);
    long load[kXcds] = {}, total = 0;
    for (unsigned w = 0; w < dealt_grid(xcd, cols); ++w) {
        const unsigned x = w % kXcds, item = w / kXcds, first = xcd[x], m = xcd[x + 1] - first;
        if (item >= m * cols) continue;
        const ItemPos p = column_item_pos(item, m, cols);
        CHECK(p.pos < m && p.cq < cols);
        ++seen[(size_t)(first + p.pos) * cols + p.cq];
        const long cost = seg_cost(it[first + p.pos].rows);
        load[x] += cost;
        total += cost;
    }
    for (int v : seen) CHECK(v == 1);
    CHECK(kXcds * *std::max_element(load, load + kXcds) <= total * 1.15);
}

// With arguments: the gate-up wave's columns on 256 CUs for each (weight format, 32-row tiles, segments, F) of a launch that streams.
int main(int argc, char **argv) {
    for (int i = 1; i + 3 < argc; i += 4)
        std::printf("%d\n", gate_up_wave_columns(true, std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2]), std::atoi(argv[i + 3]), 256));
    if (argc > 1) return 0;
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
        auto runs_of = [](const std::vector<int> &rows) {                                      // one entry per expert
            std::vector<Run> runs;
            uint32_t row = 0;
            for (size_t e = 0; e < rows.size(); row += (uint32_t)rows[e++]) runs.push_back(Run{row, (uint32_t)rows[e], (uint16_t)e});
            return runs;
        };
        // fine: cut as a bf16 launch is, between fragments of 16 rows where it is of up to 8 experts; else in tiles of 32
        auto deals = [&](const std::vector<int> &rows, unsigned cols, bool four_bit, bool fine = true) {
            const std::vector<Seg> segs = cut_runs(runs_of(rows), fine);
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
        const std::vector<int> ones = {276, 296, 256, 304, 286, 306, 254, 282}, uneven = {227, 300, 284, 280, 353, 304, 233, 279};
        CHECK(deals(two, 112, false) == 0 && deals(two, 112, true) == 0 && deals(two, 64, false) == 0 && deals(two, 16, false) == 1);
        CHECK(deals(ones, 112, false) == 1 && deals(ones, 112, true) == 1 && deals(ones, 64, false) == 1 && deals(uneven, 112, false) == 0);
        CHECK(deals(three, 112, false) == 0 && deals(three, 16, false) == 1 && deals(three, 64, false) == 0);
        CHECK(deals(even, 12, false) == 1 && deals(even, 12, true) == 1);
        CHECK(deals(skewed, 112, false) == 0 && deals(skewed, 16, false) == 0);
        // by segments an expert: 10 segments (share 1.08), 12 (1.13), 16 (1.02)
        const std::vector<int> ten = {224, 244, 239, 261, 236, 250, 258, 248}, twelve = {250, 290, 240, 266, 252, 284, 246, 260}, flat = {382, 380, 385, 384, 390, 384, 377, 383};
        CHECK(deals(ten, 112, false) == 0 && deals(ten, 64, false) == 0 && deals(ten, 16, false) == 1);
        CHECK(deals(twelve, 112, false) == 1 && deals(twelve, 112, true) == 1 && deals(flat, 112, false) == 1 && deals(flat, 112, true) == 1);
        CHECK(deals(even, 12, false, false) == 1);
        CHECK(deals(std::vector<int>(8, 896), 112, false) == 0 && deals(std::vector<int>(8, 250), 112, false) == 0);
    }
    {   // a run costs its fragments however it is cut, so whether a launch is dealt out does not hang on the cut
        int dealt[2] = {0, 0};
        const unsigned cols = 112;
        for (int draw = 0; draw < 4000; ++draw) {
            std::vector<Run> runs;
            uint32_t row = 0;
            const int mean = 255 + draw % 150;
            for (int e = 0; e < 8; ++e) {
                runs.push_back(Run{row, (uint32_t)(mean - 40 + std::rand() % 81), (uint16_t)e});
                row += runs.back().rows;
            }
            long cost[2] = {0, 0};
            bool yes[2];
            for (int fine = 0; fine < 2; ++fine) {
                const std::vector<Seg> segs = cut_runs(runs, fine);
                const int n = (int)segs.size();
                uint32_t at = 0;
                for (const Seg &s : segs) {
                    CHECK(s.row0 == at && s.rows >= 1 && s.rows <= 256);
                    at += s.rows;
                    cost[fine] += seg_cost(s.rows);
                }
                CHECK(at == row);
                std::vector<ItemSeg> it(segs.size());
                uint32_t xcd[kXcds + 1];
                yes[fine] = plan_items(segs.data(), n, items_stream(segs.data(), n), cols, draw % 2, it.data(), xcd);
                dealt[fine] += yes[fine];
            }
            const int n = draw;
            CHECK(cost[0] == cost[1] && yes[0] == yes[1]);
        }
        const int n = dealt[0];
        CHECK(dealt[0] > 400 && dealt[0] < 3600);
    }
    {   // order of the list: 'H' a segment of an expert with several, 'l' the only one of its expert, each kind by falling rows of the expert
        auto order = [](const std::vector<int> &rows, bool four_bit) {
            std::vector<Run> runs;
            uint32_t row = 0;
            for (size_t e = 0; e < rows.size(); row += (uint32_t)rows[e++]) runs.push_back(Run{row, (uint32_t)rows[e], (uint16_t)e});
            const std::vector<Seg> segs = cut_runs(runs, true);
            const int n = (int)segs.size();
            const unsigned cols = 112;
            std::vector<ItemSeg> it(segs.size());
            uint32_t xcd[kXcds + 1];
            CHECK(!plan_items(segs.data(), n, items_stream(segs.data(), n), cols, four_bit, it.data(), xcd));
            std::string kinds;
            int last[2] = {1 << 30, 1 << 30};
            for (const ItemSeg &v : it) {
                const int total = rows[v.expert];
                kinds += total > 256 ? 'H' : 'l';
                CHECK(total <= last[total > 256]);
                last[total > 256] = total;
            }
            return kinds;
        };
        const std::vector<int> skewed = {1500, 20, 90, 10, 60, 1200, 80, 30};       // groups of 3, 3, 3 and 2 segments; of 6 only ones
        // l may be out before h of the 11 where 4 l / 6 <= 3 h / 11: none before 3, 1 before 6, 2 before 9, 3 before the last 2
        const int n = 0;
        const unsigned cols = 0;
        const std::string mixed = order(skewed, false);
        CHECK(mixed == "HHHlHHHlHHHlHHlll");
        CHECK(order(skewed, true) == "HHHHHHHHHHHllllll");                          // 4-bit weights: sorted
        CHECK(order({1500, 1200, 900}, false) == std::string(6 + 5 + 4, 'H'));
        CHECK(order({227, 300, 284, 280, 353, 304, 233, 279}, false) == "HHHHHHHHHHHHll");      // only segments that are the longer ones: last
        CHECK(order({20, 90, 10, 60, 80, 30, 70, 50, 40}, false).find('H') == std::string::npos);
    }
    {   // cuts: two bf16 segments of up to 8 runs between fragments, anything else in tiles of 32
        const int n = 0;
        const unsigned cols = 0;
        auto first = [](int runs, uint32_t rows, bool bf16) {
            std::vector<Run> r;
            for (int e = 0; e < runs; ++e) r.push_back(Run{(uint32_t)e * rows, rows, (uint16_t)e});
            return (int)cut_runs(r, bf16)[0].rows;
        };
        CHECK(first(8, 340, true) == 176 && first(8, 340, false) == 192 && first(9, 340, true) == 192 && first(1, 257, true) == 144);
        CHECK(first(8, 512, true) == 256 && first(8, 256, true) == 256 && first(8, 530, true) == 192);
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
