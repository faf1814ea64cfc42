// Which workgroup of a bf16 expert launch does which (row segment, column tile, K range), as plain
// integer arithmetic shared by the host (plan) and the kernels (decode).
//
// The hardware deals consecutive workgroup ids round-robin to the 8 XCDs, each with its own L2 and its
// own share of the fabric: a launch ends when the XCD with the most work is done.  So the items of a
// launch form one list without holes, in groups of up to kGroupSegs segments.  A group is cut into blocks
// of as many column tiles (K range slowest) as make one item per CU of an XCD, column fastest: a block's
// segments share every weight tile in L2 (when they belong to one expert), its column tiles the token
// tiles.  The list is dealt out in rounds of one item per CU of the chip, 32 consecutive items to each
// XCD, and what is left after the last whole round in 8 equal parts: every XCD gets the same number of
// items and, by the order of the groups (see plan_items), a like mix of long and short ones.
//
// Against packets of 4 segments x 8 column tiles dealt out whether full or not, both with the kernels on 32x32x16 MFMAs (14 half-empty packets
// are 32 workgroups on six XCDs and 16 on two; with 11 column tiles the full packets all fall on even
// XCDs): one token on 2 of 8 experts, H 4096, F 14336: gate-up 92 -> 73 us, layer 190 -> 171 us; 32 tokens
// on 64 experts, H 2048, F 1408: 90 -> 74 us, 170 -> 154 us; 8192 tokens on the same 1.29 -> 1.25 ms.  Where it
// is better that an XCD keeps to its own experts, as with the packets, a launch deals them out (see plan_items).
// Other cuts, measured: a contiguous eighth of the list for each XCD: 8192 tokens on 64 experts +2 %,
// 4-bit decode down projection 48 -> 64 us (four XCDs get all the long segments); eighths of equal cost
// instead of equal count: 3584 tokens on 8 experts +9 % (a few more short items add a round); segments
// fastest inside a block: +2 %.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

#include "qmoe_internal.h"

namespace qmoe {

namespace bf16k {
// Weight formats of the expert matrices: bf16 row-major, bf16 in MFMA-ordered 1 KiB blocks, and
// 4-bit microscaling floats (e2m1 elements, one power-of-two e8m0 scale per 32 elements along K) in
// MFMA-ordered blocks, turned into bf16 operands in registers (exactly: every such value is a bf16).
enum { WF_ROWMAJOR = 0, WF_PACKED = 1, WF_MXFP4 = 2 };
}  // namespace bf16k

constexpr int kXcds = 8;
constexpr int kXcdCus = 32;
constexpr int kGroupSegs = 4;

struct ItemSeg {
    uint32_t row0;
    uint16_t rows;      // 1..256
    uint8_t expert;     // kMaxExperts is 256
    uint8_t grp;        // place in its group (low 4 bits) and size of the group
};
static_assert(kMaxExperts <= 256 && kGroupSegs < 16, "fields of ItemSeg");

// Workgroups of a launch of `items` items, and the item of workgroup `id` (false: none).
__host__ __device__ inline unsigned item_grid(unsigned items) {
    constexpr unsigned R = kXcds * kXcdCus;
    return items / R * R + (items % R + kXcds - 1) / kXcds * kXcds;
}
__host__ __device__ inline bool item_of(unsigned id, unsigned items, unsigned &item) {
    constexpr unsigned R = kXcds * kXcdCus;
    const unsigned full = items / R * R, x = id % kXcds, j = id / kXcds;
    if (id < full) {
        item = j / kXcdCus * R + x * kXcdCus + j % kXcdCus;
        return true;
    }
    const unsigned left = items - full;
    item = full + left * x / kXcds + (j - full / kXcds);
    return item < full + left * (x + 1) / kXcds;
}

// The same of a launch that deals its segments to the XCDs: XCD x has segments xcd[x] .. xcd[x+1] - 1.
__host__ __device__ inline unsigned dealt_grid(const uint32_t (&xcd)[kXcds + 1], unsigned cols) {
    unsigned most = 0;
    for (int x = 0; x < kXcds; ++x) most = most < xcd[x + 1] - xcd[x] ? xcd[x + 1] - xcd[x] : most;
    return kXcds * most * cols;
}

struct ItemPos { unsigned pos, cq; };       // segment in list order; column tile + K range * column tiles

// item of the list -> (segment, column).  cols = column tiles * K ranges; place(pos, in, size) hands back
// the place of a segment in its group and the size of that group.
template <class Place>
__host__ __device__ inline ItemPos item_pos(unsigned item, unsigned cols, Place &&place) {
    const unsigned q = item / cols;         // a segment of the item's group
    unsigned in, size;
    place(q, in, size);
    const unsigned first = q - in, r = item - first * cols;
    const unsigned wide = kXcdCus / size;   // columns of a block
    const unsigned blk = r / (wide * size), rb = r - blk * (wide * size);
    const unsigned left = cols - blk * wide, w = left < wide ? left : wide;
    const unsigned seg = rb / w;
    return {first + seg, blk * wide + (rb - seg * w)};
}

// item -> (segment, column) of n segments in blocks of 8 columns, all segments of a block before the next block.
// For one XCD's share of a launch that deals experts to XCDs (see plan_items), and for launches over n units of the
// device's unit list, more than kMaxSegs of them, which are not sorted by expert.  There blocks of 4 units one after
// the other are no faster or slower: 16384 tokens on 64 experts, H 2048, F 1408, 2.35 ms, skewed 20000 tokens 3.00 ms
// either way, 20000 tokens on 256 experts, F 512, 1.64 ms.
__host__ __device__ inline ItemPos column_item_pos(unsigned item, unsigned n, unsigned cols) {
    constexpr unsigned W = kXcdCus / kGroupSegs;
    const unsigned blk = item / (n * W), r = item - blk * (n * W);
    const unsigned left = cols - blk * W, w = left < W ? left : W;
    const unsigned pos = r / w;
    return {pos, blk * W + (r - pos * w)};
}

// A run of row-adjacent units of one expert, and the segments of at most 256 rows that the runs of a launch are cut into, equal
// within one tile: workgroups that share an expert's weight tiles then advance through K at the same pace and meet in L2, which a
// 256/256/256/128 cut does not give them.
struct Run { uint32_t row0, rows; uint16_t expert; };
// Tiles are of 32 rows, from when the kernels' were.  Up to 8 runs that make two bf16 segments each are cut between fragments of 16
// rows, which makes both nearly equal.  Layer us with 32 / 16, top-2 of 8 experts, H 4096, F 14336, in the common list (see plan_items):
// 1293 tokens 850 / 838, 1400 tokens 905 / 885, 1531 tokens 950 / 927, the last two enqueued in 4 K ranges 961 / 939 and 995 / 986; of 6 experts 1200
// tokens 796 / 784; 4-bit within 1 % either way; with a hot expert 1200 tokens on 6 experts 818 / 810, 1365 on 8 979 / 968, 1500 1144 / 1155.
// With more experts or segments longer and shorter ones mix on an XCD, and it costs up to 1 % (1199 tokens, top-8 of 32, H 2048, F 7040, 846 -> 854).
inline std::vector<Seg> cut_runs(const std::vector<Run> &runs, bool bf16) {
    std::vector<Seg> segs;
    segs.reserve(runs.size() + 8);
    const bool few = runs.size() <= kXcds;
    for (const Run &r : runs) {
        const uint32_t nseg = (r.rows + 255) / 256, tile = nseg == 2 && few && bf16 ? 16 : 32, tiles = (r.rows + tile - 1) / tile;
        const uint32_t base = tiles / nseg, extra = tiles % nseg;
        uint32_t row = r.row0, left = r.rows;
        for (uint32_t j = 0; j < nseg; ++j) {
            const uint32_t want = (base + (j < extra ? 1 : 0)) * tile;
            const uint32_t take = want < left ? want : left;
            segs.push_back(Seg{row, (uint16_t)take, r.expert});
            row += take;
            left -= take;
        }
    }
    return segs;
}

// What a segment costs the XCD that it is dealt to, in fragments of 16 rows, the kernels' unit, whatever it was cut in; up to
// 6 of them it takes as long as its weights.
inline long seg_cost(int rows) { return std::max((rows + 15) / 16, 6); }

// True iff every weight element of the launch is read by one workgroup only: segs are sorted by
// expert and no two belong to the same one.
inline bool items_stream(const Seg *segs, int n) {
    for (int i = 1; i < n; ++i)
        if (segs[i].expert == segs[i - 1].expert) return false;
    return n > 0;
}

// Orders the segments (sorted by expert and row) of one launch into groups.  Where experts have several
// segments a group holds segments of one expert only, the expert with the most rows first, in the common list of bf16 launches
// with most of the experts of one short segment between the others; else the groups are cut from the list sorted by length.
// Returns true if the launch deals its groups to the XCDs: segments xcd[x] .. xcd[x+1] - 1 are XCD x's alone.
// With the common list all XCDs work on the same expert at a time, and its last round is partly filled; an XCD that keeps to
// its own experts fetches fewer tokens for the same columns and ends with them, if the shares (seg_cost, the largest over the
// mean) come out even.  Time dealt out over list, bf16 / 4-bit, shares in brackets; top-2 of 8 experts, H 4096, F 14336 unless stated:
//   less than two rounds of the chip, where the list's last round weighs most: layers whose down projection alone is dealt out, 900 to 1160
//   tokens in 9 to 15 segments (1.04 to 1.14) 0.97 / 0.96 on average, in 2 K ranges 0.96 / 0.95, 1900 to 2080 tokens in 17 to 20 segments (1.04
//   to 1.19) 0.97 / 0.94: up to 1.15;
//   1.5 to 2 segments an expert: 1040 to 1250 tokens in 12 (1.05 to 1.13) 0.96 / 0.92, 13 (1.07 to 1.13) 1.00 / 0.99, 14 (1.04 to 1.16) 0.95 / 0.93
//   and 15 (1.08 to 1.14) 0.97 / 0.97, enqueued in 4 K ranges 1.03 / 0.99, 0.99 / 0.96, 0.95 / 0.93 and 0.98 / 0.97, (1.15 to 1.25) 1.00 / 1.01; 16
//   experts, F 4096 (1.01 to 1.04) 0.96 / 0.93; 64 experts, top-8, H 2048, F 1408 (1.00) 0.96 / 0.97: up to 1.15;
//   fewer: gate-up of 9 (1.10 to 1.14) 1.10 / 1.04 and 10 segments (1.07 to 1.14) 1.02 / 0.98, down projection in 4 K ranges 1.00 / 1.01 and 1.03 / 1.02;
//   16 experts, F 4096 (1.02 to 1.06) 0.98 / 0.93, F 7168 1.02 / 0.97; 32 experts, top-4, H 2048, F 2048 (1.01) 0.95 / 0.92: up to 1.04;
//   two for every expert: 1100 to 1850 tokens whole (up to 1.06) 1.00 / 1.00, (1.06 to 1.12) 1.01 / 1.00, (1.12 to 1.18) 1.02 / 1.02, enqueued 1.01 /
//   1.01, 1.02 / 1.02 and 1.03 / 1.04; 16 experts, F 4096 and 7168 (1.01 to 1.04) 0.96 / 0.98; 32 experts, top-4, H 2048, F 1536 (1.01) 0.95 / 0.96: up to 1.04;
//   more: 2300 to 3000 tokens in 24 and 26 (1.03 to 1.07) 1.01 / 0.99, 3584 in 32 (1.03) 1.01 / 1.00: up to 2.5 an expert and 1.02.
// A hot expert: 1.4 to 1.8 times as long dealt out.
inline bool plan_items(const Seg *segs, int n, bool stream, unsigned cols, bool four_bit, ItemSeg *out, uint32_t (&xcd)[kXcds + 1]) {
    struct Group { int first, count, rows; };
    std::vector<Seg> s(segs, segs + n);
    std::vector<Group> groups;
    if (stream) {
        std::stable_sort(s.begin(), s.end(), [](const Seg &x, const Seg &y) { return x.rows > y.rows; });
        for (int i = 0; i < n; i += kGroupSegs) groups.push_back(Group{i, std::min(kGroupSegs, n - i), 0});
    } else {
        for (int i = 0; i < n;) {
            int j = i, rows = 0;
            while (j < n && s[j].expert == s[i].expert) rows += s[j++].rows;
            const int parts = (j - i + kGroupSegs - 1) / kGroupSegs, base = (j - i) / parts, extra = (j - i) % parts;
            for (int p = 0; p < parts; ++p) {
                const int c = base + (p < extra ? 1 : 0);
                groups.push_back(Group{i, c, rows});
                i += c;
            }
        }
        std::stable_sort(groups.begin(), groups.end(), [](const Group &x, const Group &y) { return x.rows > y.rows; });
    }
    int at = 0;
    auto place = [&](const Group &g) {
        for (int i = 0; i < g.count; ++i) {
            const Seg &v = s[g.first + i];
            out[at++] = ItemSeg{v.row0, v.rows, (uint8_t)v.expert, (uint8_t)(i | g.count << 4)};
        }
    };
    int experts = 1;
    for (int i = 1; i < n; ++i) experts += s[i].expert != s[i - 1].expert;
    if (!stream && 2 * n <= 5 * experts) {
        // each group, the one of the most rows first, to the XCD with the least
        long load[kXcds] = {}, total = 0;
        std::vector<int> owner;
        for (const Group &g : groups) {
            long cost = 0;
            for (int i = 0; i < g.count; ++i) cost += seg_cost(s[g.first + i].rows);
            owner.push_back((int)(std::min_element(load, load + kXcds) - load));
            load[owner.back()] += cost;
            total += cost;
        }
        const long share = 100 * kXcds * *std::max_element(load, load + kXcds);      // of the mean, in percent x total
        const bool below_two_rounds = (unsigned)n * cols < 2 * kXcds * kXcdCus, one_or_two = 2 * n >= 3 * experts && n < 2 * experts;
        if (share <= (below_two_rounds || one_or_two ? 115 : n <= 2 * experts ? 104 : 102) * total) {
            for (int x = 0; x < kXcds; ++x) {
                xcd[x] = (uint32_t)at;
                for (size_t i = 0; i < groups.size(); ++i)
                    if (owner[i] == x) place(groups[i]);
            }
            xcd[kXcds] = (uint32_t)at;
            return true;
        }
    }
    // A workgroup of one of several segments is bound by the matrix units, one of an expert's only segment, where that is short, more by
    // the stream of its weights.  Sorted by rows all of the latter came last, with the matrix units idle; now three quarters of them go out
    // between the others and the rest make the end.  Us a layer sorted / mixed, Zipf-skewed: 4096 tokens on 64 experts, top-8, H 2048, F 1408
    // 657 / 632, 6000 tokens 884 / 874, 8192 tokens 1121 / 1124; 3000 tokens on 16 experts, top-2, F 4096 391 / 379; 4000 tokens on 32, top-4, F 2048
    // 460 / 454; 1500 tokens on 8 experts, H 4096, F 14336 959 / 949.  With half of them between the others the first five 643, 868, 1124,
    // 379, 464, with all of them 644, -, 1126, -, 459.  Least favourable of 14 drawn: 1085 tokens on 32, top-8, H 1664, F 3584 406 / 408.  4-bit weights, a quarter of the bytes, stay sorted (6000 tokens on 64 experts 793 / 796).
    // It costs reads, because a block of columns may now end on another XCD than it began on: gate-up and down sorted / mixed, MB, 8192 tokens on 64
    // experts 2110 / 2620 and 915 / 1000, 4096 tokens 1415 / 1715 and 630 / 720, 3000 on 16 experts, H 4096, 1535 / 1480 and 765 / 805; no launch is
    // bound by them, and 8192 tokens take as long either way.
    // Only segments of experts with one are longer than the others where experts have about 256 rows.  They are not bound by their weights then, and
    // between the others they break blocks that share weights: 1060 tokens on 8 experts 858 / 895, 1130 tokens, enqueued in 4 K ranges
    // 890 / 945, 16 experts, F 7168, 2100 tokens 827 / 848.  By the mean rows of the only segments over those of the others, mixed over sorted of 43
    // bf16 layouts of 8 and 16 experts: up to 0.85 0.991 (0.967 to 1.028), to 1 0.997 (0.973 to 1.033), beyond 1.024 (0.997 to 1.065).
    const size_t heavy = (size_t)(std::find_if(groups.begin(), groups.end(), [](const Group &g) { return g.rows <= 256; }) - groups.begin());
    long all[2] = {0, 0}, rows[2] = {0, 0}, out_segs[2] = {0, 0};       // segments, and their rows, of the groups before and from `heavy` on
    for (size_t i = 0; i < groups.size(); ++i) {
        all[i >= heavy] += groups[i].count;
        for (int j = 0; j < groups[i].count; ++j) rows[i >= heavy] += s[groups[i].first + j].rows;
    }
    if (!stream && !four_bit && rows[1] * all[0] < rows[0] * all[1]) {
        std::vector<Group> mixed;
        for (size_t i = 0, j = heavy; i < heavy || j < groups.size();) {
            const bool light = j < groups.size() && (i == heavy || 4 * (out_segs[1] + groups[j].count) * all[0] <= 3 * out_segs[0] * all[1]);
            mixed.push_back(groups[light ? j++ : i++]);
            out_segs[light] += mixed.back().count;
        }
        groups.swap(mixed);
    }
    for (const Group &g : groups) place(g);
    return false;
}

// Columns per wave of a gate-up launch.  A workgroup stays on its CU for the whole of K, so a launch
// costs whole rounds of the chip's CUs, and a weight-streaming launch moves bytes in proportion to
// rounds x columns per workgroup.  Narrower waves (28 .. 16 columns; a wave's 32 MFMA rows stay, those
// beyond its columns repeat its last one and are dropped) are taken when they make the last round full:
// 8 experts x 14336 columns are 896 workgroups of 128 columns = 3.5 rounds of 256 CUs, but exactly 4
// rounds of 112.  Layer us with 32 / the rule's columns, top-2 of 8 experts, H 4096, F 14336 unless stated (gate-up in brackets):
//   bf16 packed, up to 96 rows: 64 tokens (305) / (299) with 28, 300 tokens 483 (317) / 467 (298) with 28;
//   one round, where narrower waves only put more CUs to work: one token, top-8 of 64, H 2048, F 1408 56.4 (28.4) / 50.8 (22.7) with 16,
//   two 71.6 / 71.0 with 24, one, top-4 of 32, F 1024 47.7 / 42.8 with 16, one on 8 experts 129.3 / 128.0 with 28;
//   row-major, whose lanes read 64 bytes of a row at a time, any number of rows: 400 tokens 776 (508) / 721 (458) with 28, 700 tokens 829 (531) /
//   798 (499), 850 tokens 852 / 832; of widths that cost the same the narrower one up to 96 rows: 20 tokens 616 (383) with 28 / 600 (369) with 16,
//   64 tokens 660 (423) / 629 (394); beyond, 300 tokens with more than 96 rows 706 / 713.
// Not: bf16 packed of more than 96 rows (400 tokens 484 / 481, 430 tokens 487 / 491, 512 tokens 501 / 519, 700 tokens 550 / 578: the rows that
// repeat cost power); 4-bit weights, whose workgroups share a CU and are not bound by bytes (28 columns: 64 tokens, skewed (84) / (94),
// one token 60 / 61; only 4 to 16 tokens gain, 8 tokens 142 / 136); launches whose segments share weights, which are MFMA-bound.
inline int gate_up_wave_columns(bool stream, int wfmt, int tiles, int nseg, int F, long cus) {
    if (!stream || wfmt == bf16k::WF_MXFP4 || (wfmt == bf16k::WF_PACKED && tiles > 3)) return 32;
    const bool narrower = wfmt == bf16k::WF_ROWMAJOR && tiles <= 3;      // of widths that cost the same
    int best = 32;
    long best_cost = 0;
    for (int cw = 32; cw >= 16; cw -= 4) {
        const long wgs = (long)nseg * ((F + 4 * cw - 1) / (4 * cw));
        const long cost = (wgs + cus - 1) / cus * cw;
        if (cw == 32 || cost < best_cost + (narrower ? 1 : 0)) { best = cw; best_cost = cost; }
    }
    return best;
}

}  // namespace qmoe
