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
// items and, the groups being sorted longest first, a like mix of long and short ones.
//
// Against packets of 4 segments x 8 column tiles dealt out whether full or not, both with the kernels on 32x32x16 MFMAs (14 half-empty packets
// are 32 workgroups on six XCDs and 16 on two; with 11 column tiles the full packets all fall on even
// XCDs): one token on 2 of 8 experts, H 4096, F 14336: gate-up 92 -> 73 us, layer 190 -> 171 us; 32 tokens
// on 64 experts, H 2048, F 1408: 90 -> 74 us, 170 -> 154 us; 8192 tokens on the same 1.29 -> 1.25 ms.  Where the
// packets kept an XCD to one expert of two segments the list was slower, by 1 % for 1531 tokens on 8 experts to 6 %
// for 2048: those launches deal their experts out (see plan_items).
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

// True iff every weight element of the launch is read by one workgroup only: segs are sorted by
// expert and no two belong to the same one.
inline bool items_stream(const Seg *segs, int n) {
    for (int i = 1; i < n; ++i)
        if (segs[i].expert == segs[i - 1].expert) return false;
    return n > 0;
}

// Orders the segments (sorted by expert and row) of one launch into groups.  Where experts have several
// segments a group holds segments of one expert only, the expert with the most rows first; else the
// groups are cut from the list sorted by length.
// Returns true if the launch deals its groups to the XCDs: segments xcd[x] .. xcd[x+1] - 1 are XCD x's alone.
// With the common list all XCDs work on the same expert at a time; where an expert has few segments, an XCD that
// keeps to its own experts fetches fewer tokens for the same columns, if the shares (their cost in token tiles, the
// largest over the mean) come out even.  Us a layer (gate-up + down) with the list / dealt out, top-2 of 8 experts, H 4096,
// F 14336 unless stated:
//   32 experts, top-4, H 2048, F 1536, 4000 tokens (share 1.01) 388 (203 + 143) / 367 (198 + 131), 4-bit weights 335 (175 + 114) /
//   324 (168 + 112); 64 experts, top-8, H 2048, F 1408, 4-bit, 3000 tokens, skewed 461 (252 + 155) / 446 (250 + 143): dealt
//   out up to 1.02;
//   two segments per expert: 1100 tokens (1.10) 884 (531 + 350) / 857 (500 + 343), 1300 tokens (1.02) 940 (607 + 321) / 921 (584 +
//   319), 1531 tokens (1.05) 1047 (684 + 356) / 1027 (651 + 359), enqueued 1121 (684 + 384) / 1091 (660 + 374): dealt out up to
//   1.10, except for 4-bit weights (1531 tokens 837 (561 + 281) / 846 (572 + 284));
//   2048 tokens, two or three segments (1.03), down projection 604 / 547: its 320 items are 1.25 rounds of the chip, and
//   the list's last quarter takes as long as a round: dealt out below two rounds up to 1.10; gate-up, 7 rounds, 824 / 873, and
//   with 4 K ranges, 5 rounds, 455 / 485: the list.
// Uneven shares lose: 1300 tokens, skewed (2.5) 975 with the list / 1631.  So do more segments per expert, even
// shares or not: 2500 tokens (3 segments, 1.05) 1624 / 1667, 3584 tokens, 4-bit (4 segments, 1.02) 1812 / 1826.
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
        // each group, the one of the most rows first, to the XCD with the least; up to 3 token tiles a segment takes
        // as long as its weights
        long load[kXcds] = {}, total = 0;
        std::vector<int> owner;
        for (const Group &g : groups) {
            long cost = 0;
            for (int i = 0; i < g.count; ++i) cost += std::max((s[g.first + i].rows + 31) / 32, 3);
            owner.push_back((int)(std::min_element(load, load + kXcds) - load));
            load[owner.back()] += cost;
            total += cost;
        }
        const long share = 100 * kXcds * *std::max_element(load, load + kXcds);      // of the mean, in percent x total
        const bool few = (!four_bit && n <= 2 * experts) || (unsigned)n * cols < 2 * kXcds * kXcdCus;
        if (share <= (few ? 110 : 102) * total) {
            for (int x = 0; x < kXcds; ++x) {
                xcd[x] = (uint32_t)at;
                for (size_t i = 0; i < groups.size(); ++i)
                    if (owner[i] == x) place(groups[i]);
            }
            xcd[kXcds] = (uint32_t)at;
            return true;
        }
    }
    // A workgroup of one of several segments is bound by the matrix units, one of an expert's only segment more by the stream of its
    // weights.  Sorted by rows all of the latter came last, with the matrix units idle; now three quarters of them go out between the others
    // and the rest make the end.  Us a layer sorted / mixed, Zipf-skewed: 4096 tokens on 64 experts, top-8, H 2048, F 1408 657 / 632, 6000
    // tokens 884 / 874, 8192 tokens 1121 / 1124; 3000 tokens on 16 experts, top-2, F 4096 391 / 379; 4000 tokens on 32, top-4, F 2048
    // 460 / 454; 1500 tokens on 8 experts, H 4096, F 14336 959 / 949.  With half of them between the others the first five 643, 868, 1124,
    // 379, 464, with all of them 644, -, 1126, -, 459.  Least favourable of 14 drawn: 1085 tokens on 32, top-8, H 1664, F 3584 406 / 408.  4-bit weights, a quarter of the bytes, stay sorted (6000 tokens on 64 experts 793 / 796).
    if (!stream && !four_bit) {
        std::vector<Group> mixed;
        const size_t heavy = (size_t)(std::find_if(groups.begin(), groups.end(), [](const Group &g) { return g.rows <= 256; }) - groups.begin());
        long all[2] = {0, 0}, out_segs[2] = {0, 0};                 // segments of the groups before and from `heavy` on
        for (size_t i = 0; i < groups.size(); ++i) all[i >= heavy] += groups[i].count;
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

}  // namespace qmoe
