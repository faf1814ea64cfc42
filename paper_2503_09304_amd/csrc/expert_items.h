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
// Against packets of 4 segments x 8 column tiles dealt out whether full or not (14 half-empty packets
// are 32 workgroups on six XCDs and 16 on two; with 11 column tiles the full packets all fall on even
// XCDs): one token on 2 of 8 experts, H 4096, F 14336: gate-up 92 -> 73 us, layer 190 -> 171 us; 32 tokens
// on 64 experts, H 2048, F 1408: 90 -> 74 us, 170 -> 154 us; 8192 tokens on the same 1.29 -> 1.265 ms; launches
// that filled their packets are unchanged.
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

// item -> (unit, column) of a launch over n units of the device's unit list, in groups of kGroupSegs
// consecutive units.  The host does not know the units' rows here and cannot sort them, so the list goes
// by blocks of 8 columns, all units of a block before the next block: long and short units stay mixed to
// the end of the launch, and with 4 groups each XCD keeps to the token tiles of one.  Measured on 1531
// tokens, 8 experts (16 units of 256 and 127 rows, 4 K ranges) enqueued as one launch, us a layer: group by
// group 1146 against 1134 with the packets; by blocks 1147 and 1142 against 1143 and 1145 with the packets.
__host__ __device__ inline ItemPos unit_item_pos(unsigned item, unsigned n, unsigned cols) {
    constexpr unsigned W = kXcdCus / kGroupSegs;
    const unsigned blk = item / (n * W), r = item - blk * (n * W);
    const unsigned left = cols - blk * W, w = left < W ? left : W;
    const unsigned first = r / (w * kGroupSegs) * kGroupSegs, rb = r - first * w;
    const unsigned seg = rb / w;
    return {first + seg, blk * W + (rb - seg * w)};
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
inline void plan_items(const Seg *segs, int n, bool stream, ItemSeg *out) {
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
    for (const Group &g : groups)
        for (int i = 0; i < g.count; ++i) {
            const Seg &v = s[g.first + i];
            out[at++] = ItemSeg{v.row0, v.rows, (uint8_t)v.expert, (uint8_t)(i | g.count << 4)};
        }
}

}  // namespace qmoe
