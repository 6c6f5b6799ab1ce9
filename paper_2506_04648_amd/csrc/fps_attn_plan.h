// The order in which the attention kernels' work items are dealt to an XCD: host plan and its decoding.
#pragma once
#include "fps_internal.h"

namespace fps {

// The order in which an XCD deals its work items where its K and V are about the size of its L2 (plan_items): by
// falling length.  How long an item takes goes by how much of its window the grid's edges leave, a product over the axes.
// Each axis is divided into up to three levels of about equal window length, each the positions between two thresholds
// on both sides of the axis, and the items into sections of one level per axis, dealt one after the other.  In packed
// words: a launch's arguments are written and read over the host's bus (1 KB of them, loosely packed, cost a small call
// 0.7 us).  Not in bytes or halves, which next to words of the same index had the compiler split an address into parts
// that were no multiples of 4, and scalar loads truncate those.
constexpr int kAxisLevels = 3, kMaxSections = kAxisLevels * kAxisLevels * kAxisLevels;
constexpr int kSectionLanes = 32;   // lanes that look a slot's section up
static_assert(kMaxSections <= kSectionLanes, "a lane for the end of each section");
constexpr uint32_t kSectionStart = (1u << 26) - 1;
struct AxisLevel {
    uint32_t first_len1;     // positions first .. first + len1 - 1 (len1 in the upper half),
    uint32_t skip_count;     // and the rest of the count (upper half) `skip` further on
    uint32_t rc;             // reciprocal of the count
    __host__ __device__ static int lower(uint32_t x) { return (int)(x & 0xFFFFu); }
    __host__ __device__ static int upper(uint32_t x) { return (int)(x >> 16); }
};
struct ItemPlan {
    AxisLevel level[3][kAxisLevels];
    // slots of an XCD before the section (kSectionStart behind the end of the last one), and above them its levels along
    // T, H and W, two bits each
    uint32_t section[1 + kSectionLanes];
};

// The item of slot `slot` of XCD `xcd`, which lies in section `sec`: query block jq of tile (ut, uh, uw) of head bh.  P: an
// ItemPlan, in whatever address space.
template <typename P>
__host__ __device__ inline bool planned_item(const P& p, const Geom& g, int qblocks, uint32_t rc_qblocks, int xcd, int slot,
                                             int sec, int* bh, int* ut, int* uh, int* uw, int* jq) {
    const uint32_t word = p.section[sec];
    const int start = (int)(word & kSectionStart), per = (int)(p.section[sec + 1] & kSectionStart) - start;
    const auto &t = p.level[0][(word >> 26) & 3], &h = p.level[1][(word >> 28) & 3], &w = p.level[2][word >> 30];
    const int nt = AxisLevel::upper(t.skip_count), nh = AxisLevel::upper(h.skip_count), nw = AxisLevel::upper(w.skip_count);
    const int item = xcd * per + slot - start;
    if (item >= g.BH * nt * nh * nw * qblocks) return false;
    const int tile = quotient(item, qblocks, rc_qblocks), row = quotient(tile, nw, w.rc), layer = quotient(row, nh, h.rc);
    auto position = [](const auto& l, int i) {
        return AxisLevel::lower(l.first_len1) + i + (i >= AxisLevel::upper(l.first_len1) ? AxisLevel::lower(l.skip_count) : 0);
    };
    *jq = item - tile * qblocks;
    *bh = quotient(layer, nt, t.rc);
    *uw = position(w, tile - row * nw);
    *uh = position(h, row - layer * nh);
    *ut = position(t, layer - *bh * nt);
    return true;
}

// One axis of n tiles: the levels of its positions by the tokens in their windows, at least
// 90, 72 and 0 % of the most.  That number rises along the axis, stays and falls, so the positions above a
// threshold are a range.
inline int plan_axis(int n, int tile, int size, int r, bool shift, AxisLevel* level, long long* tokens) {
    auto in_window = [&](int u) {
        if (shift) u = n > 2 * r + 1 ? (u < r ? r : u > n - 1 - r ? n - 1 - r : u) : n / 2;
        const int lo = u > r ? u - r : 0, hi = u < n - 1 - r ? u + r : n - 1;
        return (long long)(hi == n - 1 ? size : (hi + 1) * tile) - (long long)lo * tile;
    };
    const int top = r < n - 1 ? r : n - 1;                 // a position of the most
    static const int percent[kAxisLevels] = {90, 72, 0};
    int levels = 0, lo = top, hi = top - 1;                // the range so far: lo .. hi, empty
    for (int k = 0; k < kAxisLevels; ++k) {
        const long long bound = in_window(top) * percent[k];
        auto above = [&](int u) { return 100 * in_window(u) >= bound; };
        int a = 0, b = lo;                                 // first position above
        while (a < b) { const int m = a + (b - a) / 2; if (above(m)) b = m; else a = m + 1; }
        const int first = a;
        a = hi < top ? top : hi; b = n - 1;                // last one
        while (a < b) { const int m = b - (b - a) / 2; if (above(m)) a = m; else b = m - 1; }
        const int last = a;
        const int left = lo - first, right = last - hi;
        if (left + right == 0) continue;
        const int start = left ? first : hi + 1, len1 = left ? left : right, skip = left && right ? hi + 1 - lo : 0,
                  count = left + right;
        level[levels] = AxisLevel{(uint32_t)(start | len1 << 16), (uint32_t)(skip | count << 16), reciprocal(count)};
        tokens[levels++] = in_window(count > 1 && len1 > count / 2 ? start + count / 2 : start);
        lo = first;
        hi = last;
    }
    return levels;
}

// Plans a launch of g.BH * g.M * qblocks work items of `waves` waves; returns the slots of an XCD, or 0: raster order.
//
// Dealt by falling length where there are more workgroups than CUs and an XCD's share of K and V is at most 8 MB (L2: 4).
// In raster order the launch waits for engines whose turn it is while others are free, and ends with whatever comes last.
// Attention, raster order against this, us:
//                                           K and V, an XCD's share
//   24 x 10x26x36 tokens, window 7x3x5                       7.2 MB   434 -> 404
//   7 x 12x40x48, tile (4,8,8), window 5x5x7                 4.9      498 -> 453
//   11 x 7x32x48, window 3x7x3                               3.6      118 -> 92.9
//   40 x 10x12x10, tile (2,8,16)                             3.5      66.5 -> 54.2
//   10 x 10x13x22, tile (6,8,8), BF16                        3.0      56.0 -> 47.6
//   11 x 6x21x20, window 5x1x1                               0.8      22.5 -> 20.1
// of 22 random calls of up to 8 MB the median gains 3 %.  More K and V lose by the order's wider reach -- several heads, or four
// layers of tiles along T and their windows at a time instead of two -- about what it gives or more:
//   18 x 6x56x64, tile (2,8,16), window 4x5x1               11.8      273 -> 277
//   12 x 21x30x52                                           12.9      316 -> 331    BF16 492 -> 565
//   40 x 21x45x80, window 7x5x5                            103      11660 -> 12780
// (By length within each layer only, those gain a per cent at best, 3733 -> 3701 with window 5x3x3, and lose as often, tile
// (6,8,8) 292 -> 308.)  One-wave workgroups that are all resident at once, eight a CU, do better spread as they come: 672
// items of up to 35 blocks 36.8 -> 39.5.
constexpr long long kPlannedKeyBytes = 64 << 20;
inline int plan_items(const Geom& g, const int (&radius)[3], bool shift, int qblocks, int waves, int row_bytes,
                      ItemPlan& p) {
    if (2LL * g.BH * g.M * g.TSP * row_bytes > kPlannedKeyBytes) return 0;
    const long long items = (long long)g.BH * g.M * qblocks;
    if (items <= (waves == 1 ? 2048 : 256) || items > (1 << 28)) return 0;
    if (g.nT > 0xFFFF || g.nH > 0xFFFF || g.nW > 0xFFFF) return 0;   // AxisLevel has 16 bits for them
    const int n_tiles[3] = {g.nT, g.nH, g.nW}, tile[3] = {g.Tt, g.Th, g.Tw}, size[3] = {g.T, g.H, g.W};
    long long tokens[3][kAxisLevels];
    int n[3];
    for (int i = 0; i < 3; ++i) n[i] = plan_axis(n_tiles[i], tile[i], size[i], radius[i], shift, p.level[i], tokens[i]);
    double length[kMaxSections];
    int sections = 0;
    for (int t = 0; t < n[0]; ++t)
        for (int h = 0; h < n[1]; ++h)
            for (int w = 0; w < n[2]; ++w) {
                const double len = (double)tokens[0][t] * (double)tokens[1][h] * (double)tokens[2][w];
                int i = sections++;                        // insertion sort, longest first
                for (; i > 0 && length[i - 1] < len; --i) {
                    length[i] = length[i - 1];
                    p.section[i] = p.section[i - 1];
                }
                length[i] = len;
                p.section[i] = (uint32_t)(t | h << 2 | w << 4) << 26;
            }
    int slots = 0;
    for (int s = 0; s < sections; ++s) {
        const uint32_t word = p.section[s];
        p.section[s] = word | (uint32_t)slots;
        slots += (g.BH * AxisLevel::upper(p.level[0][(word >> 26) & 3].skip_count) *
                      AxisLevel::upper(p.level[1][(word >> 28) & 3].skip_count) *
                      AxisLevel::upper(p.level[2][word >> 30].skip_count) * qblocks + 7) / 8;
    }
    p.section[sections] = (uint32_t)slots;
    for (int s = sections + 1; s <= kSectionLanes; ++s) p.section[s] = kSectionStart;
    return slots;
}

}  // namespace fps
