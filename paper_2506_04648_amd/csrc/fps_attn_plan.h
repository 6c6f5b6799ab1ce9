// The order in which the attention kernels' work items are dealt to an XCD: host plan and its decoding.
#pragma once
#include "fps_internal.h"

namespace fps {

// The order in which an XCD deals its work items where its K and V are about the size of its L2 (plan_items), and its
// last ones where they are not (plan_tail): by falling length.  How long an item takes goes by how much of its window the
// grid's edges leave, a product over the axes.  Each axis is divided into up to three levels of about equal window length,
// each the positions between two thresholds on both sides of the axis, and the items into sections of one level per axis,
// dealt one after the other.  In packed words: a launch's arguments are written and read over the host's bus (1 KB of
// them, loosely packed, cost a small call 0.7 us).  Not in bytes or halves, which next to words of the same index had the
// compiler split an address into parts that were no multiples of 4, and scalar loads truncate those.
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

// position i of a level; L: an AxisLevel, in whatever address space
template <typename L>
__host__ __device__ inline int level_position(const L& l, int i) {
    return AxisLevel::lower(l.first_len1) + i + (i >= AxisLevel::upper(l.first_len1) ? AxisLevel::lower(l.skip_count) : 0);
}

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
    *jq = item - tile * qblocks;
    *bh = quotient(layer, nt, t.rc);
    *uw = level_position(w, tile - row * nw);
    *uh = level_position(h, row - layer * nh);
    *ut = level_position(t, layer - *bh * nt);
    return true;
}

// Slot `slot` of an XCD's tail (plan_tail), which lies in section `sec`: the item, counted in raster order.  The tail is the
// items from `base` on, as many as some layers of tiles have, but not from the start of a layer.
template <typename P>
__host__ __device__ inline int tail_item(const P& p, const Geom& g, int qblocks, uint32_t rc_qblocks, int base, int slot,
                                         int sec) {
    const uint32_t word = p.section[sec];
    const auto &h = p.level[1][(word >> 28) & 3], &w = p.level[2][word >> 30];
    const int nh = AxisLevel::upper(h.skip_count), nw = AxisLevel::upper(w.skip_count);
    const int i = slot - (int)(word & kSectionStart);
    const int tile = quotient(i, qblocks, rc_qblocks), row = quotient(tile, nw, w.rc), layer = quotient(row, nh, h.rc);
    const int layer_items = g.nH * g.nW * qblocks;
    const int in_layer = (level_position(h, row - layer * nh) * g.nW + level_position(w, tile - row * nw)) * qblocks +
                         i - tile * qblocks;
    const int ahead = in_layer - (base - quotient(quotient(base, qblocks, rc_qblocks), g.nH * g.nW, g.rc_layer) * layer_items);
    return base + layer * layer_items + (ahead < 0 ? ahead + layer_items : ahead);
}

// Tokens along an axis of n tiles in the window of position u.
inline long long tokens_in_window(int u, int n, int tile, int size, int r, bool shift) {
    if (shift) u = n > 2 * r + 1 ? (u < r ? r : u > n - 1 - r ? n - 1 - r : u) : n / 2;
    const int lo = u > r ? u - r : 0, hi = u < n - 1 - r ? u + r : n - 1;
    return (long long)(hi == n - 1 ? size : (hi + 1) * tile) - (long long)lo * tile;
}

// Tokens in the fullest window over their mean.
inline double longest_over_mean(const Geom& g, const int (&radius)[3], bool shift) {
    const int n[3] = {g.nT, g.nH, g.nW}, tile[3] = {g.Tt, g.Th, g.Tw}, size[3] = {g.T, g.H, g.W};
    double ratio = 1;
    for (int i = 0; i < 3; ++i) {
        long long sum = 0, most = 0;
        for (int u = 0; u < n[i]; ++u) {
            const long long x = tokens_in_window(u, n[i], tile[i], size[i], radius[i], shift);
            sum += x;
            most = x > most ? x : most;
        }
        ratio *= (double)most * n[i] / (double)sum;
    }
    return ratio;
}

// One axis of n tiles: the levels of its positions by the tokens in their windows, at least
// 90, 72 and 0 % of the most.  That number rises along the axis, stays and falls, so the positions above a
// threshold are a range.
inline int plan_axis(int n, int tile, int size, int r, bool shift, AxisLevel* level, long long* tokens) {
    auto in_window = [&](int u) { return tokens_in_window(u, n, tile, size, r, shift); };
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

// The sections of the levels n[0] x n[1] x n[2], the longest items first, their starts not yet filled in; returns their
// number.  *spread: length of the longest items over the mean.
inline int sort_sections(const int (&n)[3], const long long (&tokens)[3][kAxisLevels], ItemPlan& p, double* spread) {
    double length[kMaxSections], all = 0, items = 0;
    int sections = 0;
    for (int t = 0; t < n[0]; ++t)
        for (int h = 0; h < n[1]; ++h)
            for (int w = 0; w < n[2]; ++w) {
                const double len = (double)tokens[0][t] * (double)tokens[1][h] * (double)tokens[2][w];
                const double count = (double)AxisLevel::upper(p.level[0][t].skip_count) *
                                     AxisLevel::upper(p.level[1][h].skip_count) * AxisLevel::upper(p.level[2][w].skip_count);
                all += len * count;
                items += count;
                int i = sections++;                        // insertion sort
                for (; i > 0 && length[i - 1] < len; --i) {
                    length[i] = length[i - 1];
                    p.section[i] = p.section[i - 1];
                }
                length[i] = len;
                p.section[i] = (uint32_t)(t | h << 2 | w << 4) << 26;
            }
    *spread = length[0] * items / all;
    return sections;
}

// Plans a launch of g.BH * g.M * qblocks work items of `waves` waves, the longest walk `blocks` key blocks; returns the
// slots of an XCD, a multiple of four, or 0: raster order.
//
// In raster order the launch waits for engines whose turn it is while others are free, and ends with whatever comes last.
// By falling length it loses some of what neighbours share in the L2, and a little for looking up the plan.  So dealt
// where there are more workgroups than CUs, the longest walk is of 12 blocks or more and 1.1 times the mean, and an XCD's
// share of K and V is at most 8 MB of packed slots (L2: 4).  Attention, time against raster order, 510 random calls of up
// to 8 MB and 257 to 5000 items of twelve tilings, both precisions:
//   longest / mean >= 1.1, blocks     1-3     4-7     8-11    12-15   16-31   32 and more
//     mean                            0.95    0.95    0.97    0.93    0.90    0.87
//     slower by 2 %, of calls         5/14    6/27    6/27    5/38    3/91    5/144
//   blocks >= 12, longest / mean      <1.05   <1.1    <1.2    <1.3    <1.5    more
//     mean                            1.00    0.98    0.91    0.90    0.88    0.87
//     slower by 2 %, of calls         3/110   5/37    5/57    1/65    3/79    4/72
// The slowest call outside the rule takes 1.27 of raster order's time, the slowest inside 1.10.  Beyond 8 MB, same rule
// otherwise, 97 random calls: 7 to 9 MB 0.96, to 12 MB 0.93, to 16 MB 0.96, to 25 MB 0.98; but us
//   12 x 21x30x52, window 3x3x3, tile (1,8,16)       15.8 MB   310 -> 320    BF16 (31.5 MB) 495 -> 540
//   12 x 21x30x52, window 3x5x7, tile (3,4,4)        17.1      770 -> 821
//   40 x 21x45x80, window 7x5x5, tile (1,8,16)       98.4      11.21 -> 11.23 ms
// (By length within each layer only, those gain a per cent at best and lose as often.)  One-wave workgroups that are all
// resident at once, eight a CU, are left in raster order; 58 random calls of up to 400 items took 0.94 of its time by
// length, up to 1024 1.00 (one in eight 2 to 10 % more) and up to 2048 0.91.
// Levels at 95 and 85 % instead of 90 and 72: 122 calls 0.91 instead of 0.89; at 80 and 50 %: 0.89, the slowest 1.23.
constexpr int kPlannedBlocks = 12;
constexpr long long kPlannedKeyBytes = 64 << 20;
inline int plan_items(const Geom& g, const int (&radius)[3], bool shift, int qblocks, int waves, int row_bytes, int blocks,
                      ItemPlan& p) {
    if (blocks < kPlannedBlocks) return 0;
    if (2LL * g.BH * g.M * g.TSP * row_bytes > kPlannedKeyBytes) return 0;
    const long long items = (long long)g.BH * g.M * qblocks;
    if (items <= (waves == 1 ? 2048 : 256) || items > (1 << 28)) return 0;
    if (g.nT > 0xFFFF || g.nH > 0xFFFF || g.nW > 0xFFFF) return 0;   // AxisLevel has 16 bits for them
    const int n_tiles[3] = {g.nT, g.nH, g.nW}, tile[3] = {g.Tt, g.Th, g.Tw}, size[3] = {g.T, g.H, g.W};
    long long tokens[3][kAxisLevels];
    int n[3];
    for (int i = 0; i < 3; ++i) n[i] = plan_axis(n_tiles[i], tile[i], size[i], radius[i], shift, p.level[i], tokens[i]);
    double spread;
    const int sections = sort_sections(n, tokens, p, &spread);
    if (spread < 1.1) return 0;                            // about all of one length
    int slots = 0;
    for (int s = 0; s < sections; ++s) {
        const uint32_t word = p.section[s];
        p.section[s] = word | (uint32_t)slots;
        slots += (g.BH * AxisLevel::upper(p.level[0][(word >> 26) & 3].skip_count) *
                      AxisLevel::upper(p.level[1][(word >> 28) & 3].skip_count) *
                      AxisLevel::upper(p.level[2][word >> 30].skip_count) * qblocks + 7) / 8;
    }
    slots = (slots + 3) / 4 * 4;                           // as the turning order wants them
    p.section[sections] = (uint32_t)slots;
    for (int s = sections + 1; s <= kSectionLanes; ++s) p.section[s] = kSectionStart;
    return slots;
}

// Launches whose K and V are beyond that: raster order, but for the end.  An XCD's last items, as many layers of tiles as make
// up one or two rounds of the workgroups that it holds at once (8 waves a CU), are dealt by falling length within the layer,
// so that the launch does not end with long items alone on their CUs; the window of those few layers stays in the L2.  Returns
// the first slot of an XCD so dealt, or -1: none.  Items of a layer must differ in length and walks be long, as in plan_items.
// Attention, us, raster order against this (FP8 two rounds, BF16, whose keys take twice the bytes, one):
//   12 x 21x30x52, window 3x3x3, tile (1,8,16)    FP8 308 -> 296, 308 -> 295      BF16 489 -> 483, 483 -> 476
//   12 x 21x30x52, window 3x5x7, tile (3,4,4)     765 -> 758, 759 -> 749
//   40 x 21x45x80, window 5x3x3, tile (1,8,16)    3838 -> 3822, 3794 -> 3771
// (calls back to back on two boxes; what the whole calls gain is the same).  1736 random calls of both precisions: mean 0.989,
// 17 slower by 2 %, the slowest 1.04.  One round in FP8 0.991; two in BF16 0.991 but the slowest 1.09, three 1.23.
inline int plan_tail(const Geom& g, const int (&radius)[3], bool shift, int qblocks, int waves, int row_bytes, int blocks,
                     int chunk, ItemPlan& p) {
    if (blocks < kPlannedBlocks || g.nH > 0xFFFF || g.nW > 0xFFFF) return -1;
    const int round = 32 * (8 / waves), wanted = (row_bytes > 128 ? 1 : 2) * round;
    const long long layer = (long long)g.nH * g.nW * qblocks;
    if (chunk <= round || layer > chunk || layer > wanted || chunk > 1 << 25) return -1;
    const long long fill = (wanted + layer - 1) / layer;
    const int layers = (int)(fill * layer > chunk ? chunk / layer : fill);
    const int n_tiles[3] = {0, g.nH, g.nW}, tile[3] = {0, g.Th, g.Tw}, size[3] = {0, g.H, g.W};
    long long tokens[3][kAxisLevels] = {{1}};
    int n[3] = {1};                                        // the layers are taken to be alike
    p.level[0][0] = AxisLevel{(uint32_t)layers << 16, (uint32_t)layers << 16, reciprocal(layers)};
    for (int i = 1; i < 3; ++i) n[i] = plan_axis(n_tiles[i], tile[i], size[i], radius[i], shift, p.level[i], tokens[i]);
    double spread;
    const int sections = sort_sections(n, tokens, p, &spread);
    if (spread < 1.1) return -1;
    const int first = chunk - layers * (int)layer;
    int slots = first;
    for (int s = 0; s < sections; ++s) {
        const uint32_t word = p.section[s];
        p.section[s] = word | (uint32_t)slots;
        slots += layers * AxisLevel::upper(p.level[1][(word >> 28) & 3].skip_count) *
                 AxisLevel::upper(p.level[2][word >> 30].skip_count) * qblocks;
    }
    for (int s = sections; s <= kSectionLanes; ++s) p.section[s] = kSectionStart;
    return first;
}

}  // namespace fps
