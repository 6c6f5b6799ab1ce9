"""CPU checks of host rules of the kernel sources, compiled here without a GPU: which attention launches
split their keys or deal their items in turns, and division by a stored reciprocal."""
import os
import random
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "fps_attn_device.h"
#include <cstdio>
#include <cstring>
using namespace fps;
int main(int argc, char**) {
    // with an argument: windows of 1 or 3 x span x 1 tiles, each of 1 to 4 scale groups of 32 or 64 tokens
    for (int span = 1; span <= 9 && argc > 1; span += 2)
        for (int i = 0; i < 8; ++i) {
            const int ns = 1 + i / 2;
            AttnArgs a;
            std::memset(&a, 0, sizeof(a));
            a.g.BS = 32; a.g.KBS = 1 + i % 2; a.g.KBG = 1; a.g.NS = ns; a.g.TSP = 32 * a.g.KBS * ns;
            a.g.nT = 3; a.g.nH = 100; a.g.nW = 1;
            a.rt = span > 1; a.rh = (span - 1) / 2;
            std::printf("%d %d %d\n", query_waves(a.g), window_blocks(a), (int)blocks_together(a));
        }
    if (argc > 1) return 0;
    // a tile of `tokens` in one scale group, `items` work items, a window of `blocks` tiles
    int tokens, items, blocks, ks;
    while (std::scanf("%d %d %d %d", &tokens, &items, &blocks, &ks) == 4) {
        AttnArgs a;
        std::memset(&a, 0, sizeof(a));
        a.g.BS = tokens <= 96 ? 32 : 128;
        a.g.KBS = a.g.KB = (tokens + a.g.BS - 1) / a.g.BS;
        a.g.KBG = a.g.BS == 128 ? a.g.KBS : 1;
        a.g.NS = 1;
        a.g.TSP = a.g.KB * a.g.BS;
        a.g.nT = blocks; a.g.nH = a.g.nW = 1;
        a.rt = blocks;
        a.total = items;
        std::printf("%d %d\n", query_waves(a.g), (int)split_keys(a, ks));
    }
    for (int row = 1; row <= 20; ++row) std::printf("%d", (int)deal_in_turns(row));
    std::printf("\n");
    unsigned bad = 0;
    for (int d : {1, 2, 3, 5, 7, 10, 12, 630, 3024, 65535, 1 << 20}) {
        const uint32_t m = reciprocal(d);
        for (long long k = 0; k < 2000; ++k)                 // n to either side of the multiples of d below 2^30
            for (int o = -1; o <= 1; ++o) {
                const long long n = ((1LL << 30) / d * k / 1999) * d + o;
                if (n >= 0 && n < (1LL << 30)) bad += quotient((int)n, d, m) != n / d;
            }
    }
    std::printf("bad quotients %u\n", bad);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.hip", d / "rules"
    src.write_text(PROGRAM)
    res = subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-I" + os.path.join(ROOT, "include"),
                          "-I" + os.path.join(ROOT, "paper_2506_04648_amd", "csrc"), str(src), "-o", str(exe)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return str(exe)


# tokens of a tile, work items, key blocks of the window, wave groups -> waves of a workgroup without them, split
RULES = [
    (128, 256, 27, 2, 4, True), (128, 257, 27, 2, 4, False),        # 8 waves a workgroup: one a CU
    (77, 256, 27, 2, 3, True), (77, 257, 27, 2, 3, False), (77, 341, 27, 2, 3, False),   # 6 waves: still one a CU
    (48, 256, 27, 4, 2, True), (48, 257, 27, 4, 2, False),          # 8 waves
    (32, 512, 27, 4, 1, True), (32, 513, 27, 4, 1, False),          # 4 waves: two a CU
    (128, 64, 6, 2, 4, True), (128, 64, 5, 2, 4, False),            # two groups: at least three blocks each
    (32, 64, 8, 4, 1, True), (32, 64, 7, 4, 1, False),              # four groups: two each
]


def test_keys_are_split_where_all_workgroups_are_resident_at_once(program):
    lines = "\n".join(" ".join(map(str, r[:4])) for r in RULES)
    out = subprocess.run([program], input=lines, capture_output=True, text=True, check=True).stdout.splitlines()
    got = [tuple(map(int, line.split())) for line in out[:-2]]
    assert got == [(r[4], int(r[5])) for r in RULES]


def test_items_of_rows_of_six_or_ten_are_dealt_in_order(program):
    out = subprocess.run([program], input="", capture_output=True, text=True, check=True).stdout.splitlines()
    assert [i + 1 for i, c in enumerate(out[-2]) if c == "1"] == [2, 4, 8, 12, 16, 20]


def test_blocks_are_taken_together_on_long_walks(program):
    """Shorter walks are slower so: up to 25 blocks in workgroups of fewer than four waves, up to 3 in others."""
    out = subprocess.run([program, "together"], capture_output=True, text=True, check=True).stdout
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert {(1, b) for b in (1, 2, 3, 9, 15, 18, 21, 27, 30)} <= {r[:2] for r in rows}
    assert {(4, b) for b in (2, 4, 18, 36)} <= {r[:2] for r in rows}
    for waves, blocks, together in rows:
        assert together == (blocks > (3 if waves == 4 else 25)), (waves, blocks)


def test_quotients_by_a_stored_reciprocal_are_exact(program):
    out = subprocess.run([program], input="", capture_output=True, text=True, check=True).stdout
    assert out.splitlines()[-1] == "bad quotients 0"


PLAN_PROGRAM = r"""
#include "fps_attn_plan.h"
#include <cstdio>
#include <cstring>
#include <vector>
using namespace fps;
int main() {
    int BH, T, H, W, Tt, Th, Tw, rt, rh, rw, shift, qblocks, waves, blocks;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d", &BH, &T, &H, &W, &Tt, &Th, &Tw, &rt, &rh, &rw, &shift, &qblocks, &waves, &blocks) == 14) {
        Geom g;
        std::memset(&g, 0, sizeof(g));
        g.BH = BH; g.T = T; g.H = H; g.W = W; g.Tt = Tt; g.Th = Th; g.Tw = Tw;
        g.nT = (T + Tt - 1) / Tt; g.nH = (H + Th - 1) / Th; g.nW = (W + Tw - 1) / Tw;
        g.M = g.nT * g.nH * g.nW; g.TSP = 128;
        ItemPlan p;
        const int slots = plan_items(g, {rt, rh, rw}, shift, qblocks, waves, 128, blocks, p);
        const int n[3] = {g.nT, g.nH, g.nW}, tile[3] = {Tt, Th, Tw}, size[3] = {T, H, W}, r[3] = {rt, rh, rw};
        auto window = [&](int i, int u) {                    // tokens of the window along axis i
            if (shift) u = n[i] > 2 * r[i] + 1 ? (u < r[i] ? r[i] : u > n[i] - 1 - r[i] ? n[i] - 1 - r[i] : u) : n[i] / 2;
            const int lo = u > r[i] ? u - r[i] : 0, hi = u + r[i] < n[i] - 1 ? u + r[i] : n[i] - 1;
            return ((hi + 1) * tile[i] < size[i] ? (hi + 1) * tile[i] : size[i]) - lo * tile[i];
        };
        // every position of a level in the same band of the most tokens, bands falling from level to level
        int bad_levels = 0;
        long long tokens[3][kAxisLevels], most[3];
        int levels[3];
        double spread = 1;                                   // longest item over the mean, of the levels' own lengths
        for (int i = 0; i < 3; ++i) {
            AxisLevel level[kAxisLevels];
            levels[i] = plan_axis(n[i], tile[i], size[i], r[i], shift, level, tokens[i]);
            most[i] = 0;
            for (int u = 0; u < n[i]; ++u) most[i] = most[i] > window(i, u) ? most[i] : window(i, u);
            auto band = [&](int u) { const long long x = 100LL * window(i, u); return x >= 90 * most[i] ? 0 : x >= 72 * most[i] ? 1 : 2; };
            std::vector<int> seen(n[i], 0);
            int last = -1;
            double sum = 0;
            long long longest = 0;
            for (int l = 0; l < levels[i]; ++l) {
                const int count = AxisLevel::upper(level[l].skip_count), first = AxisLevel::lower(level[l].first_len1),
                          len1 = AxisLevel::upper(level[l].first_len1), skip = AxisLevel::lower(level[l].skip_count);
                const int of_level = band(first);
                bad_levels += of_level <= last;
                last = of_level;
                for (int k = 0; k < count; ++k) {
                    const int u = first + k + (k >= len1 ? skip : 0);
                    if (u < 0 || u >= n[i]) { ++bad_levels; continue; }
                    ++seen[u];
                    bad_levels += band(u) != of_level;
                }
                sum += (double)tokens[i][l] * count;
                longest = longest > tokens[i][l] ? longest : tokens[i][l];
            }
            for (int c : seen) bad_levels += c != 1;
            spread *= longest * n[i] / sum;
        }
        std::vector<int> seen((size_t)BH * g.M * qblocks, 0);
        int bad = 0, rises = 0;
        double last = 1e30;
        for (int s = 0; slots && s < kMaxSections && (int)(p.section[s] & kSectionStart) < slots; ++s) {
            const uint32_t w = p.section[s];
            const double len = (double)tokens[0][(w >> 26) & 3] * tokens[1][(w >> 28) & 3] * tokens[2][w >> 30];
            rises += len > last;
            last = len;
        }
        bad += slots % 4;
        for (int xcd = 0; xcd < 8 && slots; ++xcd)
            for (int slot = 0; slot < slots; ++slot) {
                int sec = 0, bh, t, h, w, jq;
                for (int l = 1; l <= kSectionLanes; ++l) sec += (int)(p.section[l] & kSectionStart) <= slot;
                if (!planned_item(p, g, qblocks, reciprocal(qblocks), xcd, slot, sec, &bh, &t, &h, &w, &jq)) continue;
                if (bh < 0 || bh >= BH || t < 0 || t >= g.nT || h < 0 || h >= g.nH || w < 0 || w >= g.nW || jq < 0 || jq >= qblocks) ++bad;
                else ++seen[(size_t)(((bh * g.nT + t) * g.nH + h) * g.nW + w) * qblocks + jq];
            }
        for (int s : seen) bad += slots ? s != 1 : 0;
        std::printf("%d %d %d %d %.12f\n", slots, bad, rises, bad_levels, spread);
    }
}
"""


def test_items_dealt_by_length_are_each_dealt_once(tmp_path):
    """Every work item once, in range, over windows from one tile to all, cut and uncut grids, both edge rules; sections in
    falling order of their length, an axis' levels of positions within their bands.  Launches with more keys than the L2s
    hold twice, small ones, those of short walks and those of about one length stay in raster order."""
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "plan.hip", tmp_path / "plan"
    src.write_text(PLAN_PROGRAM)
    res = subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-I" + os.path.join(ROOT, "include"),
                          "-I" + os.path.join(ROOT, "paper_2506_04648_amd", "csrc"), str(src), "-o", str(exe)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    grids = [(1, 8, 16), (5, 23, 37), (10, 26, 36), (7, 9, 130), (17, 3, 5), (1, 1, 100)]
    radii = [(0, 0, 0), (1, 1, 1), (3, 1, 2), (2, 0, 4), (40, 40, 99)]
    cases = [(bh, *g, *t, *r, shift, qb, waves, blocks) for bh in (1, 3, 24) for g in grids
             for t in ((1, 8, 16), (2, 4, 4), (1, 1, 1)) for r in radii for shift in (0, 1)
             for qb, waves, blocks in ((1, 4, 12), (2, 4, 40), (1, 1, 27), (1, 4, 11))]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True,
                         text=True, check=True).stdout.split("\n")
    planned = level = 0
    for c, line in zip(cases, out):
        slots, bad, rises, bad_levels = map(int, line.split()[:4])
        spread = float(line.split()[4])
        tiles = -(-c[1] // c[4]) * -(-c[2] // c[5]) * -(-c[3] // c[6])
        small, large = c[0] * tiles * c[11] <= (2048 if c[12] == 1 else 256), 2 * c[0] * tiles * 128 * 128 > 64 << 20
        short = c[13] < 12
        if abs(spread - 1.1) > 1e-9:
            assert (slots == 0) == (small or large or short or spread < 1.1), (c, line)
        assert bad == 0 and rises == 0 and bad_levels == 0, (c, line)
        planned += slots > 0
        level += slots == 0 and not (small or large or short)
    assert planned > 100 and level > 20


TAIL_PROGRAM = r"""
#include "fps_attn_plan.h"
#include <cstdio>
#include <cstring>
#include <vector>
using namespace fps;
int main() {
    int BH, T, H, W, rt, rh, rw, shift, qblocks, waves, row_bytes, blocks;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d", &BH, &T, &H, &W, &rt, &rh, &rw, &shift, &qblocks, &waves, &row_bytes, &blocks) == 12) {
        Geom g;
        std::memset(&g, 0, sizeof(g));
        g.BH = BH; g.T = g.nT = T; g.H = H; g.W = W; g.Tt = 1; g.Th = 8; g.Tw = 16;
        g.nH = (H + 7) / 8; g.nW = (W + 15) / 16; g.M = g.nT * g.nH * g.nW; g.TSP = 128;
        g.rc_layer = reciprocal(g.nH * g.nW);
        const int total = BH * g.M * qblocks, chunk = ((total + 7) / 8 + 3) / 4 * 4, layer = g.nH * g.nW * qblocks;
        ItemPlan p;
        const int first = plan_tail(g, {rt, rh, rw}, shift, qblocks, waves, row_bytes, blocks, chunk, p);
        std::vector<int> seen(8 * chunk, 0);
        int bad = 0, rises = 0, sections = 0;
        for (int xcd = 0; xcd < 8 && first >= 0; ++xcd) {
            int longest = 1 << 30;
            for (int slot = 0; slot < chunk; ++slot) {
                int sec = 0, wi = xcd * chunk + slot;
                for (int l = 1; l <= kSectionLanes; ++l) sec += (int)(p.section[l] & kSectionStart) <= slot;
                if (slot >= first) wi = tail_item(p, g, qblocks, reciprocal(qblocks), xcd * chunk + first, slot, sec);
                if (wi < xcd * chunk || wi >= (xcd + 1) * chunk) { ++bad; continue; }
                ++seen[wi];
                if (slot < first) continue;
                // the item is where its section's levels say, and none is much longer than the first
                const int uh = wi / qblocks / g.nW % g.nH, uw = wi / qblocks % g.nW;
                auto holds = [&](const AxisLevel& l, int u) {
                    for (int k = 0; k < AxisLevel::upper(l.skip_count); ++k) if (level_position(l, k) == u) return true;
                    return false;
                };
                bad += !holds(p.level[1][(p.section[sec] >> 28) & 3], uh) || !holds(p.level[2][p.section[sec] >> 30], uw);
                auto window = [&](int u, int n, int tile, int size, int r) {
                    if (shift) u = n > 2 * r + 1 ? (u < r ? r : u > n - 1 - r ? n - 1 - r : u) : n / 2;
                    const int lo = u > r ? u - r : 0, hi = u + r < n - 1 ? u + r : n - 1;
                    return ((hi + 1) * tile < size ? (hi + 1) * tile : size) - lo * tile;
                };
                const int len = window(uh, g.nH, 8, H, rh) * window(uw, g.nW, 16, W, rw);
                if (slot == first) longest = len;
                rises += len > longest * 1.25;
            }
        }
        for (int s : seen) bad += first >= 0 && s != 1;
        // the lengths of the sections, those of their levels, never rise
        long long th[kAxisLevels], tw[kAxisLevels];
        AxisLevel level[kAxisLevels];
        plan_axis(g.nH, 8, H, rh, shift, level, th);
        plan_axis(g.nW, 16, W, rw, shift, level, tw);
        double last = 1e30;
        for (int s = 0; first >= 0 && s < kMaxSections && (int)(p.section[s] & kSectionStart) < chunk; ++s) {
            const double len = (double)th[(p.section[s] >> 28) & 3] * tw[p.section[s] >> 30];
            rises += len > last;
            sections += first >= 0;
            last = len;
        }
        const int n = first < 0 ? 0 : chunk - first;
        std::printf("%d %d %d %d %d %d %d\n", first, bad, rises, chunk, layer, n, sections);
    }
}
"""


def test_the_tail_dealt_by_length_deals_each_item_once(tmp_path):
    """The sorted end of an XCD's chunk is whole layers' worth of items, wherever in a layer it starts, each dealt once; one
    round of workgroups or two (FP8), the sections in falling order of their length; none where everything is resident at once, a
    layer is longer than that or walks are short."""
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "tail.hip", tmp_path / "tail"
    src.write_text(TAIL_PROGRAM)
    res = subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-I" + os.path.join(ROOT, "include"),
                          "-I" + os.path.join(ROOT, "paper_2506_04648_amd", "csrc"), str(src), "-o", str(exe)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    cases = [(bh, *grid, *r, shift, qb, waves, row, blocks)
             for bh in (1, 7, 12) for grid in ((21, 30, 52), (5, 90, 119), (3, 23, 37), (40, 8, 33), (2, 200, 300))
             for r in ((1, 1, 1), (2, 0, 3), (0, 40, 1)) for shift in (0, 1) for qb in (1, 3)
             for waves, row, blocks in ((4, 128, 27), (4, 256, 27), (2, 128, 105), (1, 128, 12), (3, 128, 11))]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True,
                         text=True, check=True).stdout.split("\n")
    tails = 0
    for c, line in zip(cases, out):
        first, bad, rises, chunk, layer, n, sections = map(int, line.split())
        waves, row, blocks = c[9:]
        assert bad == 0 and rises == 0, (c, line)
        rounds = 32 * (8 // waves)
        wanted = rounds * (1 if row > 128 else 2)
        if blocks < 12 or chunk <= rounds or layer > min(chunk, wanted):
            assert first == -1, (c, line)
        if first >= 0:
            assert n % layer == 0 and n <= chunk and (wanted <= n < wanted + layer or n > chunk - layer), (c, line)
            assert sections > 1, (c, line)
            tails += 1
    assert tails > 40


NARROW_PROGRAM = r"""
#include "fps_attn_device.h"
#include <cstdio>
#include <cstring>
using namespace fps;
int main() {
    int BH, n[3], tile[3], size[3], r[3], shift;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d", &BH, size, size + 1, size + 2, tile, tile + 1, tile + 2, r, r + 1, r + 2, &shift) == 11) {
        for (int i = 0; i < 3; ++i) n[i] = (size[i] + tile[i] - 1) / tile[i];
        AttnArgs a;
        std::memset(&a, 0, sizeof(a));
        Geom& g = a.g;
        g.BH = BH; g.T = size[0]; g.H = size[1]; g.W = size[2]; g.Tt = tile[0]; g.Th = tile[1]; g.Tw = tile[2];
        g.nT = n[0]; g.nH = n[1]; g.nW = n[2]; g.M = n[0] * n[1] * n[2];
        const int tokens = tile[0] * tile[1] * tile[2];
        g.BS = tokens <= 96 ? 32 : 128; g.NS = 1; g.KBS = g.KB = (tokens + g.BS - 1) / g.BS; g.KBG = g.BS == 128 ? g.KBS : 1;
        g.TSP = g.KB * g.BS;
        a.rt = r[0]; a.rh = r[1]; a.rw = r[2]; a.edge_shift = shift;
        std::printf("%.9f %d %d %d\n", longest_over_mean(g, {r[0], r[1], r[2]}, shift), window_blocks(a),
                    row_waves(a, window_blocks(a), true), row_waves(a, window_blocks(a), false));
    }
    for (int waves : {1, 2, 4})
        for (int total : {256, 258})
            for (int blocks : {29, 30}) {
                AttnArgs a;
                std::memset(&a, 0, sizeof(a));
                a.g.nT = blocks; a.g.nH = a.g.nW = a.g.NS = a.g.KBG = 1;
                a.rt = blocks; a.waves = waves; a.total = total;
                std::printf("%d", (int)narrow_in_four(a));
            }
    std::printf("\n");
    for (int items : {1, 64, 65, 128, 129, 160, 161, 256, 257, 288, 289, 320, 321, 400, 401})
        for (int blocks : {5, 6, 11, 12, 17, 18, 29, 30, 39, 40, 59, 60})
            for (double s : {1.0, 1.1, 1.3, 1.4, 1.5, 1.8}) std::printf("%d", narrow_waves(items, blocks, s));
    std::printf("\n");
}
"""


def test_launches_of_few_items_take_narrow_ones(tmp_path):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "narrow.hip", tmp_path / "narrow"
    src.write_text(NARROW_PROGRAM)
    res = subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-I" + os.path.join(ROOT, "include"),
                          "-I" + os.path.join(ROOT, "paper_2506_04648_amd", "csrc"), str(src), "-o", str(exe)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    cases = [(bh, *grid, *tile, *r, shift) for bh in (1, 3, 5, 9) for grid in ((5, 23, 37), (8, 24, 48), (1, 1, 5000))
             for tile in ((1, 8, 16), (2, 8, 16), (3, 4, 4)) for r in ((1, 1, 1), (0, 1, 2), (9, 9, 9)) for shift in (0, 1)]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True,
                         text=True, check=True).stdout.split("\n")

    def rule(items, blocks, spread):
        if blocks < 6 or items > 400:
            return 4
        if items <= 128:
            return 1 if items <= 64 else 2
        if items <= 160:
            return 2 if blocks >= 12 and spread >= 1.3 else 4
        uneven = spread >= (1.3 if blocks >= 60 else 1.4 if blocks >= 18 else 1.5)
        if items <= 256:
            narrow = blocks >= 12 and uneven
        elif items <= 288:
            narrow = blocks >= 40 and (uneven or spread < 1.1)
        else:
            narrow = blocks >= (30 if items <= 320 else 40) and spread >= 1.8
        return 2 if narrow else 4

    seen = set()
    for c, line in zip(cases, out):
        spread, blocks, waves, waves_bf16 = line.split()
        bh, size, tile, r, shift = c[0], c[1:4], c[4:7], c[7:10], c[10]
        want, items = 1.0, bh
        for s, t, k in zip(size, tile, r):
            n = -(-s // t)
            items *= n
            lengths = []
            for u in range(n):
                if shift:
                    u = min(max(u, k), n - 1 - k) if n > 2 * k + 1 else n // 2
                lengths.append(sum(min(t, s - v * t) for v in range(max(0, u - k), min(n - 1, u + k) + 1)))
            want *= max(lengths) * n / sum(lengths)
        assert abs(float(spread) - want) < 1e-6 * want, (c, line)
        slots = tile[0] * tile[1] * tile[2]
        if slots <= 96:
            assert int(waves) == int(waves_bf16) == -(-slots // 32), (c, line)
        else:
            assert int(waves_bf16) == (2 if items * -(-slots // 128) <= 128 and int(blocks) >= 6 else 4), (c, line)
        if slots > 96 and min(abs(want - edge) for edge in (1.1, 1.3, 1.4, 1.5, 1.8)) > 1e-6:
            assert int(waves) == rule(items * -(-slots // 128), int(blocks), want), (c, line)
            seen.add(int(waves))
    assert seen == {1, 2, 4}
    assert out[len(cases)] == "000001000000"
    it = iter(out[len(cases) + 1])
    for items in (1, 64, 65, 128, 129, 160, 161, 256, 257, 288, 289, 320, 321, 400, 401):
        for blocks in (5, 6, 11, 12, 17, 18, 29, 30, 39, 40, 59, 60):
            for s in (1.0, 1.1, 1.3, 1.4, 1.5, 1.8):
                assert int(next(it)) == rule(items, blocks, s), (items, blocks, s)


ROUTE_PROGRAM = r"""
#include "fps_attn_device.h"
#include <cstdio>
#include <cstring>
using namespace fps;
int main() {
    fps_shape s;
    int wt, wh, ww, shift, fp8;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d", &s.B, &s.heads, &s.T, &s.H, &s.W, &s.Tt, &s.Th, &s.Tw, &s.Qt, &s.Qh, &s.Qw, &wt, &wh, &ww, &shift, &fp8) == 16) {
        s.head_dim = 128;
        AttnArgs a;
        std::memset(&a, 0, sizeof(a));
        if (check_shape(&s, &a.g) != FPS_OK) return 1;
        a.rt = wt / 2; a.rh = wh / 2; a.rw = ww / 2; a.edge_shift = shift;
        const int workgroups = plan_launch(a, fp8 != 0);
        const Geom& g = a.g;
        // wave groups that share an item's keys, as the launchers choose them
        const int sb = g.BS == 128 ? 4 : g.KBS, ks = sb >= 3 ? 2 : 4;
        int groups = 1;
        if (sb == 4 && a.waves < 4) groups = fp8 && (a.waves == 1 || narrow_in_four(a)) ? 4 : 2;
        else if ((sb == 4 || g.NS == 1) && split_keys(a, ks)) groups = ks;
        const char* order = a.tail < 0 ? "length" : a.tail < a.chunk ? "tail" : "raster";
        std::printf("%d %d %d %d %d %s %d %d\n", sb, a.waves, groups, (int)(sb == 4 ? g.KB > 1 : g.NS > 1), a.total, order, workgroups, a.qblocks);
    }
}
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """(heads, grid, tile, sub-tile, window, shifted, fp8) of calls -> per call (32-key sub-blocks of a key block, waves of an
    item, wave groups, several blocks or groups a tile, items, order, workgroups of an XCD, items of a tile)."""
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("routes")
    src, exe, lib = d / "routes.hip", d / "routes", os.path.join(ROOT, "paper_2506_04648_amd")
    src.write_text(ROUTE_PROGRAM)
    res = subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(lib, "csrc"), str(src), "-o", str(exe),
                          "-L" + lib, "-l:libfps.so", "-Wl,-rpath," + lib], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]

    def run(calls):
        lines = [" ".join(map(str, (1, heads, *grid, *tile, *(qtile or (0, 0, 0)), *window, int(shift), int(fp8))))
                 for heads, grid, tile, qtile, window, shift, fp8 in calls]
        out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.split("\n")
        rows = [tuple(x if x.isalpha() else int(x) for x in line.split()) for line in out if line]
        assert len(rows) == len(lines)
        return rows
    return run


def test_the_gpu_cases_reach_the_kernels_that_they_name(routes):
    """(sub-blocks of a key block, waves, wave groups, several blocks or groups a tile) of the cases of the GPU tests of few
    items, FP8 and BF16, and the order of those that are to end by length."""
    from tests import test_gpu_parity as t

    def kernels(cases, shift=False):
        rows = [routes([(c[0], c[1], c[2], c[3], c[4], shift or len(c) == 7 and c[5], fp8) for c in cases]) for fp8 in (True, False)]
        return [tuple(r[i][:4] for r in rows) for i in range(len(cases))]

    one, many = 0, 1
    assert kernels([c[:3] + (None,) + c[3:4] for c in t.SPLIT_CASES]) == [
        ((4, 4, 1, one), (4, 4, 1, one)), ((4, 4, 1, one), (4, 4, 1, one)), ((4, 1, 4, one), (4, 2, 2, one)),
        ((4, 1, 4, one), (4, 2, 2, one)), ((4, 1, 4, one), (4, 2, 2, one)), ((4, 1, 4, many), (4, 2, 2, many)),
        ((3, 3, 2, one),) * 2, ((2, 2, 4, one),) * 2, ((1, 1, 4, one),) * 2, ((1, 1, 1, one),) * 2, ((2, 2, 1, one),) * 2,
        ((3, 3, 1, one),) * 2, ((3, 3, 1, one),) * 2]
    narrow = [((4, 1, 4, one), (4, 2, 2, one)), ((4, 1, 4, many), (4, 2, 2, many)), ((4, 2, 2, one),) * 2,
              ((4, 2, 2, many),) * 2, ((4, 2, 4, one), (4, 2, 2, one)), ((4, 2, 4, many), (4, 2, 2, many))]
    whole = [((4, 4, 2, one),) * 2, ((4, 4, 2, many),) * 2]
    assert kernels(t.NARROW_CASES) == narrow[:1] * 2 + narrow[1:] + [
        ((4, 2, 2, one), (4, 4, 2, one)), whole[0], ((4, 4, 1, one),) * 2] + [((4, 2, 2, one), (4, 4, 1, one))] * 2
    assert kernels(t.WHOLE_SPLIT_CASES) == [whole[0]] * 2 + [whole[1]] * 3
    assert kernels(t.RASTER_CASES, shift=True) == narrow + whole
    seen = set()
    for fp8 in (True, False):
        for case, row in zip(t.TAIL_CASES, routes([c + (False, fp8) for c in t.TAIL_CASES])):
            assert row[5] == ("raster" if not fp8 and row[7] == 3 else "tail"), (case, row)
            seen.add((fp8, row[0], row[1], row[7]))
    # in BF16 the layer of three items a tile is more than a round of workgroups
    assert {(True, 4, 4, 1), (True, 4, 4, 2), (True, 4, 4, 3), (True, 2, 2, 1), (True, 2, 4, 2), (True, 1, 1, 1)} <= seen


def test_the_cut_tiles_of_the_gpu_cases_are_taken_as_they_say(routes, items_of_tiles):
    """Kernels (sub-blocks of a key block, waves, wave groups, several groups a tile) of the GPU test's cut tiles, FP8 and BF16; all
    cases with more than one wave an item have tiles whose sub-blocks are not taken in their order, and all of them together every
    kind of wave: with rows, without, and of items left out."""
    from tests import test_gpu_parity as t
    window, cases = (3, 3, 3), t.REAL_ROW_CASES
    kernels, without, reordered = [], 0, set()
    for grid, tile, qtile in cases:
        row = routes([(2, grid, tile, qtile, window, False, fp8) for fp8 in (True, False)])
        kernels.append(tuple(r[:4] for r in row))
        for r in row:
            wrong, other, no_block, left_out, needless = items_of_tiles([(grid, tile, qtile, r[1])])[0]
            assert wrong == needless == 0 and (other > 0) == (left_out > 0) == (r[1] > 1), (grid, tile, qtile, r)
            without += no_block > 0
            if other:
                reordered.add(r[:3])
    one = ((4, 1, 4, 1), (4, 2, 2, 1))
    assert kernels == [((2, 4, 1, 1),) * 2, one, ((3, 3, 1, 1),) * 2, ((1, 4, 1, 1),) * 2, ((4, 2, 4, 1), (4, 2, 2, 1)), one,
                       ((1, 1, 1, 1),) * 2, ((4, 4, 1, 1),) * 2, ((4, 4, 1, 1),) * 2, ((4, 2, 2, 1),) * 2,
                       ((4, 4, 2, 1), (4, 4, 2, 1)), ((3, 4, 1, 1),) * 2, ((2, 2, 1, 1),) * 2]
    assert without >= 10 and len(reordered) == 9, (without, reordered)


def test_narrow_items_are_all_resident_at_once(routes):
    """Up to 256 items of 128 rows are whole workgroups one on a CU; cut in two they must fit two on a CU, 64 on an XCD, and the
    plan's sections, each rounded up, may take more.  Three calls that did, and the items of others."""
    over = [(1, (14, 51, 31), (6, 8, 8), None, (5, 5, 1), False, True),      # 252 items, 68 workgroups an XCD: 47.7 -> 64.1 us
            (1, (16, 30, 50), (1, 8, 16), None, (7, 1, 3), False, True),     # 256 items, 30.3 -> 36.0
            (1, (8, 57, 57), (1, 8, 16), None, (3, 3, 3), False, True)]      # 256 items, 37.0 -> 43.6
    for row in routes(over):
        assert row[1] == 4 and row[2] == 2 and row[5] == "raster" and 250 <= row[4] <= 256, row
    calls = [(heads, grid, tile, None, window, False, True) for heads in range(1, 18)
             for grid in ((5, 23, 37), (7, 20, 27), (16, 30, 50), (9, 46, 57), (14, 51, 31), (3, 49, 62), (2, 58, 58))
             for tile in ((1, 8, 16), (2, 8, 16), (6, 8, 8), (1, 7, 15))
             for window in ((3, 3, 3), (5, 5, 1), (7, 1, 3), (5, 7, 9))]
    narrow = 0
    for call, (sb, waves, groups, many, items, order, workgroups, per_tile) in zip(calls, routes(calls)):
        if waves == 2 and 256 < items <= 512:
            assert workgroups <= 64, (call, items, workgroups)
            narrow += 1
    assert narrow > 20


REAL_PROGRAM = r"""
#include "fps_attn_device.h"
#include <cstdio>
#include <vector>
using namespace fps;
int main() {
    fps_shape s;
    while (std::scanf("%d %d %d %d %d %d %d %d %d", &s.T, &s.H, &s.W, &s.Tt, &s.Th, &s.Tw, &s.Qt, &s.Qh, &s.Qw) == 9) {
        s.B = s.heads = 1;
        s.head_dim = 128;
        Geom g;
        if (check_shape(&s, &g) != FPS_OK) return 1;
        const int sbg = g.QSP / 32;
        long bad = 0, real = 0;
        for (int cls = 0; cls < 8; ++cls) {
            std::vector<int> want;                 // every sub-block with a token, by the definition
            for (int qs = 0; qs < g.NS * sbg; ++qs)
                if (real_tokens(g, cls, sub_tile_origin(g, qs / sbg)) > 32 * (qs % sbg)) want.push_back(qs);
            const RealSubBlocks r(g, cls, sbg);
            bad += r.total() != (int)want.size();
            for (int i = 0; i < (int)want.size(); ++i) bad += r.sub_block(i) != want[i];
            real += (long)want.size();
        }
        std::printf("%ld %ld\n", bad, real);
    }
}
"""


def test_real_sub_blocks_of_cut_tiles(tmp_path):
    """The sub-blocks that hold tokens, in order, against their enumeration: groups of 1 to 300 tokens, one or many a tile, the
    grid's last tiles cut along any of the axes."""
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    src, exe, lib = tmp_path / "real.hip", tmp_path / "real", os.path.join(ROOT, "paper_2506_04648_amd")
    src.write_text(REAL_PROGRAM)
    res = subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(lib, "csrc"), str(src), "-o", str(exe),
                          "-L" + lib, "-l:libfps.so", "-Wl,-rpath," + lib], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    rng = random.Random(5)
    lines = ["1 1 1 1 1 1 1 1 1", "40 50 60 16 16 16 1 1 1"]          # one token; 4096 groups a tile
    for _ in range(3000):
        q = [rng.choice((1, 1, 2, 3, 4, 5, 7, 8, 16)) for _ in range(3)]
        t = [x * rng.choice((1, 1, 2, 3, 5)) for x in q]
        if q[0] * q[1] * q[2] <= 300 and t[0] * t[1] * t[2] <= 4096:
            n = [x * rng.randint(1, 3) + rng.randint(0, x) for x in t]
            lines.append(" ".join(map(str, n + t + q)))
    out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.split("\n")
    rows = [tuple(map(int, line.split())) for line in out if line]
    assert len(rows) == len(lines) > 2000
    wrong = [(line, row) for line, row in zip(lines, rows) if row[0]]
    assert not wrong, wrong[:5]
    assert sum(row[1] for row in rows) > 100000


ITEM_PROGRAM = r"""
#include "fps_attn_device.h"
#include <cstdio>
#include <vector>
using namespace fps;
typedef int (*Taken)(const Geom&, int cls, int jq, int of_item, int sbg);
static long calls;                                 // sums of a wave that had to find the order
template <int SB, int W> int taken(const Geom& g, int cls, int jq, int of_item, int sbg) {
    return item_sub_block<SB, W>(g, cls, jq, of_item, sbg, [](int x) { ++calls; return x; });
}
template <int SB> Taken of_waves(int W) { return W == 1 ? taken<SB, 1> : W == 2 ? taken<SB, 2> : W == 3 ? taken<SB, 3> : taken<SB, 4>; }
int main() {
    fps_shape s;
    int of_rows;                                   // waves of an item; 0: as many as each launch of such a shape may have
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d", &s.T, &s.H, &s.W, &s.Tt, &s.Th, &s.Tw, &s.Qt, &s.Qh, &s.Qw, &of_rows) == 10) {
        s.B = s.heads = 1;
        s.head_dim = 128;
        Geom g;
        if (check_shape(&s, &g) != FPS_OK) return 1;
        const int sbg = g.QSP / 32, all = g.NS * sbg, sb = g.BS == 128 ? 4 : g.KBS;
        long wrong = 0, reordered = 0, without = 0, left_out = 0, needless = 0;
        for (int W : {1, 2, 3, 4}) {
            if (of_rows ? W != of_rows : W != query_waves(g) && (g.BS != 128 || W == 3)) continue;
            const Taken item = sb == 4 ? of_waves<4>(W) : sb == 3 ? of_waves<3>(W) : sb == 2 ? of_waves<2>(W) : of_waves<1>(W);
            for (int u = 0; u < g.M; ++u) {
                const int cls = (u / (g.nH * g.nW) == g.nT - 1) << 2 | (u / g.nW % g.nH == g.nH - 1) << 1 | (u % g.nW == g.nW - 1);
                std::vector<int> times(all);       // that a sub-block is taken
                calls = 0;
                bool other = false, saved = false;
                for (int jq = 0; jq < all / W; ++jq) {
                    int gone = 0, rows = 0;
                    for (int w = 0; w < W; ++w) {
                        const int qs = item(g, cls, jq, w, sbg);
                        wrong += qs < -2 || qs >= all;
                        gone += qs == -2;
                        without += qs == -1;
                        other |= qs != jq * W + w;
                        if (qs < 0) continue;
                        ++times[qs];
                        rows += real_tokens(g, cls, sub_tile_origin(g, qs / sbg)) > 32 * (qs % sbg);
                    }
                    wrong += gone != 0 && gone != W;               // the waves of an item leave together or not at all
                    // the kernels find out by themselves where the rows are those of one group or of one wave
                    wrong += g.NS > 1 && W > 1 && gone == 0 && rows == 0;
                    left_out += gone == W;
                    saved |= gone == W;
                }
                wrong += other && !saved;                          // another order has to save an item
                for (int qs = 0; qs < all; ++qs) {
                    const bool real = real_tokens(g, cls, sub_tile_origin(g, qs / sbg)) > 32 * (qs % sbg);
                    wrong += real ? times[qs] != 1 : times[qs] > 1;
                }
                reordered += other;
                if (all <= W) needless += calls;
            }
        }
        std::printf("%ld %ld %ld %ld %ld\n", wrong, reordered, without, left_out, needless);
    }
}
"""


@pytest.fixture(scope="module")
def items_of_tiles(tmp_path_factory):
    """(grid, tile, sub-tile, waves of an item or 0) -> per shape: violations of what an item's waves take, and of all tiles those
    whose sub-blocks are not taken in their order, waves without a sub-block, items left out, sums for tiles of one item."""
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("items")
    src, exe, lib = d / "items.hip", d / "items", os.path.join(ROOT, "paper_2506_04648_amd")
    src.write_text(ITEM_PROGRAM)
    res = subprocess.run([HIPCC, "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17",
                          "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(lib, "csrc"), str(src), "-o", str(exe),
                          "-L" + lib, "-l:libfps.so", "-Wl,-rpath," + lib], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]

    def run(shapes):
        lines = [" ".join(map(str, (*grid, *tile, *(qtile or (0, 0, 0)), waves))) for grid, tile, qtile, waves in shapes]
        out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.split("\n")
        rows = [tuple(map(int, line.split())) for line in out if line]
        assert len(rows) == len(lines)
        return rows
    return run


def test_every_real_sub_block_is_taken_by_one_wave(items_of_tiles):
    """Over all items of every tile of random shapes: each sub-block with a token once, one without at most once, no walked item
    without rows, and none of the sums that find the order where a tile is one item and nothing can be saved."""
    rng = random.Random(9)
    shapes = [((4, 9, 18), (2, 4, 8), (1, 4, 4), 0), ((40, 50, 60), (16, 16, 16), (1, 1, 1), 0)]
    for _ in range(3000):
        q = [rng.choice((1, 1, 2, 3, 4, 5, 7, 8, 16)) for _ in range(3)]
        t = [x * rng.choice((1, 1, 2, 3, 5)) for x in q]
        if q[0] * q[1] * q[2] <= 300 and t[0] * t[1] * t[2] <= 4096:
            shapes.append((tuple(x * rng.randint(1, 3) + rng.randint(0, x) for x in t), tuple(t), tuple(q), 0))
    rows = items_of_tiles(shapes)
    bad = [(shape, row) for shape, row in zip(shapes, rows) if row[0] or row[4]]
    assert not bad, bad[:5]
    assert sum(row[1] > 0 for row in rows) > 100 and sum(row[2] > 0 for row in rows) > 100 and sum(row[3] > 0 for row in rows) > 100


COPY_PROGRAM = r"""
#include "fps_attn_device.h"
namespace fps {
template <int FIRST, int N>
__global__ void copies(const uint8_t* p) {
    __shared__ uint8_t lds[4096];
    dma_chunks<FIRST, N>(p, 16 * threadIdx.x, (uint32_t)(uintptr_t)&lds[0]);
}
#define ONE(f, n) template __global__ void copies<f, n>(const uint8_t*);
ONE(0, 1) ONE(0, 2) ONE(0, 3) ONE(0, 4) ONE(1, 1) ONE(1, 2) ONE(1, 3) ONE(2, 1) ONE(2, 2) ONE(3, 1)
}
"""


def device_assembly(tmp_path, name, program):
    """gfx950 assembly of each kernel of a program, by its mangled name."""
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    src, out = tmp_path / f"{name}.hip", tmp_path / f"{name}.s"
    src.write_text(program)
    res = subprocess.run([HIPCC, "--cuda-device-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-S",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-I" + os.path.join(ROOT, "include"),
                          "-I" + os.path.join(ROOT, "paper_2506_04648_amd", "csrc"), str(src), "-o", str(out)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    parts = re.split(r"^(_Z\w+):.*$", out.read_text(), flags=re.M)
    return {kernel: body.split("s_endpgm")[0] for kernel, body in zip(parts[1::2], parts[2::2])}


def test_copies_to_lds_take_consecutive_chunks(tmp_path):
    """dma_chunks<FIRST, N>: 1 KB pieces FIRST .. FIRST + N - 1, whatever FIRST is."""
    kernels = device_assembly(tmp_path, "copies", COPY_PROGRAM)
    seen = {}
    for kernel, body in kernels.items():
        key = tuple(map(int, re.search(r"copiesILi(\d)ELi(\d)E", kernel).groups()))
        seen[key] = [int(x, 0) for x in re.findall(r"global_load_lds_dwordx4 .*offset:(\w+)", body)]
    assert seen == {(f, n): [1024 * (f + i) for i in range(n)] for f in range(4) for n in range(1, 5 - f)}


MAX_PROGRAM = r"""
#include "fps_device_common.h"
namespace fps {
// what a caller has written before is read across lanes behind the maximum
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void maximum(const uint32_t* x, uint32_t* out) {
    __shared__ uint32_t red[WAVES], held[64 * WAVES];
    const int i = threadIdx.x;
    held[i] = x[i];
    out[64 * WAVES + i] = workgroup_max<WAVES>(x[i], red);
    out[i] = held[64 * WAVES - 1 - i];
}
template __global__ void maximum<1>(const uint32_t*, uint32_t*);
template __global__ void maximum<2>(const uint32_t*, uint32_t*);
template __global__ void maximum<4>(const uint32_t*, uint32_t*);
}
"""


def test_the_maximum_of_a_workgroup_orders_its_lds(tmp_path):
    """One barrier whatever the number of waves; of a workgroup that is a wave it is the compiler's `wave barrier`."""
    kernels = device_assembly(tmp_path, "maximum", MAX_PROGRAM)
    barriers = {k: body.count("s_barrier") + body.count("; wave barrier") for k, body in kernels.items() if "maximum" in k}
    assert sorted(barriers.values()) == [1, 1, 1], barriers
