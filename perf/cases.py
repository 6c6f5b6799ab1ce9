"""The attention calls whose speed counts: what a denoising loop has the library do for one layer.

One pass is one attention call on the GPU as a program makes it: operand preparation of Q, K and V
(tile order + per-tile or per-channel FP8 quantisation, or BF16 packing) from raster bf16 tensors,
then the sliding-tile attention, on buffers that the program keeps between calls.  The results are
the attention output and the scales of the quantisation; the packed operands are private to the
library and not a result.

A case is described by plain values:
  B, heads, T, H, W          batch, heads and token grid (head_dim is 128)
  Tt, Th, Tw / Qt, Qh, Qw    tile, and the quantisation sub-tile (0, 0, 0: the tile itself)
  wt, wh, ww, shift          window in tiles; True: the window is shifted at the grid's edges
  fp8, channel_v             FP8 or BF16 mode; one V scale per channel instead of per tile
  tiled                      True: tile_order -> *_tiles entry points -> tiled output -> tile_unorder;
                             False: the fused entry points that read and write raster order
  f32_out                    fp32 instead of bf16 output
  step                       0, or the denoising step 1..50 whose regime (early, mid, late) carries
                             this case's precision and window
"""
from __future__ import annotations

import math

import torch

from paper_2506_04648_amd import fps, synth

HEAD_DIM = 128
NUM_STEPS, ALPHA1, ALPHA2 = 50, 0.2, 0.5
# outlier channels per head and tensor (about 2 % of the channels, as in the synthetic workloads)
N_OUTLIER, OUTLIER_GAIN = 3, 8.0
# the largest listed case, the dense BF16 call at 720p, is 133 Tflop on the tokens of its tiles; a drawn
# case stays under it by a margin that also covers the slower launches (see _relative_cost)
MAX_DRAWN_COST = 30e12

PLAIN = dict(B=1, Qt=0, Qh=0, Qw=0, shift=False, fp8=True, channel_v=False, tiled=False, f32_out=False, step=0)


def _case(name, heads, grid, tile, window, **more):
    c = dict(PLAIN, name=name, heads=heads)
    c.update(zip(("T", "H", "W"), grid))
    c.update(zip(("Tt", "Th", "Tw"), tile))
    c.update(zip(("wt", "wh", "ww"), window))
    c.update(more)
    return c


def listed():
    tiny, small, large = synth.TINY, synth.WAN_1_3B_480P, synth.WAN_14B_720P
    dense = synth.WAN_14B_720P_DENSE
    return [
        # the smallest workload: four launches of a few microseconds, latency and host work
        _case("tiny", tiny.heads, tiny.grid, tiny.tile, tiny.window),
        # a small clip with a ragged grid and fp32 output: a preview resolution, or one rank's heads
        _case("small-ragged", 5, (5, 23, 37), (1, 8, 16), (3, 3, 3), f32_out=True),
        # the 480p workload of the small model: sparse FP8
        _case("480p", small.heads, small.grid, small.tile, small.window),
        # the same window without quantisation (sliding tiles in BF16)
        _case("480p-bf16", small.heads, small.grid, small.tile, small.window, fp8=False),
        # the coarse tile (three blocks of 128 slots) with a window of the window ablation
        _case("480p-tile-688", small.heads, small.grid, (6, 8, 8), (3, 3, 1)),
        # the finest tile of the tile-size ablation: 48 tokens in two blocks of 32 slots
        _case("480p-tile-344", small.heads, small.grid, (3, 4, 4), (3, 5, 7)),
        # quantisation finer than the sparsity tile, two clips in a batch, shifted windows, and the
        # separate entry points for a caller that keeps its tensors in tile order
        _case("480p-sub-tiles", small.heads, small.grid, (2, 8, 16), (3, 3, 3), B=2, Qt=1, Qh=8, Qw=8,
              shift=True, tiled=True),
        # the 720p workload of the large model: sparse FP8, the headline call
        _case("720p", large.heads, large.grid, large.tile, large.window),
        # the paper's variant of it: V quantised per channel over all tokens
        _case("720p-channel-v", large.heads, large.grid, large.tile, large.window, channel_v=True),
        # the step-aware schedule on the same grid: half of its calls are late steps,
        _case("720p-late", large.heads, large.grid, large.tile, synth.WAN_14B_720P_LATE.window, step=40),
        # three in ten are mid steps with a wider window,
        _case("720p-mid", large.heads, large.grid, large.tile, synth.WAN_14B_720P_MID.window, step=20),
        # and the early ones are dense BF16: the largest call there is
        _case("720p-dense-bf16", dense.heads, dense.grid, dense.tile, dense.window, fp8=False, step=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another call of the same kinds: heads, grid (mostly ragged), tile, window and options over the
    ranges of the listed ones."""
    while True:
        tile = rng.choice([(1, 8, 16)] * 4 + [(2, 4, 4), (3, 4, 4), (2, 8, 4), (1, 7, 15), (2, 8, 16),
                                              (4, 8, 8), (6, 8, 8), (4, 16, 16)])
        tokens = _log_int(rng, 1000, 75600)
        T = min(21, max(2, _log_int(rng, 3, 21)))
        H = max(4, int(round(math.sqrt(tokens / T) * rng.uniform(0.6, 1.1))))
        W = max(4, int(round(tokens / (T * H))))
        c = _case("", _log_int(rng, 1, 40), (T, H, W), tile, (1, 1, 1))
        del c["name"]
        c["B"] = rng.choice([1, 1, 1, 2])
        c["fp8"] = rng.random() < 0.75
        c["channel_v"] = c["fp8"] and rng.random() < 0.2
        c["shift"] = rng.random() < 0.2
        c["tiled"] = rng.random() < 0.2
        c["f32_out"] = rng.random() < 0.2
        if tile in ((2, 8, 16), (4, 8, 8)) and rng.random() < 0.5:
            c["Qt"], c["Qh"], c["Qw"] = tile[0] // 2, tile[1], tile[2]
        n = [-(-g // t) for g, t in zip((T, H, W), tile)]
        dense = rng.random() < 0.2
        for key, na, top in zip(("wt", "wh", "ww"), n, (7, 7, 9)):
            c[key] = 2 * na - 1 if dense else rng.randint(1, min(top, 2 * na - 1))
        if rng.random() < 0.3:
            c["step"] = rng.randint(1, NUM_STEPS)
        if _relative_cost(c) <= MAX_DRAWN_COST:
            return c


def _axis_sum(size, tile, w, shift):
    """Sum over one axis of (tokens of query tile) * (tokens of key tile) over the kept pairs."""
    n = -(-size // tile)
    r = w // 2
    length = [min(tile, size - u * tile) for u in range(n)]
    total = 0
    for u in range(n):
        if shift and n <= 2 * r + 1:
            lo, hi = 0, n - 1
        else:
            c = min(max(u, r), n - 1 - r) if shift else u
            lo, hi = max(0, c - r), min(n - 1, c + r)
        total += length[u] * sum(length[lo:hi + 1])
    return total


def work(case):
    """What one pass cannot do without: Q, K, V read once, the output written once, and the two
    matrix products over the real tokens of the kept tile pairs."""
    c = case
    bh = c["B"] * c["heads"]
    tokens = c["T"] * c["H"] * c["W"]
    pairs = 1
    for size, tile, w in (("T", "Tt", "wt"), ("H", "Th", "wh"), ("W", "Tw", "ww")):
        pairs *= _axis_sum(c[size], c[tile], c[w], c["shift"])
    return {"bytes": bh * tokens * HEAD_DIM * (3 * 2 + (4 if c["f32_out"] else 2)),
            "flops": 4 * HEAD_DIM * bh * pairs}


def _relative_cost(case):
    """Flops weighted by how much more a unit of them costs in small tiles and on padding."""
    c = case
    q = [c["Qt"], c["Qh"], c["Qw"]] if c["Qt"] else [c["Tt"], c["Th"], c["Tw"]]
    slots = q[0] * q[1] * q[2]
    pad = 1.0
    for size, tile in (("T", "Tt"), ("H", "Th"), ("W", "Tw")):
        pad *= (-(-c[size] // c[tile]) * c[tile] / c[size]) ** 2
    return work(c)["flops"] * pad * (4.0 if slots <= 96 else 1.0)


def _shape(c):
    qtile = (c["Qt"], c["Qh"], c["Qw"]) if c["Qt"] else None
    return fps.make_shape(c["heads"], (c["T"], c["H"], c["W"]), (c["Tt"], c["Th"], c["Tw"]), B=c["B"], qtile=qtile)


def prepare(case, seed):
    """Q, K, V in raster order on the GPU -- standard normal with a few outlier channels per head, the
    distribution the library's synthetic workloads stand in for activations with -- and the buffers
    a program keeps for its calls."""
    c = case
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    shape = _shape(c)
    lead = (c["B"], c["heads"])
    raster = []
    for _ in range(3):
        x = torch.randn(lead + (c["T"], c["H"], c["W"], HEAD_DIM), generator=gen, device=dev, dtype=torch.float32)
        pick = torch.rand(lead + (HEAD_DIM,), generator=gen, device=dev).topk(N_OUTLIER, dim=-1).indices
        gain = torch.ones(lead + (HEAD_DIM,), device=dev).scatter_(-1, pick, OUTLIER_GAIN)
        x *= gain[:, :, None, None, None, :]
        raster.append(x.to(torch.bfloat16))
        del x
    prec = fps.PREC_FP8 if c["fp8"] else fps.PREC_BF16
    window = (c["wt"], c["wh"], c["ww"], fps.EDGE_SHIFT if c["shift"] else fps.EDGE_TRUNCATE)
    vscale = fps.VSCALE_CHANNEL if c["channel_v"] else fps.VSCALE_TILE
    groups = fps.num_groups(shape)
    st = {
        "shape": shape, "raster": raster, "prec": prec, "window": window, "vscale": vscale, "tiled": c["tiled"],
        "packed": [torch.empty(fps.packed_bytes(shape, prec), dtype=torch.uint8, device=dev) for _ in range(3)],
        "scales": [torch.empty(lead + (HEAD_DIM if i == 2 and c["channel_v"] else groups,), dtype=torch.float32,
                               device=dev) for i in range(3)],
        "out": torch.empty(lead + (c["T"], c["H"], c["W"], HEAD_DIM), device=dev,
                           dtype=torch.float32 if c["f32_out"] else torch.bfloat16),
        "step": None,
    }
    if c["tiled"]:
        slots = fps.num_tiles(shape) * fps.tile_slots(shape)
        st["x_tiled"] = torch.empty(lead + (slots, HEAD_DIM), dtype=torch.bfloat16, device=dev)
        st["out_tiled"] = torch.empty(lead + (slots, HEAD_DIM), dtype=st["out"].dtype, device=dev)
    if c["step"]:
        regimes = [(fps.PREC_BF16, (41, 11, 9)), (fps.PREC_FP8, (7, 5, 5)), (fps.PREC_FP8, (3, 3, 3))]
        step = c["step"]
        regimes[0 if step <= ALPHA1 * NUM_STEPS else 1 if step <= ALPHA2 * NUM_STEPS else 2] = (prec, window)
        st["step"] = fps.make_step_cfg(step, NUM_STEPS, ALPHA1, ALPHA2, regimes)
    return st


def run(state):
    """One attention call: prepare Q, K, V, attend."""
    s = state
    shape, packed, scales = s["shape"], s["packed"], s["scales"]
    prec, window = s["prec"], s["window"]
    if s["step"] is not None:
        prec, window = fps.schedule_select(s["step"])[0], None
    for role in range(3):
        x = fps.tile_order(shape, s["raster"][role], out=s["x_tiled"]) if s["tiled"] else s["raster"][role]
        if prec == fps.PREC_FP8:
            fps.quantize_tiles(shape, x, role, vscale=s["vscale"], out=packed[role], scales=scales[role],
                               raster=not s["tiled"])
        else:
            fps.pack_tiles_bf16(shape, x, role, out=packed[role], vscale=scales[2], raster=not s["tiled"])
    fp8 = prec == fps.PREC_FP8
    out = fps.attn_fwd(shape, window, prec, packed[0], packed[1], packed[2], scales[0] if fp8 else None,
                       scales[1] if fp8 else None, scales[2], vscale=s["vscale"],
                       out=s["out_tiled"] if s["tiled"] else s["out"], raster_out=not s["tiled"], step=s["step"])
    if s["tiled"]:
        out = fps.tile_unorder(shape, out, out=s["out"])
    return {"out": out, "scales": scales if fp8 else scales[2:]}


def tolerance(case):
    """Measured by permuting the 128 channels, which adds every score's products and every output's
    channels in another order.  FP8: a weight whose score lies near a rounding boundary falls on the
    other side, which moves that weight by 6 to 12 %; the listed and eight drawn cases change by
    3.3e-3 to 1.2e-2.  BF16: 2e-5 to 1.6e-4 with few of the bf16 outputs changing at all; where an
    implementation rounds the weights against another reference, more of them do."""
    return {"rel": 4e-2} if case["fp8"] else {"rel": 1e-3}
