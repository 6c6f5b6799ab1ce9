"""GPU parity: every step of the HIP path, called through the C ABI, against the CPU oracle."""
import dataclasses
import math
import sys

import numpy as np
import pytest

from oracle import e4m3
from oracle import fps_oracle as fo
from paper_2506_04648_amd import fps, synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def tiny():
    return gu.GpuRun(synth.TINY)


# ---- layout and quantisation: bit exact -----------------------------------------------------
@pytest.mark.parametrize("grid,tile", [((4, 16, 16), (2, 4, 4)), ((3, 5, 6), (2, 4, 4)),
                                       ((2, 9, 20), (1, 8, 16)), ((3, 7, 9), (2, 4, 16)),
                                       ((3, 13, 20), (2, 8, 16)), ((7, 9, 10), (6, 8, 8)),
                                       ((5, 7, 9), (3, 4, 4)), ((2, 9, 20), (1, 7, 15)),
                                       ((3, 5, 6), (2, 8, 4))])
def test_tile_order_roundtrip_bit_exact(grid, tile):
    import torch
    say("tile_order", grid, tile)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, heads=3)
    run = gu.GpuRun(w)
    for a, t in zip(run.qkv, run.tiled):
        want = fo.tile_order(a, run.g)
        got = t[0].float().cpu().numpy()
        assert np.array_equal(got[:, run.slots], want)
        assert np.all(got[:, run.pad_slots()] == 0)
        back = fps.tile_unorder(run.shape, t)
        assert np.array_equal(back[0].float().cpu().numpy(), a)
        back32 = fps.tile_unorder(run.shape, t.float().contiguous())
        assert np.array_equal(back32[0].cpu().numpy(), a)


@pytest.mark.parametrize("heads", [30, 150])
@pytest.mark.parametrize("tile,qtile", [((1, 8, 16), None), ((2, 8, 16), (1, 8, 8)), ((3, 4, 4), None)])
def test_tile_order_of_more_than_the_caches_hold(tile, qtile, heads):
    """Input and output beyond 256 MB are read another way, and from 4096 times 32 slots on a wave moves all 32: round trip of
    every head, bit for bit."""
    import torch
    say("tile_order of a large tensor", tile, qtile, heads)
    grid = (5, 23, 37)                                      # 33 and 163 MB, tiled at least 35 and 177
    one = gu.GpuRun(dataclasses.replace(synth.TINY, grid=grid, tile=tile, heads=1), qtile=qtile)
    shape = fps.make_shape(heads, grid, tile, qtile=qtile)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    x = torch.randn((1, heads) + grid + (128,), generator=gen, device="cuda:0", dtype=torch.bfloat16)
    slots = torch.from_numpy(np.asarray(one.slots)[fo.token_positions(one.g)]).to("cuda:0")
    t = fps.tile_order(shape, x)
    assert (x.numel() * 2 + t.numel() * 2 > 256 << 20) == (heads == 150) and t.numel() >= 4096 * 32 * 128
    want = torch.zeros_like(t)
    want[:, :, slots] = x.flatten(2, 4)
    assert torch.equal(t, want)
    assert torch.equal(fps.tile_unorder(shape, t), x)
    assert torch.equal(fps.tile_unorder(shape, t.float()), x.float())


def _check_quantize(run, heads_slots, label):
    g = run.g
    for role, (xq, sc) in enumerate(run.quantize()):
        codes = fps.debug_unpack_q8(run.shape, xq, role)[0].cpu().numpy()
        sc = sc[0].cpu().numpy()
        for hs in heads_slots:
            x = fo.tile_order(run.qkv[role][hs].astype(np.float64), g)
            wc, ws = fo.quantize_tiles(x, g)
            assert np.array_equal(sc[hs].view(np.uint32), ws.view(np.uint32)), (label, role, hs)
            got = codes[hs][run.slots]
            zero_sign = ((got ^ wc) == 0x80) & ((wc & 0x7F) == 0)
            mism = (got != wc) & ~zero_sign
            assert int(mism.sum()) == 0, (label, role, hs, int(mism.sum()))
            assert np.all((codes[hs][run.pad_slots()] & 0x7F) == 0)
        assert not np.any((codes & 0x7F) == 0x7F)


def test_quantize_tiny_bit_exact(tiny):
    say("quantize tiny")
    _check_quantize(tiny, range(2), "tiny")


def test_quantize_ragged_128_token_tiles_bit_exact():
    say("quantize ragged 128")
    w = dataclasses.replace(synth.TINY, grid=(2, 13, 40), tile=(1, 8, 16), heads=2, n_outlier=3)
    _check_quantize(gu.GpuRun(w), range(2), "ragged128")


@pytest.mark.parametrize("grid,tile", [((3, 13, 20), (2, 8, 16)),      # 256 tokens; last T tile half empty
                                       ((7, 9, 10), (6, 8, 8)),         # 384 tokens, ragged on every axis
                                       ((5, 16, 20), (4, 16, 16)),      # 1024 tokens
                                       ((5, 7, 9), (3, 4, 4)),          # 48 tokens in two 32-slot blocks
                                       ((2, 9, 20), (1, 7, 15)),        # 105 tokens in one 128-slot block
                                       ((13, 17, 20), (12, 16, 16)),    # 3072 tokens, 24 blocks
                                       ((25, 5, 6), (24, 32, 32))])     # 24576 tokens, 192 blocks, mostly padding
def test_quantize_tiles_of_several_blocks_bit_exact(grid, tile):
    """One scale per TILE although the kernels work on 128-token blocks (tile amax pre-pass)."""
    say("quantize multi-block", grid, tile)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, heads=2, n_outlier=3, config_id=15)
    run = gu.GpuRun(w)
    assert run.quantize()[0][1].shape[-1] == run.g.M
    _check_quantize(run, range(2), f"multi-block {tile}")


SUB_TILE_CASES = [
    ((3, 13, 20), (2, 8, 16), (1, 8, 16)),      # sub-tile = one 128-slot block, 2 per tile
    ((7, 9, 10), (6, 8, 8), (2, 8, 8)),         # 3 sub-tiles of 128 tokens
    ((5, 9, 18), (4, 8, 8), (2, 4, 8)),         # 4 sub-tiles of 64 tokens: two 32-slot blocks each
    ((3, 5, 6), (2, 4, 4), (1, 2, 4)),          # 4 sub-tiles of 8 tokens in a 32-slot block each
    ((5, 16, 20), (4, 16, 16), (2, 8, 16)),     # 8 sub-tiles of 256 tokens (two 128-slot blocks each)
    ((3, 9, 20), (2, 7, 15), (1, 7, 5)),        # 6 sub-tiles of 35 tokens in two 32-slot blocks each
]


@pytest.mark.parametrize("grid,tile,qtile", SUB_TILE_CASES)
def test_quantisation_sub_tiles_layout_and_codes_bit_exact(grid, tile, qtile):
    """Scales per sub-tile of the sparsity tile: tile order round trip, scales and codes."""
    import torch
    say("sub-tile quantise", grid, tile, qtile)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, heads=2, n_outlier=3, config_id=19)
    run = gu.GpuRun(w, qtile=qtile)
    for a, t in zip(run.qkv, run.tiled):
        got = t[0].float().cpu().numpy()
        assert np.array_equal(got[:, run.slots], fo.tile_order(a, run.g))
        assert np.all(got[:, run.pad_slots()] == 0)
        assert np.array_equal(fps.tile_unorder(run.shape, t)[0].float().cpu().numpy(), a)
    assert run.quantize()[0][1].shape[-1] == run.g.n_groups
    _check_quantize(run, range(2), f"sub-tile {tile} {qtile}")
    p16 = run.pack_bf16()
    for role in range(3):                                   # fused raster entries == tiled entries
        xq, sc = fps.quantize_tiles(run.shape, run.raster[role], role, raster=True)
        assert torch.equal(xq, run.q8[role][0]) and torch.equal(sc, run.q8[role][1])
        xp, vs = fps.pack_tiles_bf16(run.shape, run.raster[role], role, raster=True)
        assert torch.equal(xp, p16[role][0])
        assert (vs is None and p16[role][1] is None) or torch.equal(vs, p16[role][1])


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("grid,tile,qtile", SUB_TILE_CASES)
def test_attention_with_quantisation_sub_tiles(prec, grid, tile, qtile):
    import torch
    say("sub-tile attention", prec, grid, tile, qtile)
    window = (3, 3, 3)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=2, n_outlier=3,
                            config_id=20)
    run = gu.GpuRun(w, qtile=qtile)
    out, vis = run.attn(prec, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, window))
    for h in range(2):
        st = gu.compare_head(run, out, h, prec, window)
        say("  head", h, st)
        gu.assert_parity(st, f"{grid} {tile} {qtile} head {h}")
    raster = run.attn(prec, raster_out=True)
    assert torch.equal(raster, fps.tile_unorder(run.shape, out))
    if prec == fps.PREC_FP8:                                # per-channel V with sub-tile Q/K scales
        out = run.attn(prec, vscale=fps.VSCALE_CHANNEL)
        st = gu.compare_head(run, out, 0, prec, window, vscale=fps.VSCALE_CHANNEL)
        say("  per-channel V", st)
        gu.assert_parity(st, f"{grid} {tile} {qtile} per-channel V")


# Tiles of several scale groups that the grid cuts.  A work item takes the real sub-blocks of several of its tile's groups one
# after the other; in items of one sub-block (FP8: the cases so marked) the waves find out that theirs has no row.
REAL_ROW_CASES = [
    ((3, 13, 20), (2, 8, 16), (1, 8, 8)),       # 64 tokens: one sub-block of two in the last column, its other group empty
    ((3, 13, 20), (2, 8, 16), (1, 8, 16)),      # 128 tokens: one sub-block of four (FP8: one-wave items)
    ((2, 30, 30), (1, 12, 24), (1, 12, 8)),     # 96 tokens, items of three sub-blocks: two and one of three
    ((5, 10, 30), (4, 8, 16), (2, 4, 4)),       # 32 tokens, items of four of 16 groups; cut along every axis
    ((7, 9, 18), (6, 8, 16), (2, 4, 16)),       # 128 tokens, six groups: layers, rows and columns missing
    ((10, 9, 12), (2, 8, 16), (1, 8, 16)),      # few items: groups of 96 and 12 tokens (FP8: one-wave items)
    ((4, 9, 18), (1, 4, 12), (1, 4, 4)),        # 16 tokens, one-wave items in both: one whole, one cut and one empty
    ((2, 12, 16), (2, 8, 16), (1, 8, 16)),      # 128 tokens, items of four sub-blocks: two of each group
    ((5, 5, 16), (5, 8, 16), (1, 8, 16)),       # the same of five groups, three of each, a wave without a sub-block
    ((3, 13, 68), (2, 8, 16), (1, 8, 16)),      # the same, items of two sub-blocks in two wave groups
    ((3, 13, 180), (2, 8, 16), (1, 8, 16)),     # and of four in two
    ((3, 13, 20), (2, 12, 16), (1, 12, 8)),     # 96 tokens, items of four sub-blocks
    ((4, 13, 12), (3, 8, 8), (1, 8, 8)),        # 64 tokens, items of two
]


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("grid,tile,qtile", REAL_ROW_CASES)
def test_items_take_the_real_rows_of_cut_tiles(prec, grid, tile, qtile):
    import torch
    say("real rows", prec, grid, tile, qtile)
    window = (3, 3, 3)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=2, n_outlier=3, config_id=29)
    run = gu.GpuRun(w, qtile=qtile)
    out = run.attn(prec)
    for h in range(2):
        gu.assert_parity(gu.compare_head(run, out, h, prec, window), f"{grid} {tile} {qtile} head {h}")
    assert torch.all(out[0][:, run.pad_slots()] == 0)       # tile-ordered output: every padding slot is cleared
    assert torch.equal(run.attn(prec, raster_out=True), fps.tile_unorder(run.shape, out))
    # every row of the output is written, whoever takes it: into a buffer of NaN, the same again
    for dtype in (torch.float32, torch.bfloat16):
        for raster in (False, True):
            want = (fps.tile_unorder(run.shape, out) if raster else out).to(dtype)
            got = run.attn(prec, raster_out=raster, out=torch.full_like(want, math.nan))
            assert torch.equal(got, want), (dtype, raster, int(torch.isnan(got).sum()))


def test_quantize_special_values():
    """Ties of the exact quotient, e4m3-representable inputs, all-zero tiles, amax = 448."""
    import torch
    say("quantize special")
    g = fo.Geometry(1, 8, 32, 1, 8, 16)                      # two tiles of 128 tokens
    shape = fps.make_shape(1, (1, 8, 32), (1, 8, 16))
    rng = np.random.default_rng(0)
    vals = e4m3.decode(np.arange(0x7F, dtype=np.uint8))
    mids = 0.5 * (vals[:-1] + vals[1:])
    x = np.zeros((g.L_padded, 128))
    # tile 0: amax 448 -> s = 1: representable values and every midpoint, both signs
    pool = np.concatenate([vals, mids, -vals, -mids])
    pool = pool[np.abs(pool) <= 448]
    t0 = rng.choice(pool, size=(128, 128))
    t0[0, 0] = 448.0
    # tile 1: amax = 7 * c with c = 29 -> many mathematically exact midpoints x*448/amax
    amax = 7.0 * 29.0 / 64.0
    cands = np.array([(2 * n + 1) * 29.0 / 64.0 * 2.0 ** -k for n in range(16) for k in range(0, 9)])
    cands = cands[(cands <= amax)]
    t1 = rng.choice(np.concatenate([cands, -cands]), size=(128, 128))
    t1[5, 7] = amax
    x[:128], x[128:] = t0, t1
    xb = synth.round_to_bf16(x.astype(np.float32)).astype(np.float64)
    tiled = gu.to_device_bf16(xb.astype(np.float32)[None, None])
    for role in (0, 1, 2):
        xq, sc = fps.quantize_tiles(shape, tiled, role)
        codes = fps.debug_unpack_q8(shape, xq, role)[0, 0].cpu().numpy()
        wc, ws = fo.quantize_tiles(xb, g)
        assert np.array_equal(sc[0, 0].cpu().numpy(), ws)
        zero_sign = ((codes ^ wc) == 0x80) & ((wc & 0x7F) == 0)
        assert int(((codes != wc) & ~zero_sign).sum()) == 0, role
    z = torch.zeros((1, 1, g.L_padded, 128), dtype=torch.bfloat16, device="cuda:0")
    xq, sc = fps.quantize_tiles(shape, z, 1)
    assert torch.all(sc == 1.0) and torch.all(xq == 0)


# the scales' exponents lie 9 below; at -117 they are just above the least normal number, at -118 on both
# sides of it, from -119 on subnormal
@pytest.mark.parametrize("exponent", [0, 100, -117, -118, -120, -126])
@pytest.mark.parametrize("vscale", [fps.VSCALE_TILE, fps.VSCALE_CHANNEL])
def test_codes_for_every_significand_of_amax(vscale, exponent):
    """One scale group per 8-bit significand of amax; in each, every significand in 19 binades: every way
    in which a quotient can lie on or next to a rounding boundary."""
    say("quantize significands", vscale, exponent)
    rng = np.random.default_rng(12)
    g = fo.Geometry(1, 8, 16 * 128, 1, 8, 16)                # 128 tiles of 128 tokens, 128 channels
    shape = fps.make_shape(1, (1, 8, 16 * 128), (1, 8, 16))
    # axis 1 of the groups: the values of one scale (a tile's, or 16384 tokens of a channel)
    amax = (np.arange(128, 256) * 2.0 ** (exponent - 7))[:, None]
    every = np.resize(np.arange(128, 256)[:, None] * 2.0 ** -np.arange(19.0), 128 * 128) * 2.0 ** (exponent - 7)
    x = rng.permuted(np.repeat(every[None], 128, axis=0), axis=1)
    x = np.minimum(x, amax) * rng.choice([-1.0, 1.0], size=x.shape)
    x[:, :1] = amax                                          # 2432 combinations, each 6 or 7 times before this one
    x = x.reshape(g.L_padded, 128) if vscale == fps.VSCALE_TILE else np.ascontiguousarray(x.T)
    xb = synth.round_to_bf16(x.astype(np.float32))
    tiled = gu.to_device_bf16(xb[None, None])
    quantize = fo.quantize_tiles if vscale == fps.VSCALE_TILE else lambda v, _: fo.quantize_channels(v)
    wc, ws = quantize(xb.astype(np.float64), g)
    for role in (0, 1, 2) if vscale == fps.VSCALE_TILE else (2,):
        xq, sc = fps.quantize_tiles(shape, tiled, role, vscale=vscale)
        codes = fps.debug_unpack_q8(shape, xq, role)[0, 0].cpu().numpy()
        assert np.array_equal(sc[0, 0].cpu().numpy(), ws)
        zero_sign = ((codes ^ wc) == 0x80) & ((wc & 0x7F) == 0)
        assert int(((codes != wc) & ~zero_sign).sum()) == 0, role


def test_per_channel_codes_keep_the_sign_of_zeros():
    """A negative zero, and a negative value that rounds to zero, give the code of -0."""
    say("per-channel signs of zeros")
    rng = np.random.default_rng(13)
    x = np.float32(2.0) ** rng.integers(-110, 1, size=(128, 128)) * rng.choice([-1.0, 1.0], size=(128, 128))
    x[rng.random((128, 128)) < 0.3] = -0.0
    x[rng.random((128, 128)) < 0.1] = 0.0
    x[7] = 1.5                                               # every channel's largest value
    xb = synth.round_to_bf16(x.astype(np.float32))
    shape = fps.make_shape(1, (1, 8, 16), (1, 8, 16))
    xq, _ = fps.quantize_tiles(shape, gu.to_device_bf16(xb[None, None]), fps.ROLE_V, vscale=fps.VSCALE_CHANNEL)
    codes = fps.debug_unpack_q8(shape, xq, fps.ROLE_V)[0, 0].cpu().numpy()
    assert np.any((codes == 0x80) & (xb == 0)) and np.any((codes == 0x80) & (xb != 0))
    assert np.array_equal(codes >> 7, np.signbit(xb).astype(np.uint8))


@pytest.mark.parametrize("vscale", [fps.VSCALE_TILE, fps.VSCALE_CHANNEL])
def test_ties_beside_a_nan_go_to_even(vscale):
    """A scale group with a NaN has scale 1: its other values, all halfway between two codes here, are
    rounded to the even one."""
    say("ties beside NaN", vscale)
    codes = np.arange(0x08, 0x7E, dtype=np.uint8)
    ties = 0.5 * (e4m3.decode(codes) + e4m3.decode(codes + 1))
    even = np.where(codes % 2 == 0, codes, codes + 1)
    pick = np.random.default_rng(14).integers(0, codes.size, size=(128, 128))
    x = ties[pick]
    x[3] = np.nan                                            # in every channel and in the tile
    shape = fps.make_shape(1, (1, 8, 16), (1, 8, 16))
    xq, sc = fps.quantize_tiles(shape, gu.to_device_bf16(x.astype(np.float32)[None, None]), fps.ROLE_V, vscale=vscale)
    got = fps.debug_unpack_q8(shape, xq, fps.ROLE_V)[0, 0].cpu().numpy()
    assert np.all(sc.cpu().numpy() == 1.0)
    finite = np.isfinite(x)
    assert np.array_equal(got[finite], even[pick][finite])


# ---- the matrix instruction's accumulation accuracy -------------------------------------------
def test_score_accumulation_error_model(tiny):
    """Raw E4M3 scores of single tile pairs against the exact integer dot products: the layout is
    right (errors are tiny, not O(1)) and the hardware's accumulation error stays inside the bound
    the parity comparator assumes when it decides which P roundings are ambiguous."""
    say("score accumulation")
    tiny.quantize()
    worst = 0.0
    for h, u, v in [(0, 0, 0), (0, 5, 6), (1, 31, 27), (1, 12, 12), (0, 17, 21), (1, 3, 7)]:
        r, got, exact = gu.score_error_ratio(tiny, h, u, v)
        worst = max(worst, r)
        assert np.max(np.abs(got - exact)) <= 1e-3 * np.max(np.abs(exact))
    say("  tiny worst |dS| / sum|qk| = %.3e (bound %.3e)" % (worst, gu.ACC_EPS))
    assert worst <= gu.ACC_EPS
    w = dataclasses.replace(synth.TINY, grid=(2, 16, 32), tile=(1, 8, 16), heads=2, n_outlier=3,
                            config_id=11)
    run = gu.GpuRun(w)
    run.quantize()
    worst = 0.0
    for h, u, v in [(0, 0, 0), (0, 1, 2), (1, 7, 3), (1, 5, 5), (0, 6, 1)]:
        r, got, exact = gu.score_error_ratio(run, h, u, v)
        worst = max(worst, r)
    say("  128-token tiles worst |dS| / sum|qk| = %.3e" % worst)
    assert worst <= gu.ACC_EPS


def test_score_accumulation_bound_on_adversarial_codes():
    """Code patterns chosen to stress the matrix instruction's adder: a product of 448*448 beside
    127 products of 1*1 (the hardware drops the seven ones that share the large product's group of
    eight: the error is 7, not 127), cancelling large products over a small residue, uniformly
    random codes of the whole format, random powers of two over 15 binades.  All stay inside the
    accumulation bound the accepted set is built on."""
    say("adversarial codes")
    vals = e4m3.decode(np.arange(256, dtype=np.uint8))
    finite = vals[np.isfinite(vals)]
    rng = np.random.default_rng(7)

    def ratio(q, k, tile):
        w = dataclasses.replace(synth.TINY, grid=tile, tile=tile, heads=1, window=(1, 1, 1), config_id=23)
        run = gu.GpuRun(w, qkv=[a[None].astype(np.float32) for a in (q, k, np.zeros_like(q))])
        run.quantize()
        r, got, exact = gu.score_error_ratio(run, 0, 0, 0)
        return r / gu.ACC_EPS, float(np.max(np.abs(got - exact)))

    for tile in [(1, 8, 16), (2, 4, 4)]:                     # 128-slot and 32-slot blocks
        shp = tile + (128,)
        q = np.ones(shp)
        q[..., 0] = 448.0
        r, err = ratio(q, q.copy(), tile)
        say(f"  {tile} one dominant product: {r:.3f} of the bound, |err| {err:g}")
        assert r <= 1.0 and err <= 8.0
        q, k = np.ones(shp), np.ones(shp)
        q[..., 0] = q[..., 1] = k[..., 0] = 448.0
        k[..., 1] = -448.0
        r, err = ratio(q, k, tile)
        say(f"  {tile} cancelling pair: {r:.3f} of the bound, |err| {err:g}")
        assert r <= 1.0
        q, k = rng.choice(finite, shp), rng.choice(finite, shp)
        q[0, 0, 0, 0] = k[0, 0, 0, 0] = 448.0                # the tile scale is exactly 1
        r, err = ratio(q, k, tile)
        say(f"  {tile} uniformly random codes: {r:.3f} of the bound")
        assert r <= 1.0
        q = 2.0 ** rng.integers(-6, 9, shp) * rng.choice([-1.0, 1.0], shp)
        k = 2.0 ** rng.integers(-6, 9, shp) * rng.choice([-1.0, 1.0], shp)
        q[0, 0, 0, 0] = k[0, 0, 0, 0] = 448.0
        r, err = ratio(q, k, tile)
        say(f"  {tile} random powers of two: {r:.3f} of the bound")
        assert r <= 1.0


# ---- attention -------------------------------------------------------------------------------
def test_attention_tiny_fp8_full(tiny):
    say("attention tiny fp8")
    out, vis = tiny.attn(fps.PREC_FP8, visited=True)
    mask = fo.tile_mask(tiny.g, tiny.w.window)
    assert np.array_equal(vis.cpu().numpy().astype(bool), mask) and int(mask.sum()) == 200
    for h in range(2):
        st = gu.compare_head(tiny, out, h, fps.PREC_FP8, tiny.w.window)
        say("  head", h, st)
        gu.assert_parity(st, f"tiny fp8 head {h}")


@pytest.mark.parametrize("window", [(1, 3, 3), (3, 7, 7), (1, 1, 1), (2, 2, 2)])
def test_attention_tiny_bf16(tiny, window):
    say("attention tiny bf16", window)
    out, vis = tiny.attn(fps.PREC_BF16, window=window, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(tiny.g, window))
    for h in range(2):
        st = gu.compare_head(tiny, out, h, fps.PREC_BF16, window)
        say("  head", h, st)
        gu.assert_parity(st, f"tiny bf16 head {h}")


@pytest.mark.parametrize("window", [(3, 7, 7), (1, 1, 1), (2, 4, 6)])
def test_attention_tiny_fp8_windows(tiny, window):
    say("attention tiny fp8 window", window)
    out, vis = tiny.attn(fps.PREC_FP8, window=window, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(tiny.g, window))
    st = gu.compare_head(tiny, out, 1, fps.PREC_FP8, window)
    say("  ", st)
    gu.assert_parity(st, f"tiny fp8 {window}")


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("grid,tile,window", [
    ((3, 5, 6), (2, 4, 4), (3, 3, 3)),          # ragged on every axis, 32-token tiles
    ((2, 13, 40), (1, 8, 16), (3, 3, 3)),       # ragged 128-token tiles, several tiles per axis
    ((1, 8, 16), (1, 8, 16), (1, 1, 1)),        # a single tile
    ((1, 3, 5), (1, 8, 16), (5, 5, 5)),         # a single, mostly padded tile
    ((5, 8, 16), (1, 8, 16), (2, 1, 1)),        # temporal-only window, even size
    ((3, 13, 20), (2, 8, 16), (3, 3, 3)),       # 256-token tiles (2 blocks); one key block all padding
    ((7, 9, 10), (6, 8, 8), (3, 1, 3)),         # 384-token tiles (3 blocks), ragged on every axis
    ((5, 16, 20), (4, 16, 16), (3, 1, 1)),      # 1024-token tiles (8 blocks)
    ((5, 7, 9), (3, 4, 4), (3, 3, 3)),          # 48-token tiles: two 32-slot blocks, 16 slots of padding
    ((3, 5, 12), (2, 8, 4), (3, 1, 3)),         # 64-token tiles: two 32-slot blocks
    ((2, 9, 20), (1, 7, 15), (3, 3, 3)),        # 105-token tiles in one 128-slot block
    ((13, 17, 20), (12, 16, 16), (3, 3, 3)),    # 3072-token tiles (24 blocks); skipped padding-only blocks
])
def test_attention_small_shapes(prec, grid, tile, window):
    say("attention small", prec, grid, tile, window)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=2, n_outlier=3,
                            config_id=7)
    run = gu.GpuRun(w)
    out, vis = run.attn(prec, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, window))
    for h in range(2):
        st = gu.compare_head(run, out, h, prec, window)
        say("  head", h, st)
        gu.assert_parity(st, f"{grid} {tile} {window} head {h}")


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("heads,grid,tile", [(1, (1, 8, 20), (1, 8, 16)),      # 2 work items: fewer than a group of four
                                             (3, (3, 9, 60), (1, 8, 16)),      # 72 items, 4 a row: 9 per XCD, rounded to 12
                                             (2, (2, 9, 40), (2, 8, 16)),      # 2 per tile, 6 a row
                                             (3, (3, 5, 22), (2, 4, 4))])      # one-wave workgroups, 6 a row
def test_every_item_of_an_even_row_is_computed(prec, heads, grid, tile):
    """Rows of an even number of work items are dealt in a turning order: each item once."""
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=(3, 3, 3), heads=heads, n_outlier=3, config_id=16)
    run = gu.GpuRun(w)
    out = run.attn(prec)
    for h in range(heads):
        st = gu.compare_head(run, out, h, prec, w.window)
        say("  head", h, st)
        gu.assert_parity(st, f"{grid} {tile} head {h}")


# heads, grid, tile, window, heads compared.  Where a launch is small and a window has six or eight blocks the keys are shared:
# by two wave groups for three sub-blocks, by four for two or one; tiles of 128 slots, at most 64 of them here, are cut into
# items of 32 rows (FP8) whose keys four groups share, or of 64 rows and two groups (BF16).  test_launch_rules.py has the routes
SPLIT_CASES = [
    (2, (4, 8, 16), (1, 8, 16), (7, 1, 1), (0, 1)),          # 4 blocks: neither cut nor split
    (2, (3, 8, 16), (1, 8, 16), (5, 1, 1), (0,)),            # 3 blocks: neither
    (2, (6, 8, 16), (1, 8, 16), (11, 1, 1), (0, 1)),         # 6 blocks: the fewest
    (2, (6, 8, 16), (1, 8, 16), (7, 1, 1), (0, 1)),          # walks of 4, 5 and 6 blocks
    (2, (5, 13, 37), (1, 8, 16), (3, 3, 3), (0, 1)),         # odd counts, cut tiles with idle items, walks of one block
    (2, (3, 13, 40), (2, 8, 16), (3, 3, 3), (0, 1)),         # tiles of two blocks
    (2, (4, 13, 20), (1, 7, 11), (3, 3, 3), (0, 1)),         # 77 tokens: three sub-blocks, keys in two
    (2, (5, 7, 18), (3, 4, 4), (3, 3, 5), (0, 1)),           # 48 tokens: two sub-blocks, keys in four
    (2, (4, 14, 18), (2, 4, 4), (3, 3, 3), (0, 1)),          # 32 tokens: one sub-block, keys in four
    (40, (4, 8, 26), (2, 4, 4), (3, 3, 3), (0, 39)),         # 1120 items: too many to split
    (40, (6, 8, 26), (3, 4, 4), (3, 3, 3), (0, 39)),         # 1120 items
    (40, (4, 14, 22), (1, 7, 11), (3, 3, 3), (0, 39)),       # 640 items
    (5, (5, 20, 43), (1, 7, 11), (3, 3, 3), (0, 4)),         # 300 items of three waves
]


@pytest.mark.parametrize("prec,vscale", [(fps.PREC_FP8, fps.VSCALE_TILE), (fps.PREC_FP8, fps.VSCALE_CHANNEL),
                                         (fps.PREC_BF16, fps.VSCALE_TILE)])
@pytest.mark.parametrize("heads,grid,tile,window,compared", SPLIT_CASES)
def test_keys_split_over_wave_groups(prec, vscale, heads, grid, tile, window, compared):
    say("split", prec, vscale, heads, grid, tile, window)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=heads, n_outlier=3, config_id=17)
    run = gu.GpuRun(w)
    out, vis = run.attn(prec, vscale=vscale, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, window))
    for h in compared:
        st = gu.compare_head(run, out, h, prec, window, vscale=vscale)
        say("  head", h, st)
        gu.assert_parity(st, f"{grid} {tile} head {h}")


@pytest.mark.parametrize("prec,vscale", [(fps.PREC_FP8, fps.VSCALE_TILE), (fps.PREC_FP8, fps.VSCALE_CHANNEL),
                                         (fps.PREC_BF16, fps.VSCALE_TILE)])
def test_keys_split_over_wave_groups_of_tiles_in_sub_tiles(prec, vscale):
    """Tiles of two 128-slot scale groups, cut along every axis."""
    say("split, sub-tiles", prec, vscale)
    w = dataclasses.replace(synth.TINY, grid=(3, 13, 40), tile=(2, 8, 16), window=(3, 3, 3), heads=2, n_outlier=3,
                            config_id=18)
    run = gu.GpuRun(w, qtile=(1, 8, 16))
    out = run.attn(prec, vscale=vscale)
    for h in range(2):
        st = gu.compare_head(run, out, h, prec, w.window, vscale=vscale)
        say("  head", h, st)
        gu.assert_parity(st, f"head {h}")


# heads, grid, tile, sub-tile, window, heads compared
NARROW_CASES = [
    (1, (7, 13, 37), (1, 8, 16), None, (3, 3, 3), (0,)),     # 42 items of 128 rows: 32 rows each, keys in four
    (1, (7, 8, 16), (1, 8, 16), None, (13, 1, 1), (0,)),     # 7 blocks: groups of one and of two
    (2, (3, 13, 40), (2, 8, 16), None, (3, 3, 3), (0, 1)),   # 48 items, two blocks a tile, idle waves
    (3, (6, 13, 37), (1, 8, 16), None, (3, 3, 3), (0, 2)),   # 108 items: 64 rows, keys in two; blocks of 8, 5, 7 and 3 halves
    (4, (3, 13, 40), (2, 8, 16), (1, 8, 16), (3, 3, 3), (0, 3)),   # 96 items, two scale groups a tile
    (3, (6, 13, 37), (1, 8, 16), None, (5, 3, 3), (0, 2)),   # 108 items of up to 30 blocks: FP8 keys in four
    (2, (7, 13, 37), (2, 8, 16), None, (5, 3, 3), (0, 1)),   # 96 items of up to 48, two blocks a tile
    (5, (5, 21, 37), (1, 8, 16), None, (3, 3, 3), (0, 4)),   # 225 items of very different length
    (13, (2, 24, 48), (1, 8, 16), None, (3, 5, 5), (0, 12)),   # 234 items of like length: 128 rows, keys in two
    (3, (10, 24, 48), (1, 8, 16), None, (5, 5, 5), (0, 2)),  # 270 items of up to 1.25 times the mean: 128 rows
    (6, (15, 8, 48), (1, 8, 16), None, (29, 1, 5), (5,)),    # 270 of one length: FP8 64 rows
    (5, (7, 21, 37), (1, 8, 16), None, (7, 3, 3), (4,)),     # 315 of twice the mean: FP8 64 rows, more than fit at once
]


@pytest.mark.parametrize("prec,vscale,f32", [(fps.PREC_FP8, fps.VSCALE_TILE, True), (fps.PREC_FP8, fps.VSCALE_CHANNEL, True),
                                             (fps.PREC_FP8, fps.VSCALE_TILE, False), (fps.PREC_BF16, fps.VSCALE_TILE, True),
                                             (fps.PREC_BF16, fps.VSCALE_TILE, False)])
@pytest.mark.parametrize("heads,grid,tile,qtile,window,compared", NARROW_CASES)
def test_narrow_items(prec, vscale, f32, heads, grid, tile, qtile, window, compared):
    """Launches of few items: 32 (FP8) or 64 rows each, the keys shared by four or two wave groups."""
    say("narrow items", prec, vscale, f32, heads, grid, tile, qtile, window)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=heads, n_outlier=3, config_id=27)
    run = gu.GpuRun(w, qtile=qtile)
    out, vis = run.attn(prec, vscale=vscale, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, window))
    if not f32:
        import torch
        half = run.attn(prec, vscale=vscale, out_dtype=torch.bfloat16)
        assert torch.equal(half, out.to(torch.bfloat16))
        return
    for h in compared:
        st = gu.compare_head(run, out, h, prec, window, vscale=vscale)
        say("  head", h, st)
        gu.assert_parity(st, f"{grid} {tile} head {h}")


# heads, grid, tile, sub-tile, window, shifted, heads compared: 129 to 256 items of 128 rows that are not cut, keys in two groups
# of four waves
WHOLE_SPLIT_CASES = [
    (5, (5, 13, 37), (1, 8, 16), None, (3, 1, 3), False, (0, 4)),          # 150 items of up to 9 blocks, idle waves, odd counts
    (6, (4, 13, 37), (1, 8, 16), None, (9, 9, 9), True, (0, 5)),           # 144 items of 24, all of one length
    (5, (7, 13, 20), (2, 8, 16), None, (3, 1, 1), False, (0, 4)),          # 160 items, two blocks a tile, one of them cut off
    (6, (4, 13, 40), (2, 8, 16), None, (1, 3, 3), False, (0, 5)),          # 144 items of 12
    (6, (4, 13, 40), (2, 8, 16), (1, 8, 16), (1, 3, 3), True, (0, 5)),     # and a scale group each
]


@pytest.mark.parametrize("prec,vscale", [(fps.PREC_FP8, fps.VSCALE_TILE), (fps.PREC_FP8, fps.VSCALE_CHANNEL),
                                         (fps.PREC_BF16, fps.VSCALE_TILE)])
@pytest.mark.parametrize("heads,grid,tile,qtile,window,shift,compared", WHOLE_SPLIT_CASES)
def test_keys_split_over_groups_of_four_waves(prec, vscale, heads, grid, tile, qtile, window, shift, compared):
    say("split, whole items", prec, vscale, heads, grid, tile, qtile, window, shift)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=heads, n_outlier=3, config_id=29)
    win = window + ((fps.EDGE_SHIFT,) if shift else ())
    run = gu.GpuRun(w, qtile=qtile)
    out, vis = run.attn(prec, window=win, vscale=vscale, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, win))
    for h in compared:
        st = gu.compare_head(run, out, h, prec, win, vscale=vscale)
        gu.assert_parity(st, f"{grid} {tile} head {h}")


# heads, grid, tile, sub-tile, window: every kernel of few items of 128-slot tiles
RASTER_CASES = [
    (1, (7, 13, 37), (1, 8, 16), None, (3, 3, 3)),           # 42 items
    (2, (3, 13, 40), (2, 8, 16), None, (3, 3, 3)),           # 48, two blocks a tile
    (3, (6, 13, 37), (1, 8, 16), None, (3, 3, 3)),           # 108
    (4, (3, 13, 40), (2, 8, 16), (1, 8, 16), (3, 3, 3)),     # 96, two scale groups a tile
    (3, (6, 13, 37), (1, 8, 16), None, (5, 3, 3)),           # 108 of up to 30 blocks
    (2, (7, 13, 37), (2, 8, 16), None, (5, 3, 3)),           # 96 of up to 48
    (5, (5, 13, 37), (1, 8, 16), None, (3, 1, 3)),           # 150, not cut
    (6, (4, 13, 40), (2, 8, 16), None, (1, 3, 3)),           # 144
]


@pytest.mark.parametrize("prec,vscale", [(fps.PREC_FP8, fps.VSCALE_TILE), (fps.PREC_FP8, fps.VSCALE_CHANNEL),
                                         (fps.PREC_BF16, fps.VSCALE_TILE)])
@pytest.mark.parametrize("heads,grid,tile,qtile,window", RASTER_CASES)
def test_few_items_in_raster_order_and_shifted_windows(prec, vscale, heads, grid, tile, qtile, window):
    """The output a caller of the fused entry points gets: fp32 and bf16, every element of a NaN-filled buffer, the same numbers
    as in tile order; windows shifted at the grid's edges."""
    import torch
    say("few items, raster, shifted", prec, vscale, heads, grid, tile, qtile, window)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=heads, n_outlier=3, config_id=30)
    win = window + (fps.EDGE_SHIFT,)
    run = gu.GpuRun(w, qtile=qtile)
    tiled = run.attn(prec, window=win, vscale=vscale)
    st = gu.compare_head(run, tiled, heads - 1, prec, win, vscale=vscale)
    gu.assert_parity(st, f"{grid} {tile}")
    want = fps.tile_unorder(run.shape, tiled)
    if prec == fps.PREC_FP8:
        (q, sq), (k, sk), (v, sv) = run.q8
    else:
        (q, sq), (k, sk), (v, sv) = run.p16
    for dtype in (torch.float32, torch.bfloat16):
        out = torch.full((1, heads) + grid + (128,), float("nan"), dtype=dtype, device="cuda:0")
        fps.attn_fwd(run.shape, win, prec, q, k, v, sq, sk, sv, vscale=vscale, out=out, raster_out=True)
        assert torch.equal(out, want.to(dtype))


# heads, grid, tile, sub-tile, window: more keys than the L2s hold, so that the last items of an XCD are dealt by length
TAIL_CASES = [
    (40, (3, 45, 80), (1, 8, 16), None, (3, 3, 3)),          # one item a tile
    (36, (4, 30, 52), (2, 8, 16), None, (1, 3, 3)),          # two
    (28, (6, 30, 52), (6, 8, 8), None, (1, 3, 3)),           # three
    (42, (3, 30, 52), (3, 4, 4), None, (1, 5, 7)),           # small groups: two waves
    (18, (8, 30, 52), (2, 8, 16), (1, 8, 8), (1, 3, 3)),     # and four
    (70, (4, 30, 52), (2, 4, 4), None, (1, 5, 5)),           # one
]


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("heads,grid,tile,qtile,window", TAIL_CASES)
def test_the_end_of_a_long_launch_is_dealt_once(prec, heads, grid, tile, qtile, window):
    """Every head has the same inputs: every slot of a NaN-filled output is written, all heads alike, one against the oracle."""
    import torch
    say("tail", prec, heads, grid, tile, qtile, window)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=1, n_outlier=3, config_id=31)
    run = gu.GpuRun(w, qtile=qtile)
    run.quantize()
    shape = fps.make_shape(heads, grid, tile, qtile=qtile)
    assert 2 * heads * run.g.M * run.tsp * (128 if prec == fps.PREC_FP8 else 256) > 64 << 20
    packed, scales = [], []
    for role in range(3):
        x = run.raster[role].expand((1, heads) + grid + (128,)).contiguous()
        p, s = (fps.quantize_tiles(shape, x, role, raster=True) if prec == fps.PREC_FP8 else
                fps.pack_tiles_bf16(shape, x, role, raster=True))
        packed.append(p)
        scales.append(s)
    out = torch.full((1, heads, run.g.M * run.tsp, 128), float("nan"), dtype=torch.float32, device="cuda:0")
    fps.attn_fwd(shape, window, prec, *packed, *scales, out=out)
    assert torch.isfinite(out).all()
    assert torch.equal(out, out[:, :1].expand_as(out))
    tiles = [u for u in gu.sample_q_tiles(run.g, np.random.default_rng(4)) if u < run.g.M]    # one layer has no interior
    st = gu.compare_head(run, out[:, :1], 0, prec, window, q_tiles=tiles)
    # the padding rows of every tile are zero, the sampled tiles within the bars
    gu.assert_parity(st, f"tail {grid} {tile}")


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("heads,grid,tile,qtile,window,shift", [
    (40, (3, 13, 40), (1, 8, 16), None, (3, 3, 3), False),        # 720 items, cut along h and w
    (10, (3, 26, 70), (1, 8, 16), None, (3, 3, 3), True),         # 600
    (14, (5, 13, 20), (2, 8, 16), None, (3, 3, 3), False),        # 336: two query blocks a tile, idle ones in cut tiles
    (12, (5, 13, 20), (2, 8, 16), (1, 8, 16), (3, 3, 3), False),  # 288, a scale group each
    (8, (14, 13, 20), (6, 8, 8), None, (3, 3, 1), False),         # 432: three query blocks
    (8, (9, 30, 20), (4, 16, 16), None, (3, 1, 3), False),        # 768: eight query blocks
    (20, (5, 14, 33), (1, 7, 11), None, (5, 1, 5), False),        # three waves
    (12, (7, 8, 37), (3, 4, 4), None, (3, 3, 3), False),          # two waves
    (60, (4, 10, 30), (2, 4, 4), None, (3, 5, 3), False)])        # 2880 one-wave workgroups
def test_items_dealt_by_length(prec, heads, grid, tile, qtile, window, shift):
    """Launches of more workgroups than CUs whose heads fit an XCD's L2 and whose walks are of different length: each item
    once."""
    say("by length", prec, heads, grid, tile, qtile, window, shift)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=heads, n_outlier=3, config_id=26)
    win = window + ((fps.EDGE_SHIFT,) if shift else ())
    run = gu.GpuRun(w, qtile=qtile)
    mask = fo.tile_mask(run.g, win)
    # what the rule asks for, so that no case is dealt in raster order unnoticed: items, blocks of the longest walk (its
    # keys in blocks of at most 128), longest walk over the mean
    tsp = fps.tile_slots(run.shape)
    sb = 4 if fps.block_slots(run.shape) == 128 else tsp // 32
    items, blocks = heads * run.g.M * (tsp // 32 // sb), int(mask.sum(1).max()) * max(1, tsp // 128)
    keys = mask @ fo.valid_tokens(run.g).reshape(run.g.M, -1).sum(1)
    assert items > (2048 if sb == 1 else 256) and blocks >= 12 and keys.max() > 1.12 * keys.mean()
    assert 2 * heads * run.g.M * tsp * (128 if prec == fps.PREC_FP8 else 256) <= 64 << 20
    out, vis = run.attn(prec, window=win, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), mask)
    tiles = None if run.g.L_padded < 6000 else gu.sample_q_tiles(run.g, np.random.default_rng(3))
    for h in (0, heads - 1):
        st = gu.compare_head(run, out, h, prec, win, q_tiles=tiles)
        gu.assert_parity(st, f"by length head {h}")


@pytest.mark.parametrize("vscale", [fps.VSCALE_TILE, fps.VSCALE_CHANNEL])
@pytest.mark.parametrize("tile,qtile", [((2, 4, 4), None), ((3, 4, 4), None), ((2, 8, 4), None),
                                        ((2, 4, 8), (1, 4, 4)), ((2, 8, 8), (2, 4, 8)), ((1, 4, 12), (1, 4, 4))])
@pytest.mark.parametrize("tiles,window", [(1, 1), (4, 3), (5, 5), (9, 9)])
def test_small_groups_two_or_four_a_step(vscale, tile, qtile, tiles, window):
    """Lists of 1, 2, 3, .. blocks of small scale groups, of which the kernel takes two or four at a time."""
    say("groups a step", vscale, tile, qtile, tiles, window)
    w = dataclasses.replace(synth.TINY, grid=(tile[0], tile[1], tile[2] * tiles - 1), tile=tile, window=(1, 1, window),
                            heads=2, n_outlier=3, config_id=27)
    run = gu.GpuRun(w, qtile=qtile)
    out = run.attn(fps.PREC_FP8, vscale=vscale)
    for h in range(2):
        st = gu.compare_head(run, out, h, fps.PREC_FP8, w.window, vscale=vscale)
        gu.assert_parity(st, "groups a step")


@pytest.mark.parametrize("vscale", [fps.VSCALE_TILE, fps.VSCALE_CHANNEL])
@pytest.mark.parametrize("tile,qtile", [((2, 4, 4), None), ((3, 4, 4), None), ((2, 8, 16), (1, 8, 8)),
                                        ((2, 8, 8), (2, 4, 8)), ((2, 4, 8), (1, 4, 4)), ((1, 4, 12), (1, 4, 4))])
@pytest.mark.parametrize("rise", [1.25, 2.0])
def test_blocks_taken_together_keep_their_weights_bits(vscale, tile, qtile, rise):
    """Of the first four scale groups each has scores 2^20 (or 2^32) times the last one's weights, and channels of V to itself:
    a group's weights are rounded against the largest score met so far, not against one of a group still to come, or
    its channels would be lost.  Every key of a group has one score, so 448 P is one number between 224 and 448, whose
    code is off by at most 2^-4 of it; V's codes are exact, its sums of one sign within the matrix instruction's 2^-11."""
    import torch
    say("weights' bits", vscale, tile, qtile, rise)
    q = qtile or tile
    per_tile = tile[0] * tile[1] * tile[2] // (q[0] * q[1] * q[2])
    n = -(-36 // per_tile)                                  # walks of at least 36 blocks
    grid, heads = (tile[0], tile[1], tile[2] * n), 24       # too many items for a split of the keys
    shape = fps.make_shape(heads, grid, tile, qtile=qtile)
    at = [torch.arange(size) // s for size, s in zip(grid, q)]
    nh, nw = grid[1] // q[1], grid[2] // q[2]
    rank = (at[0][:, None, None] * nh + at[1][None, :, None]) * nw + at[2][None, None, :]     # order of the groups
    level = rank.clamp(max=3)
    shade = torch.tensor([1.0, 1.5, 1.75])[torch.arange(rank.numel()).view(rank.shape) % 3]
    key = (rise * level).double()
    val = torch.zeros(grid + (128,))
    for r in range(4):
        val[..., r::4] = torch.where(level == r, shade, torch.zeros(()))[..., None]
    score = 128 * key.view(-1) / math.sqrt(128)
    want = torch.softmax(score, 0) @ val.view(-1, 128).double()

    def on_device(x):
        return x.to("cuda:0", torch.bfloat16).expand((1, heads) + grid + (128,)).contiguous()
    packed = [fps.quantize_tiles(shape, on_device(x), role, vscale=vscale, raster=True)
              for role, x in enumerate((torch.ones(grid + (128,)), key[..., None], val))]
    (qq, sq), (kq, sk), (vq, sv) = packed
    out = fps.attn_fwd(shape, (1, 1, 2 * n - 1), fps.PREC_FP8, qq, kq, vq, sq, sk, sv, vscale=vscale,
                       out_dtype=torch.float32, raster_out=True)
    off = (out.double().cpu() / want - 1).abs().amax()
    say("  largest relative error", float(off))
    assert off <= 2.0 ** -4 + 2.0 ** -10


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("heads", [1, 8])                 # keys split over wave groups, and not
@pytest.mark.parametrize("tile,qtile", [((1, 8, 16), None), ((2, 8, 16), None), ((2, 4, 4), None),
                                        ((2, 8, 16), (1, 8, 8))])
@pytest.mark.parametrize("blocks", [64, 66, 130])
def test_lists_of_key_blocks_longer_than_a_wave(prec, heads, tile, qtile, blocks):
    """The kernels list the next 64 key blocks at a time, one a lane: walks that end with, just past and well past
    a full list, one row of tiles whose last is cut."""
    say("block lists", prec, heads, tile, qtile, blocks)
    slots = tile[0] * tile[1] * tile[2]
    per_tile = 4 if qtile else max(1, slots // 128)
    n = blocks // per_tile + 1                             # the whole tiles' walk is the longest
    w = dataclasses.replace(synth.TINY, grid=(tile[0], tile[1], tile[2] * n - tile[2] // 2), tile=tile,
                            window=(1, 1, 2 * n - 1), heads=heads, n_outlier=3, config_id=25)
    run = gu.GpuRun(w, qtile=qtile)
    out = run.attn(prec)
    st = gu.compare_head(run, out, heads - 1, prec, w.window, q_tiles=[0, n - 1])
    gu.assert_parity(st, "block lists")


@pytest.mark.parametrize("tile,qtile", [((2, 4, 4), None), ((3, 4, 4), None), ((2, 4, 8), (1, 4, 4)), ((1, 4, 12), (1, 4, 4)),
                                        ((3, 6, 8), (1, 6, 8)), ((2, 8, 8), (2, 4, 8))])
@pytest.mark.parametrize("blocks,vscale", [(65, fps.VSCALE_TILE), (67, fps.VSCALE_CHANNEL), (130, fps.VSCALE_TILE)])
def test_lists_of_small_groups_longer_than_a_wave(tile, qtile, blocks, vscale):
    """Every kernel that takes two or four small groups a step, on a list of more than 64 whose last step is not full: one
    row of groups, the last of them cut, in too many items for a split of the keys."""
    say("lists of small groups", tile, qtile, blocks, vscale)
    q = qtile or tile
    w = dataclasses.replace(synth.TINY, grid=(q[0], q[1], q[2] * blocks + q[2] // 2), tile=tile, window=(1, 1, 299), heads=8,
                            n_outlier=3, config_id=28)
    run = gu.GpuRun(w, qtile=qtile)
    out = run.attn(fps.PREC_FP8, vscale=vscale)
    st = gu.compare_head(run, out, 7, fps.PREC_FP8, w.window, vscale=vscale, q_tiles=[0, run.g.M - 1])
    gu.assert_parity(st, "lists of small groups")


@pytest.mark.parametrize("tile,qtile", [((1, 1, 1), None), ((1, 1, 2), (1, 1, 1))])
def test_heads_of_a_million_blocks(tile, qtile):
    """Heads whose block numbers are beyond what a division by a float reciprocal gives exactly.  BF16: the weights are
    rounded to 2^-12 of themselves, the rest is fp32."""
    import torch
    say("a million blocks", tile, qtile)
    grid, tw = (1, 1024, 1024), tile[2]
    shape = fps.make_shape(1, grid, tile, qtile=qtile)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    x = [torch.randn((1, 1) + grid + (128,), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(3)]
    packed = [fps.pack_tiles_bf16(shape, t, role, raster=True) for role, t in enumerate(x)]
    out = fps.attn_fwd(shape, (1, 3, 3), fps.PREC_BF16, packed[0][0], packed[1][0], packed[2][0], sv=packed[2][1],
                       out_dtype=torch.float32, raster_out=True)[0, 0, 0]
    del packed
    q, k, v = (t[0, 0, 0].float() for t in x)
    offsets = [(dh, dw) for dh in (-1, 0, 1) for dw in range(1 - 2 * tw, 2 * tw)]
    row, col = torch.arange(1024, device="cuda:0")[:, None], torch.arange(1024, device="cuda:0")[None, :]

    def beside(t, o):
        return torch.roll(t, (-o[0], -o[1]), (0, 1))
    scores = []
    for o in offsets:
        r, c = row + o[0], col + o[1]
        kept = (r >= 0) & (r < 1024) & (c >= 0) & (c < 1024) & ((c // tw - col // tw).abs() <= 1)
        scores.append(((q * beside(k, o)).sum(-1) / math.sqrt(128)).masked_fill(~kept, float("-inf")))
    p = torch.softmax(torch.stack(scores), 0)
    want, size = torch.zeros_like(out), torch.zeros_like(out)
    for i, o in enumerate(offsets):
        want += p[i][..., None] * beside(v, o)
        size += p[i][..., None] * beside(v, o).abs()
    excess = ((out - want).abs() - 2.0 ** -11 * size).amax()
    say("  largest error beyond the weights' rounding", float(excess))
    assert excess <= 0


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("tile,rest", [((1, 1, 128), r) for r in (1, 31, 32, 33, 64, 65, 96, 97, 127)] +
                         [((1, 2, 128), r) for r in (1, 48, 63, 64, 65, 127)])
def test_cut_tiles_at_the_edges_of_sub_blocks(prec, tile, rest):
    """A tile cut by the grid's edge holds its real tokens first and is walked by 32-key sub-blocks:
    every count of them, one token to either side of each boundary, with one and two blocks a tile,
    for keys and for query rows, in both output layouts."""
    import torch
    say("cut tiles", prec, tile, rest)
    w = dataclasses.replace(synth.TINY, grid=(2, 2 * tile[1] + 1, 128 + rest), tile=tile, window=(3, 3, 3), heads=1,
                            n_outlier=3, config_id=31)
    run = gu.GpuRun(w)
    out = run.attn(prec)
    st = gu.compare_head(run, out, 0, prec, w.window)
    say("  ", st)
    gu.assert_parity(st, f"{tile} rest {rest}")
    assert torch.equal(run.attn(prec, raster_out=True), fps.tile_unorder(run.shape, out))
    if prec == fps.PREC_FP8:
        _check_quantize(run, [0], f"cut {tile} {rest}")


@pytest.mark.parametrize("heads", [1, 40])                # keys split over wave groups, and not
@pytest.mark.parametrize("grid,tile", [((4, 12, 12), (2, 4, 4)), ((6, 12, 12), (3, 4, 4)), ((3, 15, 48), (1, 5, 16)),
                                       ((3, 24, 48), (1, 8, 16)), ((4, 16, 48), (2, 8, 16))])
@pytest.mark.parametrize("outlying", ["zero", "large"])
def test_bf16_v_groups_of_very_different_magnitude(outlying, grid, tile, heads):
    """One V tile of zeros, or of values 2^34 times the others' whose keys have no weight, beside tiles
    of values of 1e-6: the other tiles' weights keep their bits."""
    say("V magnitudes", outlying, grid, tile, heads)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=(3, 3, 3), heads=heads, n_outlier=0, config_id=35)
    q, k, v = (a.copy() for a in synth.qkv_raster(dataclasses.replace(w, heads=1), 0, [0]))
    v *= np.float32(1e-6)
    group = np.s_[0, tile[0]:2 * tile[0], tile[1]:2 * tile[1], tile[2]:2 * tile[2]]
    if outlying == "zero":
        v[group] = 0.0
    else:
        q, k[group] = np.abs(q), -16 * np.abs(k[group])    # scores about -190: weights below 2^-100
        v[group] *= np.float32(2.0 ** 34)
    run = gu.GpuRun(w, qkv=[np.repeat(synth.round_to_bf16(a), heads, axis=0) for a in (q, k, v)])
    out = run.attn(fps.PREC_BF16)
    st = gu.compare_head(run, out, heads - 1, fps.PREC_BF16, w.window)
    say("  ", st)
    gu.assert_parity(st, f"{outlying} {grid} {tile}")


SMALL_GROUP_CASES = [                            # tile, sub-tile; key blocks of 1, 2 or 3 sub-blocks
    ((1, 1, 1), None), ((1, 1, 17), None), ((2, 4, 4), None),                     # one wave a workgroup
    ((1, 3, 11), None), ((3, 4, 4), None), ((1, 8, 8), None),                     # two
    ((1, 5, 13), None), ((1, 5, 16), None), ((2, 3, 16), None),                   # three: 65, 80, 96 tokens
    ((2, 4, 8), (1, 4, 4)), ((1, 4, 12), (1, 4, 4)),              # 4 and 3 sub-tiles of 16: four waves, one
    ((2, 8, 8), (2, 4, 8)), ((3, 6, 8), (1, 6, 8)),               # 2 and 3 sub-tiles of 64 and 48: four, two
    ((2, 10, 16), (1, 5, 16)), ((1, 10, 16), (1, 5, 16)),         # 4 and 2 sub-tiles of 80: four, three
]


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
@pytest.mark.parametrize("tile,qtile", SMALL_GROUP_CASES)
def test_small_scale_groups_for_every_workgroup_shape(prec, tile, qtile):
    """Scale groups of at most 96 tokens: every number of sub-blocks and waves, with tiles cut along
    h and w (so that groups hold fewer tokens, or none) and a window that leaves tiles out."""
    import torch
    say("small groups", prec, tile, qtile)
    grid = (2 * tile[0], max(1, 3 * tile[1] - tile[1] // 2), max(1, 4 * tile[2] - (2 * tile[2]) // 3))
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=(3, 3, 3), heads=2, n_outlier=3, config_id=33)
    run = gu.GpuRun(w, qtile=qtile)
    out, vis = run.attn(prec, visited=True)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, w.window))
    st = gu.compare_head(run, out, 1, prec, w.window)
    say("  ", st)
    gu.assert_parity(st, f"{tile} {qtile}")
    assert torch.equal(run.attn(prec, raster_out=True), fps.tile_unorder(run.shape, out))
    if prec == fps.PREC_FP8:
        _check_quantize(run, range(2), f"small groups {tile} {qtile}")
        out = run.attn(prec, vscale=fps.VSCALE_CHANNEL)
        st = gu.compare_head(run, out, 1, prec, w.window, vscale=fps.VSCALE_CHANNEL)
        gu.assert_parity(st, f"{tile} {qtile} per-channel V")


@pytest.mark.parametrize("tile,qtile", SMALL_GROUP_CASES + [((1, 8, 16), None), ((2, 8, 16), None), ((3, 9, 10), None),
                                                            ((2, 8, 16), (1, 8, 16))])
def test_bf16_packing_for_every_block_shape(tile, qtile):
    """One to three blocks of 32 or 128 slots a group, whole and cut: the fused and the separate call
    give the same bytes, and V's scales are those of the groups' largest values."""
    import torch
    say("bf16 packing", tile, qtile)
    grid = (2 * tile[0], max(1, 3 * tile[1] - tile[1] // 2), max(1, 4 * tile[2] - (2 * tile[2]) // 3))
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=(3, 3, 3), heads=3, n_outlier=3, config_id=36)
    run = gu.GpuRun(w, qtile=qtile)
    for role, (xp, vs) in enumerate(run.pack_bf16()):
        fused, fused_vs = fps.pack_tiles_bf16(run.shape, run.raster[role], role, raster=True)
        assert torch.equal(xp, fused)
        if role == fps.ROLE_V:
            assert torch.equal(vs, fused_vs)
            for h in range(3):
                _, scales = fo.quantize_tiles(fo.tile_order(run.qkv[role][h].astype(np.float64), run.g), run.g)
                amax = synth.round_to_bf16(scales.astype(np.float32) * np.float32(448.0))   # the scales are amax / 448
                want = np.where(amax > 0, np.exp2(np.floor(np.log2(amax)) - 14.0), 1.0)
                real = _groups_with_tokens(run.g)
                assert np.array_equal(vs[0, h].cpu().numpy()[real], want[real])
        else:
            assert vs is None and fused_vs is None


def _groups_with_tokens(g):
    """Groups that hold a real token (the scale of the others is 1 by definition)."""
    return np.flatnonzero(fo.quantize_tiles(np.repeat(fo.valid_tokens(g)[:, None], 128, axis=1).astype(np.float64), g)[1] != 1.0)


@pytest.mark.parametrize("heads,tile", [(5, (2, 4, 4)), (12, (2, 4, 4)), (45, (2, 4, 4)), (45, (2, 8, 8)), (90, (2, 4, 4)),
                                        (90, (2, 8, 8))])
def test_per_channel_maxima_of_many_blocks(heads, tile):
    """1, 2 and 8 blocks a workgroup, the last of a head with fewer, and (90 heads) read past the caches: every channel's scale,
    wherever its maximum is."""
    import torch
    say("per-channel maxima", heads, tile)
    grid = (9, 27, 42)                                      # 385 blocks a head, of 32 slots, or of 128: 120
    shape = fps.make_shape(heads, grid, tile)
    gen = torch.Generator(device="cuda:0").manual_seed(heads)
    x = torch.randn((1, heads) + grid + (128,), generator=gen, device="cuda:0", dtype=torch.bfloat16)
    flat = x.view(heads, -1, 128)
    for c in range(128):                                    # a maximum of its own, in the first, last or another token
        at = [0, flat.shape[1] - 1, (c * 7919) % flat.shape[1]][c % 3]
        flat[:, at, c] = 8.0 + c * (-1) ** c
    want = (flat.float().abs().amax(dim=1).cpu() / torch.tensor(448.0)).numpy()
    for raster in (True, False):
        src = x if raster else fps.tile_order(shape, x)
        _, sc = fps.quantize_tiles(shape, src, fps.ROLE_V, vscale=fps.VSCALE_CHANNEL, raster=raster)
        assert np.array_equal(sc[0].cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("grid,tile,window", [((4, 16, 16), (2, 4, 4), (1, 3, 3)),
                                              ((2, 13, 40), (1, 8, 16), (3, 3, 3)),
                                              ((3, 13, 20), (2, 8, 16), (3, 3, 3))])
def test_per_channel_v_scales(grid, tile, window):
    """The paper's own V quantisation (Sec. 3.2): one scale per channel over all tokens."""
    import torch
    say("per-channel V", grid, tile)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window, heads=2, n_outlier=3,
                            config_id=13)
    run = gu.GpuRun(w)
    xq, sc = fps.quantize_tiles(run.shape, run.tiled[2], fps.ROLE_V, vscale=fps.VSCALE_CHANNEL)
    xq_r, sc_r = fps.quantize_tiles(run.shape, run.raster[2], fps.ROLE_V, vscale=fps.VSCALE_CHANNEL,
                                    raster=True)
    assert torch.equal(xq, xq_r) and torch.equal(sc, sc_r) and sc.shape == (1, 2, 128)
    codes = fps.debug_unpack_q8(run.shape, xq, fps.ROLE_V)[0].cpu().numpy()
    for h in range(2):
        wc, ws = fo.quantize_channels(fo.tile_order(run.qkv[2][h].astype(np.float64), run.g))
        assert np.array_equal(sc[0, h].cpu().numpy(), ws)
        got = codes[h][run.slots]
        zero_sign = ((got ^ wc) == 0x80) & ((wc & 0x7F) == 0)
        assert int(((got != wc) & ~zero_sign).sum()) == 0
    out = run.attn(fps.PREC_FP8, vscale=fps.VSCALE_CHANNEL)
    for h in range(2):
        st = gu.compare_head(run, out, h, fps.PREC_FP8, window, vscale=fps.VSCALE_CHANNEL)
        say("  head", h, st)
        gu.assert_parity(st, f"per-channel V head {h}")


@pytest.mark.parametrize("prec", [fps.PREC_FP8, fps.PREC_BF16])
def test_shifted_window_edge_rule(prec):
    say("shifted window", prec)
    w = dataclasses.replace(synth.TINY, grid=(5, 13, 40), tile=(1, 8, 16), window=(3, 1, 3), heads=1,
                            n_outlier=3, config_id=14)
    run = gu.GpuRun(w)
    win = w.window + (fps.EDGE_SHIFT,)
    out, vis = run.attn(prec, window=win, visited=True)
    mask = fo.tile_mask(run.g, win)
    assert np.array_equal(vis.cpu().numpy().astype(bool), mask)
    assert np.all(mask.sum(axis=1) == 3 * 1 * 3)
    st = gu.compare_head(run, out, 0, prec, win)
    say("  ", st)
    gu.assert_parity(st, "shifted window")


def test_shared_outlier_channels_stress():
    """Q and K share their outlier channels: the score spread is ~10x larger (|S'| ~ 100, rows
    close to one-hot), outside the input distribution the tolerances are stated for.  The error of
    the hardware's FP8 accumulation (about 2^-14 of sum|q_c k_c|) then moves the softmax weights
    themselves by a few 1e-3, so only looser bounds are asserted here: finite, padded rows zero,
    max excess <= 1e-1 RMS, mean <= 5e-3 RMS."""
    say("attention stress")
    w = dataclasses.replace(synth.TINY, grid=(2, 8, 32), tile=(1, 8, 16), window=(3, 1, 3), heads=1,
                            config_id=8)
    q, k, v = synth.qkv_raster(w)
    q_out = q.reshape(-1, 128).std(axis=0) > 4
    k_out = k.reshape(-1, 128).std(axis=0) > 4
    k = k.copy()
    k[..., k_out] /= 8                                     # undo K's own outlier channels ...
    k[..., q_out] *= 8                                     # ... and put them where Q has its own
    k = synth.round_to_bf16(k)
    run = gu.GpuRun(w, qkv=(q, k, v))
    out = run.attn(fps.PREC_FP8)
    st = gu.compare_head(run, out, 0, fps.PREC_FP8, w.window)
    say("  ", st)
    assert st["finite"] and st["pad_rows_zero"]
    assert st["max_excess"] <= 1e-1 and st["mean_err"] <= 5e-3


def test_garbage_in_padded_slots_cannot_leak():
    import torch
    say("attention padded garbage")
    w = dataclasses.replace(synth.TINY, grid=(2, 13, 40), tile=(1, 8, 16), window=(3, 3, 3), heads=1,
                            n_outlier=3, config_id=9)
    run = gu.GpuRun(w)
    clean = run.attn(fps.PREC_FP8).clone()
    pad = torch.from_numpy(run.pad_slots()).to("cuda:0")
    for t in run.tiled:
        t[0, 0, pad] = 0.0078125                        # small: cannot raise any tile's amax
    del run.q8
    dirty = run.attn(fps.PREC_FP8)
    assert torch.equal(clean, dirty)


def test_bf16_output_is_rounded_fp32_output(tiny):
    import torch
    say("bf16 output")
    o32 = tiny.attn(fps.PREC_FP8, out_dtype=torch.float32)
    o16 = tiny.attn(fps.PREC_FP8, out_dtype=torch.bfloat16)
    assert torch.equal(o16, o32.to(torch.bfloat16))


@pytest.mark.parametrize("grid,tile", [((4, 16, 16), (2, 4, 4)), ((3, 5, 6), (2, 4, 4)),
                                       ((2, 13, 40), (1, 8, 16)), ((3, 13, 20), (2, 8, 16))])
def test_fused_raster_entry_points_match_the_unfused_path(grid, tile):
    """fps_quantize_raster == fps_tile_order + fps_quantize_tiles (bit for bit), and the raster
    output layout of fps_attn_fwd == fps_tile_unorder of the tiled output."""
    import torch
    say("fused raster", grid, tile)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=(3, 3, 3), heads=2, n_outlier=3,
                            config_id=12)
    run = gu.GpuRun(w)
    q8 = run.quantize()
    for role in range(3):
        xq, sc = fps.quantize_tiles(run.shape, run.raster[role], role, raster=True)
        assert torch.equal(xq, q8[role][0]) and torch.equal(sc, q8[role][1])
    p16 = run.pack_bf16()
    for role in range(3):
        xp, vs = fps.pack_tiles_bf16(run.shape, run.raster[role], role, raster=True)
        assert torch.equal(xp, p16[role][0])
        assert (vs is None and p16[role][1] is None) or torch.equal(vs, p16[role][1])
    for prec in (fps.PREC_FP8, fps.PREC_BF16):
        for dt in (torch.float32, torch.bfloat16):
            tiled = run.attn(prec, out_dtype=dt)
            raster = run.attn(prec, out_dtype=dt, raster_out=True)
            assert raster.shape == (1, 2) + tuple(grid) + (128,)
            assert torch.equal(raster, fps.tile_unorder(run.shape, tiled))


def test_two_runs_are_bit_identical_and_inputs_stay_untouched(tiny):
    import torch
    say("determinism")
    a = tiny.attn(fps.PREC_FP8).clone()
    before = [t.clone() for pair in tiny.q8 for t in pair] + [t.clone() for t in tiny.raster + tiny.tiled]
    b = tiny.attn(fps.PREC_FP8)
    assert torch.equal(a, b)
    fps.quantize_tiles(tiny.shape, tiny.raster[2], fps.ROLE_V, raster=True)
    fps.quantize_tiles(tiny.shape, tiny.tiled[0], fps.ROLE_Q)
    torch.cuda.synchronize()
    after = [t for pair in tiny.q8 for t in pair] + tiny.raster + tiny.tiled
    assert all(torch.equal(x, y) for x, y in zip(before, after))


def _random_case(rng):
    """A random small configuration: grid, tile, optional quantisation sub-tile, window, edge rule,
    precision, V scale granularity."""
    def divisors(n):
        return [d for d in range(1, n + 1) if n % d == 0]
    while True:
        tile = tuple(int(rng.choice(c)) for c in ([1, 2, 3, 4, 6], [1, 2, 4, 5, 8, 16], [2, 4, 5, 8, 16]))
        ts = tile[0] * tile[1] * tile[2]
        if not 8 <= ts <= 512:
            continue
        n_tiles = (int(rng.integers(1, 4)), int(rng.integers(1, 4)), int(rng.integers(1, 5)))
        grid = tuple(max(1, n * t - int(rng.integers(0, t))) for n, t in zip(n_tiles, tile))
        if grid[0] * grid[1] * grid[2] > 2600:
            continue
        qtile = None
        if rng.random() < 0.4:
            qtile = tuple(int(rng.choice(divisors(t))) for t in tile)
        window = tuple(int(rng.integers(1, 6)) for _ in range(3))
        if rng.random() < 0.3:
            window += (fps.EDGE_SHIFT,)
        prec = fps.PREC_FP8 if rng.random() < 0.7 else fps.PREC_BF16
        vscale = fps.VSCALE_CHANNEL if (prec == fps.PREC_FP8 and rng.random() < 0.3) else fps.VSCALE_TILE
        return grid, tile, qtile, window, prec, vscale


@pytest.mark.parametrize("seed", range(16))
def test_random_configurations(seed):
    """Seeded random shapes, tiles, sub-tiles, windows, edge rules and modes against the oracle."""
    rng = np.random.default_rng(1000 + seed)
    grid, tile, qtile, window, prec, vscale = _random_case(rng)
    say("random case", seed, grid, tile, qtile, window, prec, vscale)
    w = dataclasses.replace(synth.TINY, grid=grid, tile=tile, window=window[:3], heads=1, n_outlier=3,
                            config_id=100 + seed)
    run = gu.GpuRun(w, qtile=qtile)
    out, vis = run.attn(prec, window=window, visited=True, vscale=vscale)
    assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, window))
    if prec == fps.PREC_FP8:
        _check_quantize(run, [0], f"random {seed}") if vscale == fps.VSCALE_TILE else None
    st = gu.compare_head(run, out, 0, prec, window, vscale=vscale)
    say("  ", st)
    gu.assert_parity(st, f"random case {seed}: {grid} {tile} {qtile} {window} {prec} {vscale}")


def test_mfma_rate_kernel_runs():
    """The MFMA-only micro-benchmark kernel (yardstick of the roofline): every thread writes one
    finite value, and a thread's value grows linearly with the trip count (accumulator chains)."""
    import torch
    say("mfma rate")
    a = torch.full((8 * 256,), float("nan"), dtype=torch.float32, device="cuda:0")
    b = torch.full((8 * 256,), float("nan"), dtype=torch.float32, device="cuda:0")
    assert fps.debug_mfma_rate(8, 4, a) == 8 * 4 * 4 * 8 * 65536.0
    fps.debug_mfma_rate(8, 8, b)
    torch.cuda.synchronize()
    assert torch.isfinite(a).all() and torch.isfinite(b).all() and (a != 0).all()
    assert torch.equal(b, 2 * a)


def test_issue_mix_kernel_counts_shader_clocks():
    """The matrix/vector issue-mix micro-benchmark: every wave reports a clock count, and an
    MFMA-only loop of the E4M3 16x16x128 instruction takes its 8 passes (32 clocks) per instruction
    on a SIMD that holds one wave."""
    import torch
    say("issue mix")
    wgs, iters = 8, 200
    sink = torch.full((wgs * 256,), float("nan"), dtype=torch.float32, device="cuda:0")
    cyc = torch.zeros(wgs * 4, dtype=torch.int64, device="cuda:0")
    fps.debug_issue_mix(0, 0, 0, 1, wgs, iters, sink, cyc)
    torch.cuda.synchronize()
    per_mfma = cyc.double() / (iters * 8)
    assert torch.isfinite(sink).all() and (cyc > 0).all()
    assert 30.0 <= float(per_mfma.min()) and float(per_mfma.max()) <= 40.0, per_mfma
    for kind, nv, op in [(1, 4, 0), (2, 8, 1), (3, 16, 0)]:
        cyc.zero_()
        fps.debug_issue_mix(kind, nv, op, 2, wgs, iters, sink, cyc)
        torch.cuda.synchronize()
        assert (cyc > 0).all() and torch.isfinite(sink).all()
    with pytest.raises(fps.FpsError):
        fps.debug_issue_mix(0, 5, 0, 1, wgs, iters, sink, cyc)          # not one of the built group sizes


def test_batch_and_heads_are_interchangeable():
    """Tensors are indexed by b*heads + h: (B=2, heads=3) equals (B=1, heads=6) bit for bit."""
    import torch
    say("batch")
    w = dataclasses.replace(synth.TINY, grid=(2, 13, 40), tile=(1, 8, 16), window=(3, 3, 3), heads=6,
                            n_outlier=3, config_id=18)
    run = gu.GpuRun(w)
    flat = fps.make_shape(6, w.grid, w.tile, B=1)
    two = fps.make_shape(3, w.grid, w.tile, B=2)
    outs = []
    for sh, lead in ((flat, (1, 6)), (two, (2, 3))):
        x = [r.reshape(lead + r.shape[2:]) for r in run.raster]
        q8 = [fps.quantize_tiles(sh, x[i], i, raster=True) for i in range(3)]
        assert q8[0][1].shape == lead + (run.g.M,)
        o = fps.attn_fwd(sh, w.window, fps.PREC_FP8, q8[0][0], q8[1][0], q8[2][0], q8[0][1], q8[1][1],
                         q8[2][1], out_dtype=torch.float32, raster_out=True)
        assert o.shape == lead + tuple(w.grid) + (128,)
        outs.append(o.reshape(-1))
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])


def test_side_stream_and_graph_replay(tiny):
    """The library launches on the stream it is given and allocates nothing, so the whole path
    (three fused quantise passes + attention) can run on a side stream and be captured into a HIP
    graph; every replay, with eager work and synchronisations in between, reproduces the eager
    result bit for bit."""
    import torch
    say("stream + graph")
    shape, w = tiny.shape, tiny.w
    M = tiny.g.M
    packed = [torch.empty(fps.packed_bytes(shape, fps.PREC_FP8), dtype=torch.uint8, device="cuda:0") for _ in range(3)]
    scales = [torch.empty((1, w.heads, M), dtype=torch.float32, device="cuda:0") for _ in range(3)]
    out = torch.empty((1, w.heads) + tuple(w.grid) + (128,), dtype=torch.float32, device="cuda:0")

    def path():
        for i in range(3):
            fps.quantize_tiles(shape, tiny.raster[i], i, out=packed[i], scales=scales[i], raster=True)
        fps.attn_fwd(shape, w.window, fps.PREC_FP8, packed[0], packed[1], packed[2], scales[0], scales[1],
                     scales[2], out=out, raster_out=True)

    path()
    torch.cuda.synchronize()
    want = out.clone()
    side = torch.cuda.Stream()                      # default priority
    side.wait_stream(torch.cuda.current_stream())
    out.zero_()
    with torch.cuda.stream(side):
        path()
    side.synchronize()
    assert torch.equal(out, want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        path()
    for rep in range(4):
        out.fill_(float(rep))                        # eager work between the replays
        for p_ in packed:
            p_.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), rep


def test_calls_on_two_streams_at_once_do_not_disturb_each_other(tiny):
    """The library keeps no device state between calls: two different shapes driven from two
    streams at the same time give what each gives alone."""
    import torch
    say("two streams at once")
    other = gu.GpuRun(dataclasses.replace(synth.TINY, grid=(5, 13, 20), tile=(1, 8, 16), window=(3, 3, 3),
                                          heads=3, n_outlier=3, config_id=29))
    runs = [tiny, other]
    want = []
    for r in runs:
        r.quantize()
        want.append(r.attn(fps.PREC_FP8).clone())
    outs = [torch.empty_like(o) for o in want]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]          # default priority
    for st in streams:
        st.wait_stream(torch.cuda.current_stream())
    for rep in range(8):
        for r, o, st in zip(runs, outs, streams):
            with torch.cuda.stream(st):
                (q, sq), (k, sk), (v, sv) = r.q8
                fps.attn_fwd(r.shape, r.w.window, fps.PREC_FP8, q, k, v, sq, sk, sv, out=o)
    for st in streams:
        st.synchronize()
    for o, x in zip(outs, want):
        assert torch.equal(o, x)


def test_step_config_selects_regime(tiny):
    import torch
    say("step config")
    regimes = [(fps.PREC_BF16, (3, 7, 7)), (fps.PREC_FP8, (3, 3, 3)), (fps.PREC_FP8, (1, 3, 3))]
    for step, idx in ((1, 0), (20, 1), (50, 2)):
        cfg = fps.make_step_cfg(step, 50, 0.2, 0.5, regimes)
        prec, win = fps.schedule_select(cfg)
        assert (prec, win) == regimes[idx]
        want = tiny.attn(prec, window=win)
        got = tiny.attn(prec, window=(9, 9, 9), step=cfg)     # explicit window must be overridden
        assert torch.equal(want, got)


def test_largest_granularity_of_the_tile_size_ablation():
    """(24,32,32) tiles (Table 3's largest): 24576 slots per tile, 192 blocks; the comparator
    fetches the kernel's scores block pair by block pair."""
    say("24x32x32 tiles")
    w = dataclasses.replace(synth.TINY, grid=(25, 5, 6), tile=(24, 32, 32), window=(3, 1, 1), heads=1,
                            n_outlier=3, config_id=16)
    run = gu.GpuRun(w)
    assert run.tsp == 24576 and run.g.M == 2
    for prec in (fps.PREC_BF16, fps.PREC_FP8):
        out, vis = run.attn(prec, visited=True)
        assert np.array_equal(vis.cpu().numpy().astype(bool), fo.tile_mask(run.g, w.window))
        st = gu.compare_head(run, out, 0, prec, w.window)
        say("  ", prec, st)
        gu.assert_parity(st, f"24x32x32 prec {prec}")


def test_step_config_with_granularity_per_regime():
    """Eq. 6: every regime has its own tile granularity g(t) and window W(t).  The caller
    quantises with the tile of the step's regime; a call whose inputs have another tile is
    refused."""
    say("step config with g(t)")
    regimes = [(fps.PREC_FP8, (1, 1, 3), (6, 8, 8)),        # early: coarse tiles, sparse window
               (fps.PREC_FP8, (3, 3, 3), (1, 8, 16)),       # mid: fine tiles, dense window
               (fps.PREC_FP8, (1, 3, 3), (2, 8, 16))]       # late: in between
    runs = {}
    for step, idx in ((3, 0), (20, 1), (44, 2)):
        cfg = fps.make_step_cfg(step, 50, 0.2, 0.5, regimes)
        prec, win, tile = fps.schedule_select(cfg, with_tile=True)
        assert (prec, win, tile) == regimes[idx]
        w = dataclasses.replace(synth.TINY, grid=(7, 13, 20), tile=tile, window=win, heads=1,
                                n_outlier=3, config_id=17)
        run = runs[idx] = gu.GpuRun(w)
        out = run.attn(prec, window=(9, 9, 9), step=cfg)     # the explicit window is overridden
        st = gu.compare_head(run, out, 0, prec, win)
        say("  step", step, tile, win, st)
        gu.assert_parity(st, f"step {step}")
    with pytest.raises(fps.FpsError) as e:                   # inputs of the late regime at an early step
        runs[2].attn(fps.PREC_FP8, step=fps.make_step_cfg(3, 50, 0.2, 0.5, regimes))
    assert e.value.status == fps.FPS_ERR_INVALID_ARG
    # a regime may also fix the quantisation sub-tile: same sparsity tile, finer scales
    fine = [(fps.PREC_FP8, (1, 3, 3), (2, 8, 16), (1, 8, 16))] * 3
    cfg = fps.make_step_cfg(44, 50, 0.2, 0.5, fine)
    assert fps.schedule_select(cfg, with_tile=True) == fine[0]
    with pytest.raises(fps.FpsError):
        runs[2].attn(fps.PREC_FP8, step=cfg)                 # quantised per tile, regime wants per sub-tile
    w = dataclasses.replace(synth.TINY, grid=(7, 13, 20), tile=(2, 8, 16), window=(1, 3, 3), heads=1,
                            n_outlier=3, config_id=17)
    run = gu.GpuRun(w, qtile=(1, 8, 16))
    st = gu.compare_head(run, run.attn(fps.PREC_FP8, step=cfg), 0, fps.PREC_FP8, (1, 3, 3))
    say("  sub-tile regime", st)
    gu.assert_parity(st, "sub-tile regime")


# ---- full-size shapes, sampled against the oracle ---------------------------------------------
def _sampled_parity(w, prec, window, head_picks, seed, n_interior=2, run=None):
    run = run or gu.GpuRun(w)
    out, vis = run.attn(prec, window=window, visited=True)
    mask = fo.tile_mask(run.g, window)
    assert np.array_equal(vis.cpu().numpy().astype(bool), mask)
    rng = np.random.default_rng(seed)
    for h in head_picks:
        tiles = gu.sample_q_tiles(run.g, rng, n_interior)
        st = gu.compare_head(run, out, h, prec, window, q_tiles=tiles)
        say(f"  {w.name} head {h} tiles {len(tiles)}", st)
        gu.assert_parity(st, f"{w.name} head {h}")
    return run, int(mask.sum())


def test_wan_1_3b_480p_fp8_sampled():
    say("480p fp8")
    run, pairs = _sampled_parity(synth.WAN_1_3B_480P, fps.PREC_FP8, synth.WAN_1_3B_480P.window,
                                 [0, 5, 11], seed=1)
    assert pairs == 6100
    # scales of every head and codes of one head per tensor, bit exact
    for role, (xq, sc) in enumerate(run.q8):
        sc = sc[0].cpu().numpy()
        for h in range(run.w.heads):
            ws = fo.tile_scales(fo.tile_order(run.qkv[role][h], run.g), run.g)
            assert np.array_equal(sc[h], ws)
        h = (5, 0, 11)[role]
        codes = fps.debug_unpack_q8(run.shape, xq, role)[0, h].cpu().numpy()[run.slots]
        wc, _ = fo.quantize_tiles(fo.tile_order(run.qkv[role][h].astype(np.float64), run.g), run.g)
        zero_sign = ((codes ^ wc) == 0x80) & ((wc & 0x7F) == 0)
        assert int(((codes != wc) & ~zero_sign).sum()) == 0, (role, h)


def test_wan_1_3b_480p_bf16_sparse_sampled():
    say("480p bf16")
    _sampled_parity(synth.WAN_1_3B_480P, fps.PREC_BF16, (3, 3, 3), [3], seed=2, n_interior=1)


def test_wan_14b_720p_fp8_sampled_in_bench_configuration():
    say("720p fp8")
    w = synth.WAN_14B_720P
    run, pairs = _sampled_parity(w, fps.PREC_FP8, w.window, [0, 17, 39], seed=3, n_interior=1)
    assert pairs == 20592
    for role, (xq, sc) in enumerate(run.q8):
        sc = sc[0].cpu().numpy()
        for h in range(0, w.heads, 7):
            ws = fo.tile_scales(fo.tile_order(run.qkv[role][h], run.g), run.g)
            assert np.array_equal(sc[h], ws)


def test_wan_14b_720p_dense_references_and_schedule_windows_sampled():
    """The other launches bench.py times on the 720p grid: the dense window in both precisions (the
    reference points of the speed-up) and the two FP8 windows of the step-aware schedule."""
    w = synth.WAN_14B_720P
    run = gu.GpuRun(w)
    nT, nH, nW = run.g.n_tiles_axis
    dense = (2 * nT - 1, 2 * nH - 1, 2 * nW - 1)
    for prec, window, pairs, head in [(fps.PREC_FP8, dense, 396900, 8), (fps.PREC_BF16, dense, 396900, 23),
                                      (fps.PREC_FP8, (7, 5, 5), 61560, 31), (fps.PREC_FP8, (3, 3, 3), 12688, 4)]:
        say("720p", "fp8" if prec == fps.PREC_FP8 else "bf16", window)
        _, kept = _sampled_parity(w, prec, window, [head], seed=5, n_interior=1, run=run)
        assert kept == pairs


def test_tensors_beyond_4_gib_index_correctly():
    """Offsets are 64-bit in every kernel: in a batch whose raster, packed and output tensors all
    exceed 2^32 bytes, the last heads give bit for bit what the same heads give alone."""
    import torch
    say("tensors beyond 4 GiB")
    w = dataclasses.replace(synth.WAN_1_3B_480P, heads=4, config_id=23)
    small = gu.GpuRun(w)
    reps = 200
    big = fps.make_shape(w.heads * reps, w.grid, w.tile)
    assert fps.packed_bytes(big, fps.PREC_FP8) > 2 ** 32
    results = []
    for shape, rasters in ((small.shape, small.raster),
                           (big, [r.repeat(1, reps, 1, 1, 1, 1) for r in small.raster])):
        assert shape is small.shape or rasters[0].numel() * 2 > 2 ** 32
        q8 = [fps.quantize_tiles(shape, r, role, raster=True) for role, r in enumerate(rasters)]
        o8 = fps.attn_fwd(shape, w.window, fps.PREC_FP8, q8[0][0], q8[1][0], q8[2][0],
                          q8[0][1], q8[1][1], q8[2][1], out_dtype=torch.bfloat16, raster_out=True)
        p16 = [fps.pack_tiles_bf16(shape, r, role, raster=True) for role, r in enumerate(rasters)]
        o16 = fps.attn_fwd(shape, w.window, fps.PREC_BF16, p16[0][0], p16[1][0], p16[2][0],
                           None, None, p16[2][1], out_dtype=torch.bfloat16, raster_out=True)
        torch.cuda.synchronize()
        n = shape.heads
        keep = [t.view(n, -1)[-w.heads:].clone() for pair in q8 + p16 for t in pair if t is not None]
        keep += [o.view(torch.int16).view(n, -1)[-w.heads:].clone() for o in (o8, o16)]
        results.append(keep)
        del q8, p16, o8, o16, rasters
    for i, (a, b) in enumerate(zip(*results)):
        assert torch.equal(a, b), f"tensor {i} of the last heads differs"
    assert float(results[0][-2].view(torch.bfloat16).float().abs().max()) > 0
