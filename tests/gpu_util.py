"""Helpers for the GPU parity tests: run the HIP path through the binding and compare with the
oracle on the same seeded inputs.  (Test code: it may call both sides; they never call each other.)"""
import numpy as np

from oracle import e4m3
from oracle import fps_oracle as fo
from paper_2506_04648_amd import fps, synth
from tests import accepted_set as acs

MAX_TOL = 2e-2      # max |err| <= 2e-2 * RMS(oracle output)
MEAN_TOL = 2e-3     # mean |err| <= 2e-3 * RMS
SMALL_SAMPLE = 2 ** 17   # output elements below which one P-code flip can dominate the mean
ACC_EPS = acs.ACC_EPS    # accumulation bound of the E4M3 matrix instruction (tests/accepted_set.py)
# How much of a comparison may rest on the accepted set rather than on the plain bars.  An FP8 tie
# flip moves one output by up to tens of per cent of the RMS, so single outputs beyond 2e-2 are
# expected; they must stay rare, and the slack granted must stay small on average.
MAX_FRACTION_BEYOND_PLAIN_BAR = 1e-2     # share of outputs with |err| > MAX_TOL * RMS
MAX_SLACK_MEAN = 0.3                     # mean slack per output, in units of the RMS
# Largest slack of a single output.  One open P code on a near one-hot row moves that row's output
# by 1/16 of |v| / l-share; at an outlier channel of V (8 x 4.5 sigma) under a dense window, where
# the output RMS is 0.06 sigma, that is some tens of RMS.  Observed: 9.3 (dense 720p), 5 (sparse).
MAX_SLACK_MAX = 64.0
MAX_MEAN_ERR_SMALL_SAMPLE = 4 * MEAN_TOL # un-slacked mean bar of a tiny sample with ambiguous P codes


def geometry(w: synth.Workload, qtile=None) -> fo.Geometry:
    return fo.Geometry(*w.grid, *w.tile, *(qtile or (0, 0, 0)))


def to_device_bf16(x_np):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x_np)).to("cuda:0").to(torch.bfloat16)


class GpuRun:
    """Inputs of a workload on the GPU, tile-ordered and packed by the library's own kernels."""

    def __init__(self, w: synth.Workload, qkv=None, call_index=0, heads=None, qtile=None):
        import torch
        self.w = w
        self.heads = list(range(w.heads)) if heads is None else list(heads)
        self.shape = fps.make_shape(len(self.heads), w.grid, w.tile, qtile=qtile)
        self.g = geometry(w, qtile)
        self.qkv = synth.qkv_raster(w, call_index, self.heads) if qkv is None else qkv
        self.raster = [to_device_bf16(a[None]) for a in self.qkv]
        self.tiled = [fps.tile_order(self.shape, r) for r in self.raster]
        self.torch = torch
        # The library's tiled tensors give every tile TSP >= TS slots: each quantisation sub-tile
        # (the whole tile unless a finer one is given) is rounded up to whole blocks and the
        # sub-tiles of a tile follow each other.  The oracle's tile order has exactly TS rows per
        # tile in (rt, rh, rw) order.  slots[i] = library slot of oracle row i.
        self.tsp = fps.tile_slots(self.shape)
        g = self.g
        assert self.tsp >= g.TS and fps.num_tiles(self.shape) == g.M
        assert fps.num_groups(self.shape) == g.n_groups and self.tsp % g.NS == 0
        qt, qh, qw = g.qtile
        r = np.arange(g.TS)
        rw, rh, rt = r % g.Tw, (r // g.Tw) % g.Th, r // (g.Tw * g.Th)
        sub = ((rt // qt) * (g.Th // qh) + rh // qh) * (g.Tw // qw) + rw // qw
        rank_in_sub = ((rt % qt) * qh + rh % qh) * qw + rw % qw
        in_tile = sub * (self.tsp // g.NS) + rank_in_sub
        self.slots = (np.arange(g.M)[:, None] * self.tsp + in_tile[None, :]).reshape(-1)

    def pad_slots(self):
        """Boolean mask over the M*TSP library slots: True where the slot holds no real token."""
        pad = np.ones(self.g.M * self.tsp, dtype=bool)
        pad[self.slots] = ~fo.valid_tokens(self.g)
        return pad

    def quantize(self, vscale=fps.VSCALE_TILE):
        self.q8 = [fps.quantize_tiles(self.shape, t, r, vscale=vscale) for t, r in zip(self.tiled, (0, 1, 2))]
        self.q8_vscale = vscale
        return self.q8

    def pack_bf16(self):
        self.p16 = [fps.pack_tiles_bf16(self.shape, t, r) for t, r in zip(self.tiled, (0, 1, 2))]
        return self.p16

    def attn(self, prec, window=None, out_dtype=None, visited=False, step=None, raster_out=False,
             vscale=fps.VSCALE_TILE, out=None):
        torch = self.torch
        out_dtype = out_dtype or torch.float32
        vis = torch.zeros((self.g.M, self.g.M), dtype=torch.uint8, device="cuda:0") if visited else None
        if prec == fps.PREC_FP8:
            if not hasattr(self, "q8") or self.q8_vscale != vscale:
                self.quantize(vscale)
            (q, sq), (k, sk), (v, sv) = self.q8
        else:
            if not hasattr(self, "p16"):
                self.pack_bf16()
            (q, _), (k, _), (v, sv) = self.p16
            sq = sk = None
        window = self.w.window if window is None else window
        out = fps.attn_fwd(self.shape, window, prec, q, k, v, sq, sk, sv, vscale=vscale, out=out,
                           out_dtype=out_dtype, visited=vis, step=step, raster_out=raster_out)
        torch.cuda.synchronize()
        return (out, vis) if visited else out

    def oracle_inputs(self, head_slot):
        """Tile-ordered float64 Q, K, V of one (selected) head for the oracle."""
        return tuple(fo.tile_order(a[head_slot].astype(np.float64), self.g) for a in self.qkv)


SCORE_CALL_MAX_SLOTS = 4096      # fps_debug_scores_q8 covers tile pairs up to this many slots


def gpu_raw_scores(run: GpuRun, head_slot, part):
    """The kernel's own raw score accumulators for one query tile over its window (valid keys
    only, same column order as the oracle's parts), fetched through fps_debug_scores_q8, or block
    pair by block pair (only blocks that hold real tokens) for tiles too large for that call."""
    g = run.g
    (q8, _), (k8, _), _ = run.q8
    tiles = part["key_tiles"]
    if run.tsp <= SCORE_CALL_MAX_SLOTS:
        raw = run.torch.cat([fps.debug_scores_q8(run.shape, q8, k8, head_slot, part["u"], int(v))
                             for v in tiles], dim=1)
        run.torch.cuda.synchronize()
        raw = raw.cpu().numpy()
        in_tile = run.slots[:g.TS]                                   # oracle in-tile rank -> library slot
        local = np.searchsorted(tiles, part["cols"] // g.TS) * run.tsp + in_tile[part["cols"] % g.TS]
        return raw[in_tile][:, local]
    bs = fps.block_slots(run.shape)
    in_tile = run.slots[:g.TS]                                       # oracle in-tile rank -> library slot
    raw = np.zeros((g.TS, part["cols"].size), dtype=np.float32)
    q_rows = np.flatnonzero(part["rows_valid"])                      # oracle ranks of the real query rows
    q_slot = in_tile[q_rows]
    k_tile, k_slot = part["cols"] // g.TS, in_tile[part["cols"] % g.TS]
    buf = run.torch.empty((bs, bs), dtype=run.torch.float32, device="cuda:0")
    for jq in np.unique(q_slot // bs):
        rq = q_slot // bs == jq
        for v in tiles:
            for jk in np.unique(k_slot[k_tile == v] // bs):
                sel = np.flatnonzero((k_tile == v) & (k_slot // bs == jk))
                fps.debug_scores_block_q8(run.shape, q8, k8, head_slot, part["u"], int(jq), int(v), int(jk), out=buf)
                blk = buf.cpu().numpy()
                raw[np.ix_(q_rows[rq], sel)] = blk[np.ix_(q_slot[rq] % bs, k_slot[sel] % bs)]
    return raw


def kernel_selected_member(part, raw_gpu):
    """The member of the accepted set that the kernel's OWN score accumulators select: Eq. 3 and
    the 1/448 quantisation of P applied, in float64, to the scores the library reports.  Not the
    parity reference (that is the oracle's output, with the oracle-derived accepted set around
    it): a second, tighter test that the kernel's output is consistent with its scores, so that a
    wrong rounding or a wrong weight cannot hide behind an element the accepted set leaves open.
    Returns (part-like dict, output rows)."""
    S = np.asarray(raw_gpu, dtype=np.float64) * part["pair_scale"]
    m = np.ceil(S.max(axis=1))
    p = np.exp2(S - m[:, None])
    l = p.sum(axis=1)
    ph = e4m3.round_to_e4m3(e4m3.FP8_MAX * p) / e4m3.FP8_MAX
    o = (ph @ part["v"]) / l[:, None]
    o[~part["rows_valid"]] = 0.0
    return dict(part, S=S, m=m, p=p, l=l, ph=ph), o


def fp8_checks(run: GpuRun, head_slot, part, ref_rows, got_rows):
    """The three FP8 checks of one query tile.
    (1) slack: the accepted set around the oracle's output, from the oracle's quantities alone.
    (2) score_ratio: the kernel's reported score accumulators against the oracle's exact products,
        in units of the accumulation bound the accepted set assumes (<= 1 required).
    (3) consistency: the kernel's output against the member of the accepted set its own scores
        select, with no accumulation allowance on the scores (only the float32 evaluation of the
        exponential, the sub-normal range and the PV product's accumulation remain); and every P
        code by which that member differs from the oracle's must be one the accepted set leaves
        open.  Returns (slack, stats)."""
    slack, stats, may_differ = acs.fp8_slack(part, ref_rows)
    raw_gpu = gpu_raw_scores(run, head_slot, part)
    stats["score_ratio"] = acs.scores_within_model(raw_gpu, part)
    sel, o_sel = kernel_selected_member(part, raw_gpu)
    sel_slack, _, _ = acs.fp8_slack(sel, o_sel, acc_eps=0.0, pv_eps=acs.ACC_EPS)
    stats["sel_excess"] = float(np.max(np.maximum(np.abs(got_rows - o_sel) - sel_slack, 0.0)))
    stats["sel_slack_sum"] = float(sel_slack[part["rows_valid"]].sum())
    differs = sel["ph"] * np.exp2(sel["m"] - part["m"])[:, None] != part["ph"]
    differs[~part["rows_valid"]] = False
    stats["code_flips"] = int(np.count_nonzero(differs))
    stats["flips_outside_accepted_set"] = int(np.count_nonzero(differs & ~may_differ))
    return slack, stats


def compare_head(run: GpuRun, out_gpu, head_slot, prec, window, q_tiles=None, vscale=fps.VSCALE_TILE):
    """Oracle vs GPU for one head (optionally a subset of query tiles).  Returns a dict of
    normalised errors; asserts nothing."""
    g = run.g
    qt, kt, vt = run.oracle_inputs(head_slot)
    oprec = fo.PREC_FP8 if prec == fps.PREC_FP8 else fo.PREC_BF16
    ref, parts = fo.attention(qt, kt, vt, g, window, prec=oprec, q_tiles=q_tiles, return_parts=True,
                              vscale=fo.VSCALE_CHANNEL if vscale == fps.VSCALE_CHANNEL else fo.VSCALE_TILE)
    tiles = list(range(g.M)) if q_tiles is None else list(q_tiles)
    rows = (np.asarray(tiles)[:, None] * g.TS + np.arange(g.TS)[None, :]).reshape(-1)   # oracle rows
    got_all = out_gpu[0, head_slot].double().cpu().numpy()                               # library slots
    got = got_all[run.slots[rows]]
    valid = fo.valid_tokens(g)[rows]
    slack = np.zeros_like(ref)
    tot = dict(ambiguous=0, p_elems=0, rows_ref_may_rise=0, code_flips=0, flips_outside_accepted_set=0,
               sel_slack_sum=0.0)
    score_ratio = sel_excess = 0.0
    if prec == fps.PREC_BF16:
        # BF16 mode rounds every softmax weight to fp16 (relative error <= 2^-12 each) before the
        # PV product; to first order an output moves by at most 2^-12 * sum_j p_j |v_j| / l.  The
        # bound matters only where |O| is far above the RMS (a peaked row on a large V value);
        # 2^-11 leaves a factor two for the fp32 accumulation and the fp32 exp2.
        for n, part in enumerate(parts):
            sl = 2.0 ** -11 * (part["p"] @ np.abs(part["v"])) / part["l"][:, None]
            sl[~part["rows_valid"]] = 0.0
            slack[n * g.TS:(n + 1) * g.TS] = sl
    else:
        for n, part in enumerate(parts):
            rs = slice(n * g.TS, (n + 1) * g.TS)
            slack[rs], st = fp8_checks(run, head_slot, part, ref[rs], got[rs])
            for key in tot:
                tot[key] += st[key]
            score_ratio = max(score_ratio, st["score_ratio"])
            sel_excess = max(sel_excess, st["sel_excess"])
    pad_zero = bool(np.all(got[~valid] == 0)) and bool(np.all(got_all[run.pad_slots()] == 0))
    rms = float(np.sqrt(np.mean(ref[valid] ** 2)))
    err = np.abs(got - ref)
    n_out = max(1, int(valid.sum()) * ref.shape[1])
    return dict(rms=rms,
                max_err=float(err.max() / rms),
                max_excess=float(np.max(np.maximum(err - slack, 0.0)) / rms),
                mean_err=float(err[valid].mean() / rms),
                mean_excess=float(np.maximum(err - slack, 0.0)[valid].mean() / rms),
                beyond_plain_bar=float(np.count_nonzero(err[valid] > MAX_TOL * rms) / n_out),
                valid_outputs=n_out,
                slack_max=float(slack.max() / rms),
                slack_mean=float(slack[valid].mean() / rms),
                ambiguous=tot["ambiguous"], p_elems=tot["p_elems"], rows_ref_may_rise=tot["rows_ref_may_rise"],
                score_ratio=score_ratio,
                sel_max_excess=sel_excess / rms, sel_slack_mean=tot["sel_slack_sum"] / n_out / rms,
                code_flips=tot["code_flips"], flips_outside_accepted_set=tot["flips_outside_accepted_set"],
                pad_rows_zero=pad_zero,
                finite=bool(np.all(np.isfinite(got))))


def assert_parity(stats, label=""):
    """The bars of the comparison.
    Against the oracle: no output further from the oracle's than the accepted set allows plus
    2e-2 RMS (max bar); the plain mean error, without any slack, within 2e-3 RMS (mean bar); the
    share of outputs that lie beyond the plain 2e-2 bar, and the mean slack, capped.
    What ties the kernel to the accepted set: its reported scores inside the accumulation bound
    the set is built on; its output within 2e-2 RMS of the member of the set that those scores
    select; no P code of that member differing from the oracle's where the set leaves none open."""
    assert stats["finite"], (label, stats)
    assert stats["pad_rows_zero"], (label, stats)
    assert stats["score_ratio"] <= 1.0, (label, stats)
    assert stats["max_excess"] <= MAX_TOL, (label, stats)
    assert stats["sel_max_excess"] <= MAX_TOL, (label, stats)
    assert stats["flips_outside_accepted_set"] == 0, (label, stats)
    assert stats["slack_mean"] <= MAX_SLACK_MEAN, (label, stats)
    assert stats["slack_max"] <= MAX_SLACK_MAX, (label, stats)
    # In a case of a few thousand outputs a single tie flip on a peaked row (a legitimate
    # alternative result, inside the accepted set) moves the plain mean past 2e-3 and is a visible
    # share of the outputs; there the mean bar applies to the error beyond the slack, and the plain
    # mean still has to stay within a few times the bar.  Large samples meet the plain bars.
    if stats["valid_outputs"] < SMALL_SAMPLE and stats["code_flips"] > 0:
        assert stats["mean_excess"] <= MEAN_TOL, (label, stats)
        assert stats["mean_err"] <= MAX_MEAN_ERR_SMALL_SAMPLE, (label, stats)
    else:
        assert stats["mean_err"] <= MEAN_TOL, (label, stats)
        assert stats["beyond_plain_bar"] <= MAX_FRACTION_BEYOND_PLAIN_BAR, (label, stats)


def sample_q_tiles(g: fo.Geometry, rng, n_interior=3):
    """Corners, edge and face tiles, tiles whose rows are partly padding, and a few interior ones."""
    nT, nH, nW = g.n_tiles_axis
    idx = lambda t, h, w: (t * nH + h) * nW + w
    picks = {idx(0, 0, 0), idx(nT - 1, nH - 1, nW - 1), idx(0, nH - 1, 0), idx(nT - 1, 0, nW - 1),
             idx(nT // 2, 0, nW // 2), idx(nT // 2, nH - 1, nW // 2), idx(0, nH // 2, nW // 2),
             idx(nT // 2, nH // 2, nW - 1)}
    for _ in range(n_interior):
        picks.add(idx(int(rng.integers(1, max(2, nT - 1))), int(rng.integers(1, max(2, nH - 1))),
                      int(rng.integers(1, max(2, nW - 1)))))
    return sorted(picks)


def score_error_ratio(run: GpuRun, head_slot, u, v):
    """max over the tile pair of |S_gpu - S_exact| / sum_c |q_c k_c| for the raw E4M3 scores."""
    g = run.g
    assert g.NS == 1
    qt, kt, _ = run.oracle_inputs(head_slot)
    qc, _ = fo.quantize_tiles(qt[u * g.TS:(u + 1) * g.TS], fo.Geometry(1, 1, g.TS, 1, 1, g.TS))
    kc, _ = fo.quantize_tiles(kt[v * g.TS:(v + 1) * g.TS], fo.Geometry(1, 1, g.TS, 1, 1, g.TS))
    qh, kh = e4m3.decode(qc), e4m3.decode(kc)
    exact = qh @ kh.T                                   # exact in float64: 128 products of 8 bits
    absdot = np.abs(qh) @ np.abs(kh).T
    (q8, _), (k8, _), _ = run.q8
    got = fps.debug_scores_q8(run.shape, q8, k8, head_slot, u, v)
    run.torch.cuda.synchronize()
    got = got.double().cpu().numpy()
    in_tile = run.slots[:g.TS]
    pad = np.ones(run.tsp, dtype=bool)
    pad[in_tile] = False
    assert np.all(got[pad] == 0) and np.all(got[:, pad] == 0)       # padding slots: zero codes
    got = got[in_tile][:, in_tile]
    return float(np.max(np.abs(got - exact) / np.maximum(absdot, 1e-30))), got, exact
