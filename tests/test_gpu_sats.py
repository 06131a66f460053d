"""GPU parity of SATS calibration (Section 3.1, Eq. 6-10) through the C ABI.

Comparison rules (the GPU accumulates g and u in float32 and enters p as
two bf16 terms; the oracle is float64 on the same stored values):
  * candidate thresholds: the Eq. 3 order statistics agree to 1e-4 relative
    (an order statistic of nearly identical values);
  * errors and sparsities are compared at the GPU's own thresholds.  A
    candidate is a sample magnitude, so at least one neuron sits exactly on
    it, and neurons within float32 rounding of a threshold (1e-5 relative)
    may be removed on one side and kept on the other: per row, the GPU's
    error must lie (to 1e-4 relative) between the oracle's errors with those
    neurons kept and with them removed, and the sparsity within their count;
  * a stack: the oracle runs on the GPU's own layer inputs (exported by the
    forward call), and the GPU's choice must be the oracle's, or one the
    oracle scores equally close to the target sparsity.
"""
import numpy as np
import pytest

from harness import from_dev, gate_dev, to_dev, weights_dev
from oracle import calibrate, numerics, sats as osats
from workloads import synth

pytestmark = pytest.mark.gpu

LEVELS = sorted([0.0] + [round(0.05 * i, 4) for i in range(1, 20)] + [0.33, 0.5001, 0.999])


def _layer(seed, d, dff, n, w_std=None):
    c = synth.small_case(seed, 1, d, dff, "bf16", n, w_std=w_std or 1.0 / np.sqrt(d))
    return c["x"], c["W_gate"][0], c["W_up_T"][0], c["W_down"][0]


def _bounds(H, W, ts, rel=1e-5):
    """Per row and candidate, the oracle's Eq. 6 term with the neurons within
    `rel` of the threshold kept and with them removed (low, high), and the
    number of such neurons per candidate."""
    g, p, y = osats.layer_terms(H, *W)
    a = np.abs(g)
    ny = np.linalg.norm(y, axis=1)
    lo = np.zeros((len(H), len(ts)))
    hi = np.zeros_like(lo)
    nnear = np.zeros(len(ts), int)
    for k, t in enumerate(ts):
        near = np.abs(a - t) <= rel * t
        nnear[k] = near.sum()
        sure = (a < t) & ~near
        e1 = np.linalg.norm(np.where(sure, p, 0.0) @ W[2], axis=1) / (ny + 1e-6)
        e2 = np.linalg.norm(np.where(sure | near, p, 0.0) @ W[2], axis=1) / (ny + 1e-6)
        lo[:, k], hi[:, k] = np.minimum(e1, e2), np.maximum(e1, e2)
    return lo, hi, nnear, g


def _within(got, lo, hi, rel=1e-4, atol=1e-6):
    slack = rel * np.maximum(np.abs(lo), np.abs(hi)) + atol
    return (got >= lo - slack) & (got <= hi + slack)


def _gpu_curves(x, wg, wu, wd, levels, rows=True):
    import torch
    import paper_2607_08991_amd as sats
    n, d = x.shape
    dff = wg.shape[1]
    er = torch.zeros((n, len(levels)), dtype=torch.float32, device="cuda") if rows else None
    t, err, sp = sats.sats_calibration_curves(to_dev(x, "bf16"), gate_dev(wg, "bf16"), to_dev(wu, "bf16"),
                                              to_dev(wd, "bf16"), n, d, dff, levels, err_rows=er)
    return t, err, sp, (er.cpu().numpy() if rows else None)


# the benchmark's grid: 0 and 19 percentiles, i.e. products of 15 candidates
# (with y) and of 4 (four calibration rows per tile, y from the first)
LEVELS20 = [0.0] + [round(0.05 * i, 4) for i in range(1, 20)]


@pytest.mark.parametrize("seed,d,dff,n,levels", [(61, 256, 1024, 40, LEVELS), (62, 128, 512, 17, LEVELS),
                                                 (63, 512, 1536, 64, LEVELS), (64, 256, 1024, 37, LEVELS20),
                                                 (65, 384, 768, 16, LEVELS20)])
def test_curves_match_oracle(seed, d, dff, n, levels):
    x, wg, wu, wd = _layer(seed, d, dff, n)
    t, err, sp, er = _gpu_curves(x, wg, wu, wd, levels)
    H = numerics.decode(x, "bf16")
    W = [numerics.decode(w, "bf16") for w in (wg, wu, wd)]
    g = osats.layer_terms(H, *W)[0]
    absg = np.abs(g)
    # candidates: Eq. 3 order statistics
    for k, q in enumerate(levels):
        ref = calibrate.percentile_threshold(absg, q)
        assert t[k] == pytest.approx(ref, rel=1e-4, abs=1e-30), (k, q)
    assert t[0] == 0.0 and np.all(np.diff(t) >= 0)
    # errors and sparsities at the GPU's thresholds
    ts = t.astype(np.float64)
    lo, hi, nnear, _ = _bounds(H, W, ts)
    assert err[0] == 0.0
    assert _within(er, lo, hi).all()
    assert _within(err, lo.mean(0), hi.mean(0)).all()
    sp_ref = osats.sparsity_curve(g, ts)
    assert np.all(np.abs(sp - sp_ref) <= (nnear + 0.5) / absg.size)


def test_curves_llama_layer_sampled():
    """One Llama-3.1-8B-shaped layer (4096 x 14336), 48 calibration rows: all
    candidates on the GPU; the oracle recomputes 16 rows at 5 candidates."""
    from workloads import get_config
    cfg = get_config(1)
    wg, wu, wd = synth.layer_weights(cfg.seed, 0, cfg.d, cfg.d_ff, cfg.dtype)
    x = synth.activations(cfg.seed, synth.S_CAL, 48, cfg.d, cfg.dtype)
    t, err, sp, er = _gpu_curves(x, wg, wu, wd, LEVELS)
    H = numerics.decode(x[:16], "bf16")
    W = [numerics.decode(w, "bf16") for w in (wg, wu, wd)]
    pick = [0, 5, 9, 14, 20]
    lo, hi, _, _ = _bounds(H, W, t[pick].astype(np.float64))
    got = er[:16][:, pick]
    assert _within(got, lo, hi).all()
    # the realized sparsity of each candidate on the calibration set is its level
    N = 48 * cfg.d_ff
    for k, q in enumerate(LEVELS):
        if 0 < q < 1:
            assert abs(sp[k] - (np.ceil(q * N) - 1) / N) <= 4.0 / N


def test_calibrate_stack_matches_oracle():
    import torch
    import paper_2607_08991_amd as sats
    L, d, dff, n = 3, 256, 1024, 96
    c = synth.small_case(71, L, d, dff, "bf16", n, w_std=1.0 / np.sqrt(d))
    x = c["x"]
    dw = list(weights_dev(c, "bf16"))
    ts, b, s = sats.sats_calibrate_sats(to_dev(x, "bf16"), n, *dw, d, dff, L, 0.5,
                                        coarse_step=0.1, fine_step=0.02, guardrail=True)
    # the GPU's own layer inputs on the base path
    lin = torch.empty((L, n, d), dtype=torch.bfloat16, device="cuda")
    out = torch.empty((n, d), dtype=torch.bfloat16, device="cuda")
    lut = torch.ones(1, dtype=torch.uint8, device="cuda")
    ids = torch.zeros(n, dtype=torch.int32, device="cuda")
    thr = torch.zeros(L, dtype=torch.float32, device="cuda")
    sats.sats_mlp_forward_inspect(to_dev(x, "bf16"), ids, *dw, thr, lut, out, n, d, dff, L, layer_in=lin)
    torch.cuda.synchronize()
    H = from_dev(lin)
    r = osats.calibrate(x, c["W_gate"], c["W_up_T"], c["W_down"], 0.5, "bf16", coarse_step=0.1, fine_step=0.02,
                        layer_inputs=H)
    # guardrail layer: its CATS threshold
    assert ts[L - 1] == pytest.approx(float(r["thresholds"][L - 1]), rel=1e-4)
    # free layers: each GPU threshold is an oracle candidate of the refined stage (same level)
    b2, idx2, s2, c2 = r["fine"]
    S = r["guardrail"][L - 1]
    for l in range(L - 1):
        tsl, errl, spl = c2[l]
        k = int(np.argmin(np.abs(tsl - ts[l])))
        assert tsl[k] == pytest.approx(float(ts[l]), rel=1e-4)
        S += spl[k]
    S /= L
    # the GPU's choice is as close to the target as the oracle's (same breakpoints)
    assert abs(S - 0.5) <= abs(s2 - 0.5) + 2e-3
    assert abs(s - S) <= 2e-3
    # Eq. 7 at the GPU's budget b*: each free layer's threshold is the largest
    # oracle candidate whose error is within b*, up to the float32 slack of
    # the GPU's errors (1e-4 relative, as in the curve comparisons above)
    slack = 1e-4 * b + 1e-7
    assert b >= 0.0
    for l in range(L - 1):
        tsl, errl, spl = c2[l]
        k = int(np.argmin(np.abs(tsl - ts[l])))
        assert errl[k] <= b + slack, (l, errl[k], b)
        assert not np.any(errl[k + 1:] <= b - slack), (l, errl[k + 1:], b)


def test_kept_buffers_across_shapes_and_release():
    """The calibration keeps its device buffers from call to call (grown when a
    call needs more, freed by sats_release): calls of different shapes in a row,
    a smaller call after a larger one, and a call after sats_release give the
    bits of the first call of their shape."""
    import paper_2607_08991_amd as sats
    small = _layer(64, 256, 1024, 24)
    big = _layer(65, 512, 2048, 96)
    first = _gpu_curves(*small, LEVELS)
    fb = _gpu_curves(*big, LEVELS)
    again = _gpu_curves(*small, LEVELS)        # reuses the grown buffers
    sats.sats_release()
    fresh = _gpu_curves(*small, LEVELS)        # buffers allocated anew
    bb = _gpu_curves(*big, LEVELS)
    for a, b in ((first, again), (first, fresh), (fb, bb)):
        for u, v in zip(a, b):
            np.testing.assert_array_equal(np.asarray(u), np.asarray(v))


def test_many_levels_select_against_its_own_counts():
    """1024 levels (16 select calls of 64 levels): the Eq. 3 order statistics
    against the oracle's, and against the library's own count of the values
    below each (#{|g| < t_k} = rank - 1 but for ties at t_k, which float32
    makes rare).  With this many levels, distinct prefixes of one call share
    a slot of the select's prefix table in its 20- or 28-bit passes (checked
    on the returned thresholds), so its fallback search is reached."""
    import math
    from fractions import Fraction
    n, d, dff = 64, 256, 1024
    x, wg, wu, wd = _layer(71, d, dff, n)
    levels = [round(float(q), 6) for q in np.linspace(0.0005, 0.9995, 1024)]
    t, err, sp, _ = _gpu_curves(x, wg, wu, wd, levels, rows=False)
    H = numerics.decode(x, "bf16")
    W = [numerics.decode(w, "bf16") for w in (wg, wu, wd)]
    absg = np.abs(osats.layer_terms(H, *W)[0])
    N = absg.size
    ref = np.array([calibrate.percentile_threshold(absg, q) for q in levels])
    np.testing.assert_allclose(t, ref, rtol=1e-4, atol=1e-30)
    assert np.all(np.diff(t) >= 0)
    rank = np.array([min(max(math.ceil(Fraction(repr(q)) * N), 1), N) for q in levels])
    below = np.rint(sp * N).astype(np.int64)
    gap = (rank - 1) - below
    assert gap.min() >= 0 and gap.max() <= 3, (gap.min(), gap.max())
    assert np.count_nonzero(gap) <= 8
    # slot sharing of the 20- and 28-bit prefixes within a call of 64 levels
    bits = t.astype(np.float32).view(np.uint32).astype(np.int64)
    shared = 0
    for c0 in range(0, len(levels), 64):
        for hs in (12, 4):
            pre = np.unique(bits[c0:c0 + 64] >> hs)
            shared += len(pre) - len(np.unique(pre & 0xFFF))
    assert shared > 0


@pytest.mark.parametrize("n", [512, 560])
def test_four_candidate_product_of_64_row_workgroups(n):
    """The last four of nineteen positive candidates (four rows per MFMA tile,
    workgroups of 64 rows once those fill the chip, ||y||^2 kept from the first
    product) against the same candidates on their own (two rows per tile, y in
    the product): the products and their order of k are the same, so only the
    column tiles' sums of squares are added in another order (float32, 128 and
    64 columns: relative 1e-6 of a norm)."""
    import torch
    import paper_2607_08991_amd as sats
    d, dff = 4096, 128
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((n, d), generator=g, device="cuda").to(torch.bfloat16)
    w = [(torch.randn((dff, d), generator=g, device="cuda") * 0.02).to(torch.bfloat16) for _ in range(3)]
    levels = [round(i / 20, 10) for i in range(20)]
    rows = torch.empty((n, 20), dtype=torch.float32, device="cuda")
    t, err, sp = sats.sats_calibration_curves(x, *w, n, d, dff, levels, err_rows=rows)
    tail = torch.empty((n, 4), dtype=torch.float32, device="cuda")
    t4, err4, sp4 = sats.sats_calibration_curves(x, *w, n, d, dff, levels[16:], err_rows=tail)
    np.testing.assert_array_equal(t[16:], t4)
    np.testing.assert_array_equal(sp[16:], sp4)
    np.testing.assert_allclose(rows[:, 16:].cpu().numpy(), tail.cpu().numpy(), rtol=4e-6)
    np.testing.assert_allclose(err[16:], err4, rtol=1e-6)


@pytest.mark.parametrize("n", [1, 16, 17, 128, 129])
def test_four_candidate_product_of_few_rows(n):
    """... in workgroups of 16 rows, while all of them run at once (128 rows at this
    width on 256 compute units), and of 32 beyond."""
    test_four_candidate_product_of_64_row_workgroups(n)


@pytest.mark.parametrize("seed,d,dff,n", [(71, 128, 512, 65), (72, 128, 4096, 1), (73, 128, 4096, 128),
                                          (74, 128, 4096, 129), (75, 384, 4160, 300)])
def test_gate_up_passes_of_64_and_tiles(seed, d, dff, n):
    """Gate and up of the rows in passes of 64 while all of those run at once (128
    rows of 4096 columns on 256 compute units), on the tiled product beyond.  As
    test_curves_match_oracle, with a neuron near a threshold also where its g lies
    within 4e-6: products of bf16 are exact in float32, and a running sum of
    magnitude below 12 rounds by at most 6e-8 of that in each of its few steps (the
    small thresholds of the low levels are reached by cancellation)."""
    x, wg, wu, wd = _layer(seed, d, dff, n)
    t, err, sp, er = _gpu_curves(x, wg, wu, wd, LEVELS20)
    H, W = numerics.decode(x, "bf16"), [numerics.decode(w, "bf16") for w in (wg, wu, wd)]
    g, p, y = osats.layer_terms(H, *W)
    a, ny = np.abs(g), np.linalg.norm(y, axis=1)
    flat = np.sort(a.reshape(-1))
    for k, q in enumerate(LEVELS20):
        assert abs(t[k] - calibrate.percentile_threshold(a, q)) <= 4e-6 + 1e-5 * t[k], (k, q)
        near = np.abs(a - t[k]) <= 4e-6 + 1e-5 * t[k]
        sure = (a < t[k]) & ~near
        e = [np.linalg.norm(np.where(m, p, 0.0) @ W[2], axis=1) / (ny + 1e-6) for m in (sure, sure | near)]
        # the removed set lies between the two: its product from each by at most the near neurons'
        slack = np.linalg.norm(np.where(near, np.abs(p), 0.0) @ np.abs(W[2]), axis=1) / (ny + 1e-6) + 1e-4 * e[1] + 1e-6
        assert (np.abs(er[:, k] - e[0]) <= slack).all(), (k, q)
        assert abs(err[k] - er[:, k].mean()) <= 1e-5 * err[k] + 1e-7
        assert abs(sp[k] - np.searchsorted(flat, t[k]) / flat.size) <= (near.sum() + 0.5) / flat.size
