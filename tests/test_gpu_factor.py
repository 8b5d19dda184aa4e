"""The factored rule kernels (csrc/gm_nodes.hpp: per-axis factors formed once per
region), which adaptive runs of dimension >= 7 use: every mapping at the edges
of its range, both fully symmetric rules, every family, against the chain-form
kernels (gm_eval_regions) on every region of the last active set and against the
oracle on a sample; and parameters on either side of the line beyond which a run
keeps the chain form (the axes' largest |log factor| adding up to 500).

Tolerance: the per-region bar of parity.py, 1e-13 of the magnitudes summed.  The
factored value of a node differs from the chain's by the rounding of d factors
and d products, and the chain's own by that of an exponent or angle s, |s| 2^-53
a few times: below 3e-14 for every case here (|s| <= 60)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2511_01573_amd import gm, workloads as W
from parity import assert_regions_match

pytestmark = pytest.mark.gpu

FACTORED = [1, 2, 4, 5, 6]  # families with a factored kernel
MAPPINGS = {7: (1, 4), 8: (1, 4, 16), 10: (1, 16, 64), 11: (4, 64), 13: (4, 16), 16: (16, 64)}


def _stopped_run(fam, p, lo, hi, iters, rule=0, lanes=0, init_log2=9):
    opts = {"max_iters": iters, "rule": rule, "lanes_per_region": lanes,
            "init_log2_regions": init_log2}
    for k, v in opts.items():
        gm.set_option(k, v)
    try:
        _, _, st = gm.integrate(fam, p, lo, hi, 1e-12, 1e-300, 1 << 16)
        assert st in (gm.MAX_ITERS, gm.MAX_REGIONS, gm.OK)
        act = gm.last_active(len(lo))
    finally:
        for k, v in {"max_iters": 10000, "lanes_per_region": 0, "init_log2_regions": 12}.items():
            gm.set_option(k, v)
    try:
        chain = gm.eval_regions(fam, p, lo, hi, act["c"], act["h"], act["lvl"])
    finally:
        gm.set_option("rule", 0)
    return act, chain


def _check(fam, p, lo, hi, act, chain, rule, label):
    n = act["lvl"].size
    assert n > 0
    vol = 1.0
    for a, b in zip(lo, hi):
        vol = vol * (b - a)
    idx = np.unique(np.linspace(0, n - 1, min(n, 24)).astype(int))
    ref = O.rule_many(fam, p, act["c"][idx], act["h"][idx], act["lvl"][idx], vol, rule_id=rule)
    assert_regions_match(act["Q"][idx], act["err"][idx], act["axis"][idx], ref, label)
    q, err, axis = chain
    # every region against the chain form; the scale of the sample's largest
    # (err cancels magnitudes of the size of scaleE, a multiple of scaleQ)
    ratio = np.max(ref["scaleE"] / np.maximum(ref["scaleQ"], 1e-300))
    scale = np.max(ref["scaleQ"] * np.ldexp(1.0, act["lvl"][idx])) * np.ldexp(1.0, -act["lvl"])
    assert np.all(np.abs(act["Q"] - q) <= 1e-13 * scale), label
    assert np.all(np.abs(act["err"] - err) <= 1e-13 * scale * max(ratio, 1.0)), label
    assert np.array_equal(act["axis"], axis), label


@pytest.mark.parametrize("d", sorted(MAPPINGS))
@pytest.mark.parametrize("fam", FACTORED)
def test_degree7_mappings(fam, d):
    p = W.family_params(fam, d, seed=700 * fam + d)
    lo, hi = W.unit_box(d)
    for lanes in MAPPINGS[d]:
        print(f"case fam={fam} d={d} lanes={lanes}", flush=True)
        act, chain = _stopped_run(fam, p, lo, hi, 4 if d <= 11 else 3, lanes=lanes)
        _check(fam, p, lo, hi, act, chain, 0, f"fam{fam} d{d} lanes{lanes}")


@pytest.mark.parametrize("d,iters,init_log2", [(7, 3, 7), (8, 2, 12), (9, 9, 3), (12, 2, 6),
                                               (16, 2, 6)])
@pytest.mark.parametrize("fam", FACTORED)
def test_degree9_mappings(fam, d, iters, init_log2):
    p = W.family_params(fam, d, seed=900 * fam + d)
    lo, hi = W.unit_box(d)
    print(f"case degree 9 fam={fam} d={d}", flush=True)
    act, chain = _stopped_run(fam, p, lo, hi, iters, rule=2, init_log2=init_log2)
    _check(fam, p, lo, hi, act, chain, 2, f"degree 9 fam{fam} d{d}")


@pytest.mark.parametrize("fam,a,u,box", [
    (2, 50.0, 0.5, (0.0, 1.0)),        # the paper's f2
    (2, 2e13, 2.0, (0.0, 1.0)),        # factors 1 / (x - 2)^2: log factors 61 + 1.4 per axis
    (2, 6e15, 2.0, (0.0, 1.0)),        # beyond the line
    (4, 7.9, 1.0, (0.0, 1.0)),         # span 499
    (4, 8.0, 1.0, (0.0, 1.0)),         # 512
    (5, -62.0, 0.0, (0.0, 1.0)),       # growing factors, span 496
    (5, -63.0, 0.0, (0.0, 1.0)),       # 504
    (6, -3.0, 9.0, (0.0, 10.0)),       # a cut outside most of the box
    (1, 3.0, 0.25, (-2.0, 3.0)),
])
def test_both_sides_of_the_line(fam, a, u, box):
    d = 8
    lo, hi = np.full(d, box[0]), np.full(d, box[1])
    # alternate the sign of the exponents where the family allows it
    av = np.full(d, a)
    if fam in (1, 5):
        av[1::2] *= -0.5
    p = np.concatenate([av, np.full(d, u)])
    print(f"case line fam={fam} a={a}", flush=True)
    act, _ = _stopped_run(fam, p, lo, hi, 2)
    vol = (box[1] - box[0]) ** d
    idx = np.unique(np.linspace(0, act["lvl"].size - 1, 40).astype(int))
    ref = O.rule_many(fam, p, act["c"][idx], act["h"][idx], act["lvl"][idx], vol)
    # beyond e^-60 the oracle's own sum of exponents rounds by up to 500 2^-53
    # times the d additions, 4.4e-13
    tol = 4.4e-13 if fam in (4, 5) else 1e-13
    assert np.all(np.abs(act["Q"][idx] - ref["Q"]) <= tol * np.maximum(np.abs(ref["Q"]), ref["scaleQ"]))
    assert np.all(np.abs(act["err"][idx] - ref["err"]) <= tol * ref["scaleE"])


@pytest.mark.parametrize("rule", [0, 2])
@pytest.mark.parametrize("d", [7, 8, 9, 10])
@pytest.mark.parametrize("fam", FACTORED)
def test_adjoint(fam, d, rule):
    """The factored adjoint (d = 7..10) on a small tree with retired leaves and an
    active set, against the oracle's node-by-node derivative sums: 1e-12 of the
    largest component, as for every gradient (sums of the same nodes in another
    grouping)."""
    p = W.family_params(fam, d, seed=1100 + 10 * fam + d)
    lo, hi = W.unit_box(d)
    opts = {"max_iters": 3, "rule": rule, "init_log2_regions": d if d < 9 else 4}
    for k, v in opts.items():
        gm.set_option(k, v)
    try:
        print(f"case adjoint fam={fam} d={d} rule={rule}", flush=True)
        I, _, g, st = gm.integrate_grad(fam, p, lo, hi, 1e-4, 1e-300, 1 << 16)
    finally:
        for k, v in {"max_iters": 10000, "rule": 0, "init_log2_regions": 12}.items():
            gm.set_option(k, v)
    ref = O.integrate_grad(fam, p, lo, hi, 1e-4, 1e-300, 1 << 16,
                           init_log2=opts["init_log2_regions"], max_iters=3, rule_id=rule)
    assert st == ref["status"]
    assert abs(I - ref["I"]) <= 1e-12 * abs(ref["I"]) + 1e-300
    scale = max(np.abs(ref["grad"]).max(), 1e-300)
    assert np.abs(g - ref["grad"]).max() <= 1e-12 * scale, (g, ref["grad"])


@pytest.mark.parametrize("d,lanes", [(7, (0, 1, 4)), (8, (1, 4, 16)), (9, (0, 16)), (10, (1, 16, 64)),
                                     (11, (4, 64)), (13, (4, 16)), (16, (16, 64))])
def test_corner_quotient_mappings(d, lanes):
    """The corner peak with four nodes to a reciprocal, at the edges of its mappings."""
    p = W.family_params(3, d, seed=2100 + d)
    lo, hi = W.unit_box(d)
    for ln in lanes:
        print(f"case corner d={d} lanes={ln}", flush=True)
        act, chain = _stopped_run(3, p, lo, hi, 4 if d <= 11 else 3, lanes=ln)
        _check(3, p, lo, hi, act, chain, 0, f"corner d{d} lanes{ln}")


@pytest.mark.parametrize("a", [2.8e7, 3.0e7, -(1 - 2.0 ** -27) / 8, -(1 - 2.0 ** -29) / 8, -0.2])
def test_corner_both_sides_of_the_line(a):
    """1 + sum a_j x_j reaching up or down to either side of the quotient form's
    range (2^+-27.8 at d = 8), and through zero.  Where it falls towards 0, the
    smallest at a node is above 0.02, and the rounding of the d terms (2^-53 each)
    is raised to the power d + 1: 72 2^-53 / 0.02 = 4e-13."""
    d = 8
    lo, hi = W.unit_box(d)
    p = np.concatenate([np.full(d, a), np.zeros(d)])
    print(f"case corner line a={a}", flush=True)
    if a == -0.2:  # singular inside the box: reported as before
        assert gm.integrate(3, p, lo, hi, 1e-12, 1e-300, 1 << 16)[2] == gm.NONFINITE
        return
    act, _ = _stopped_run(3, p, lo, hi, 2)
    idx = np.unique(np.linspace(0, act["lvl"].size - 1, 40).astype(int))
    ref = O.rule_many(3, p, act["c"][idx], act["h"][idx], act["lvl"][idx], 1.0)
    assert np.all(np.abs(act["Q"][idx] - ref["Q"]) <= 4e-13 * np.maximum(np.abs(ref["Q"]), ref["scaleQ"]))
    assert np.all(np.abs(act["err"][idx] - ref["err"]) <= 4e-13 * ref["scaleE"])


@pytest.mark.parametrize("n", [8191, 8192, 8193])
def test_list_layouts(n):
    """Region lists on either side of the line (32768 coordinates) below which the
    host lays them out: the bits of the same regions in short lists."""
    d = 4
    rng = np.random.default_rng(n)
    p = W.family_params(4, d, seed=9)
    lvl = rng.integers(0, 12, n).astype(np.int32)
    h = np.repeat(np.ldexp(0.5, -(lvl // d))[:, None], d, axis=1)
    c = h + rng.uniform(0.0, 1.0, (n, d)) * (1.0 - 2.0 * h)
    lo, hi = W.unit_box(d)
    print(f"case list n={n}", flush=True)
    whole = gm.eval_regions(4, p, lo, hi, c, h, lvl)
    for a in range(0, n, 3000):
        part = gm.eval_regions(4, p, lo, hi, c[a:a + 3000], h[a:a + 3000], lvl[a:a + 3000])
        for x, y in zip(whole, part):
            assert np.array_equal(x[a:a + 3000], y)
