"""Workloads of the framework that its speed is measured on.

Each case is one call of a public entry point of paper_2511_01573_amd, as a
program that integrates the library's families on the unit box makes it:
single integrals (ordinary, allocation-free, high-dimensional), the degree-9
and Gauss-Kronrod rules, a batch of mixed integrals, the gradient (with its
autograd function) and the rule on a caller's region list.  Parameters are
drawn as workloads.family_params draws them: a ~ U(0,1)^d rescaled to a sum
that sets the difficulty, u ~ U(0,1)^d (the discontinuous family's cuts stay
inside the box), from the seed alone.

A case holds
  call     integrate | noalloc | batch | grad | autograd | regions
  family   the integrand (batch: drawn per item), d its dimension
  sum_a    sum of a_j (batch: a factor on each family's own difficulty)
  rel_tol, log2_store   tolerance and capacity 2^log2_store of the region set
  rule, err_model, prune   the process-wide options of the call
  init_log2   log2 of the initial partition's cells (12 is the library's default)
  n        items (batch) or regions (regions)
"""
from __future__ import annotations

import math
from fractions import Fraction

import numpy as np
import torch

from paper_2511_01573_amd import autograd, gm, workloads as W

ABS_TOL = 1e-16
BATCH_FAMILIES = ("gaussian", "oscillatory", "product_peak")


def _case(name, call, family, d, sum_a, rel_tol, log2_store, rule=0, err_model=0, prune=0, n=1,
          init_log2=12):
    c = dict(call=call, family=family, d=d, sum_a=sum_a, rel_tol=rel_tol, log2_store=log2_store,
             rule=rule, err_model=err_model, prune=prune, init_log2=init_log2, n=n)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest ordinary call: a peak in three dimensions, a few thousand regions, so
        # launches and status reads are what it costs
        _case("single_d3_gaussian", "integrate", "gaussian", 3, 15.0, 1e-6, 17),
        # the allocation-free entry point of a serving loop, an even smaller call
        _case("noalloc_d5_c0", "noalloc", "c0", 5, 2.5, 1e-4, 16),
        # the d = 8 suite's tightest tolerance on a family with a transcendental outer function
        _case("suite_d8_gaussian", "integrate", "gaussian", 8, 13.0, 1e-7, 24),
        # the suite's ordinary tolerance on its discontinuous family: regions pile up along the cut
        _case("suite_d8_discontinuous", "integrate", "discontinuous", 8, 10.0, 1e-5, 24),
        # the suite's largest run: it fills the store of 2^24 regions or comes close
        _case("suite_d8_oscillatory", "integrate", "oscillatory", 8, 9.0, 1e-7, 24),
        # the suite's family of costly nodes (a power and a reciprocal each)
        _case("suite_d8_corner_peak", "integrate", "corner_peak", 8, 2.0, 1e-7, 24),
        # high dimension: 2^13 corners a region, several lanes to a region
        _case("high_d13_product_peak", "integrate", "product_peak", 13, 30.0, 1e-4, 24),
        # the degree-9 rule with its null-rule error model at a tight tolerance
        _case("degree9_d8_c0", "integrate", "c0", 8, 4.0, 1e-6, 24, rule=2, err_model=1),
        # the tensor-product Gauss-Kronrod rule in few dimensions, where it is the rule of choice;
        # it starts from the whole box, as its benchmark runs do
        _case("kronrod_d4_product_peak", "integrate", "product_peak", 4, 60.0, 1e-6, 16, rule=1,
              init_log2=3),
        # many small integrals of mixed dimension and family in one call
        _case("batch_mixed_4096", "batch", "mixed", 10, 0.35, 1e-6, 27, n=4096),
        # parameter gradient of a tight integral with the degree-9 rule (forward tree + adjoint)
        _case("grad9_d8_gaussian", "grad", "gaussian", 8, 24.0, 1e-7, 25, rule=2),
        # the rule alone on a caller's list of regions, a ragged count
        _case("regions_d7_polynomial", "regions", "poly_f7", 7, 1.0, 1e-6, 0, n=30011),
    ]


def _spread(rng, lo, hi):
    """A number in [lo, hi], spread over its logarithm."""
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    call = rng.choice(["integrate", "integrate", "integrate", "noalloc", "batch", "grad",
                       "autograd", "regions"])
    family = rng.choice(["oscillatory", "product_peak", "corner_peak", "gaussian", "c0",
                         "discontinuous"])
    rule = rng.choice([0, 0, 2])
    err_model = rng.choice([0, 1]) if rule == 2 else 0
    opts = dict(rule=rule, err_model=err_model)
    tol = _spread(rng, 1e-6, 1e-4)
    if call == "batch":
        return _case(None, "batch", "mixed", rng.randint(4, 10), rng.uniform(0.2, 0.35),
                     _spread(rng, 1e-5, 1e-3), 26, n=round(_spread(rng, 3, 3000)), **opts)
    if call == "regions":
        family = "poly_f7" if rng.random() < 0.2 else family
        d = rng.randint(2, 14)
        n = round(_spread(rng, 1, min(60000, 3e7 / 2 ** d)))
        return _case(None, "regions", family, d, _difficulty(family, d), 1e-6, 0, n=n, **opts)
    if call == "integrate" and rng.random() < 0.15:  # Gauss-Kronrod: few dimensions
        family = rng.choice(["product_peak", "gaussian", "c0"])
        d = rng.randint(2, 5)
        return _case(None, "integrate", family, d, d * (3.0 if family == "c0" else 12.0),
                     _spread(rng, 1e-6, 1e-4), 16, rule=1, init_log2=3)
    if call in ("grad", "autograd"):
        d, store = rng.randint(2, 9), 21
    elif call == "noalloc":
        d, store = rng.randint(2, 12), 16
    else:
        d = rng.randint(2, 16)
        store = rng.randint(18, 23) if d <= 10 else 33 - d
    prune = rng.choice([0, 0, 1]) if call in ("integrate", "noalloc") and d <= 10 else 0
    # in few dimensions, and at degree 9, the default partition would already resolve these
    # integrands: start coarser, and for degree 9 with sharper ones
    coarse, sharp = (8, 2.5) if rule == 2 else (5, 1.0)
    return _case(None, call, family, d, sharp * _difficulty(family, d), tol, store, prune=prune,
                 init_log2=3 if d <= coarse else 12, **opts)


def _difficulty(family, d):
    """Sum of a_j: the d = 8 suite's, scaled with the dimension between 4 and 10."""
    return W.DIFFICULTY_D8.get(gm.FAMILIES[family], 8.0) * min(max(d, 4), 10) / 8.0


def _batch(case, seed):
    """n items, d ~ U{3..d_max}, one of three families, rel_tol spread from the case's to 1e-3."""
    rng = np.random.default_rng(seed)
    out = dict(families=[], params=[], ds=[], los=[], his=[], rel_tols=[])
    for _ in range(case["n"]):
        d = int(rng.integers(3, case["d"] + 1))
        fam = BATCH_FAMILIES[int(rng.integers(0, 3))]
        a = rng.uniform(0.0, 1.0, d)
        u = rng.uniform(0.0, 1.0, d)
        a *= case["sum_a"] * W.DIFFICULTY_D8[gm.FAMILIES[fam]] * d / 8.0 / a.sum()
        out["families"].append(fam)
        out["params"].append(np.concatenate([a, u]))
        out["ds"].append(d)
        out["los"].append(np.zeros(d))
        out["his"].append(np.ones(d))
        out["rel_tols"].append(10.0 ** rng.uniform(math.log10(case["rel_tol"]), -3.0))
    return out


def _params(case, seed):
    return W.family_params(gm.FAMILIES[case["family"]], case["d"], seed, case["sum_a"])


def prepare(case, seed):
    gm.lib()
    s = dict(case)
    if case["call"] == "batch":
        s["items"] = _batch(case, seed)
        return s
    d = case["d"]
    s["params"] = _params(case, seed)
    s["lo"], s["hi"] = np.zeros(d), np.ones(d)
    if case["call"] == "regions":
        s["c"], s["h"], s["lvl"] = W.random_regions(d, case["n"], seed)
    if case["call"] == "autograd":
        s["theta"] = torch.from_numpy(s["params"]).clone().requires_grad_(True)
    return s


def run(s):
    for key in ("rule", "err_model", "prune"):
        gm.set_option(key, s[key])
    gm.set_option("init_log2_regions", s["init_log2"])
    call = s["call"]
    cap = 1 << s["log2_store"]
    if call == "batch":
        b = s["items"]
        n = len(b["ds"])
        _, est, err, status = gm.integrate_batch(b["families"], b["params"], b["ds"], b["los"],
                                                 b["his"], b["rel_tols"], [ABS_TOL] * n, cap)
        return {"est": est, "err": err, "status": status}
    if call == "regions":
        q, err, axis = gm.eval_regions(s["family"], s["params"], s["lo"], s["hi"], s["c"], s["h"],
                                       s["lvl"])
        return {"est": q, "err": err, "axis": axis}
    if call == "autograd":
        value = autograd.integral(s["theta"], s["family"], s["lo"], s["hi"], s["rel_tol"], ABS_TOL,
                                  cap)
        (grad,) = torch.autograd.grad(value, s["theta"])
        return {"est": value, "grad": grad}
    if call == "grad":
        est, err, grad, status = gm.integrate_grad(s["family"], s["params"], s["lo"], s["hi"],
                                                   s["rel_tol"], ABS_TOL, cap)
        return {"est": est, "err": err, "grad": grad, "status": status}
    fn = gm.integrate if call == "integrate" else gm.integrate_noalloc
    est, err, status = fn(s["family"], s["params"], s["lo"], s["hi"], s["rel_tol"], ABS_TOL, cap)
    return {"est": est, "err": err, "status": status}


def work(case):
    """Every node of every evaluated region costs at least one multiply-add, and
    each region's geometry (d centres and widths, shared by two siblings) and
    its value, error, level and axis have to be read and written once.  How many
    regions a run evaluates is the run's own affair: it is read off one."""
    if case["call"] == "regions":
        n, d = case["n"], case["d"]
        evals = n * _nodes(d, case["rule"])
        return {"bytes": n * (16 * d + 4 + 20), "flops": 2.0 * evals}
    run(prepare(case, 1))
    st = gm.last_stats()
    evals, regions = st["evals"], st["regions_evaluated"]
    if case["call"] in ("grad", "autograd"):  # the adjoint visits the leaves of the tree
        leaves = st["finished"] + st["final_active"]
        evals += leaves * _nodes(case["d"], case["rule"])
        regions += leaves
    return {"bytes": float(regions * (8 * case["d"] + 20)), "flops": 2.0 * evals}


def _nodes(d, rule):
    if rule == 1:
        return 15 ** d
    if rule == 2:
        return 1 + 6 * d + 6 * d * (d - 1) + 4 * d * (d - 1) * (d - 2) // 3 + 2 ** d
    return 1 + 2 * d + 2 * d * d + 2 ** d


# Closed forms on the unit box (and their parameter derivatives where the
# integral is a product over the axes), in 64 bits.
def _axis_factors(family, a, u):
    """Per axis: int_0^1 g(x) dx and its derivatives in a and u, for the
    families that are products of one-axis factors."""
    if family == "gaussian":
        F = [math.sqrt(math.pi) / (2 * x) * (math.erf(x * (1 - y)) + math.erf(x * y))
             for x, y in zip(a, u)]
        e0 = [math.exp(-(x * y) ** 2) for x, y in zip(a, u)]
        e1 = [math.exp(-(x * (1 - y)) ** 2) for x, y in zip(a, u)]
        da = [(-f + (1 - y) * q + y * p) / x for f, p, q, x, y in zip(F, e0, e1, a, u)]
        return F, da, [p - q for p, q in zip(e0, e1)]
    if family == "product_peak":
        F = [x * (math.atan(x * (1 - y)) + math.atan(x * y)) for x, y in zip(a, u)]
        da = [f / x + x * ((1 - y) / (1 + (x * (1 - y)) ** 2) + y / (1 + (x * y) ** 2))
              for f, x, y in zip(F, a, u)]
        du = [x * x * (1 / (1 + (x * y) ** 2) - 1 / (1 + (x * (1 - y)) ** 2))
              for x, y in zip(a, u)]
        return F, da, du
    if family == "c0":  # (its kink keeps the quadrature's u-derivatives from converging to these)
        return [(2 - math.exp(-x * y) - math.exp(-x * (1 - y))) / x for x, y in zip(a, u)], None, None
    if family == "discontinuous":
        return [math.expm1(x * min(y, 1.0)) / x for x, y in zip(a, u)], None, None
    return None


def _closed(family, p):
    d = len(p) // 2
    a, u = [float(x) for x in p[:d]], [float(x) for x in p[d:]]
    if family == "oscillatory":
        amp = [2 * math.sin(x / 2) / x for x in a]
        phase = 2 * math.pi * u[0] + math.fsum(x / 2 for x in a)
        I, S = math.cos(phase) * math.prod(amp), math.sin(phase) * math.prod(amp)
        damp = [math.cos(x / 2) / x - f / x for f, x in zip(amp, a)]
        da = [I * q / f - 0.5 * S for q, f in zip(damp, amp)]
        return I, da + [-2 * math.pi * S] + [0.0] * (d - 1)
    if family == "corner_peak":
        sums = [(Fraction(1), 1)]
        for x in a:
            sums += [(s + Fraction(x), -g) for s, g in sums]
        total = sum((g * (10 ** 120 * s.denominator // s.numerator) for s, g in sums), 0)
        den = math.factorial(d)
        for x in a:
            den *= Fraction(x)
        return float(Fraction(total, 10 ** 120) / den), None
    if family == "poly_f7":
        return None, None
    F, da, du = _axis_factors(family, a, u)
    I = math.prod(F)
    if da is None:
        return I, None
    return I, [I / f * g for f, g in zip(F, da)] + [I / f * g for f, g in zip(F, du)]


def _node_values(family, a, u, x):
    if family == "oscillatory":
        return np.cos(2 * np.pi * u[0] + x @ a)
    if family == "product_peak":
        return np.prod(1.0 / (a ** -2.0 + (x - u) ** 2), axis=1)
    if family == "corner_peak":
        return (1.0 + x @ a) ** -(len(a) + 1.0)
    if family == "gaussian":
        return np.exp(-np.sum((a * (x - u)) ** 2, axis=1))
    if family == "c0":
        return np.exp(-np.sum(a * np.abs(x - u), axis=1))
    if family == "discontinuous":
        return np.where((x > u).any(axis=1), 0.0, np.exp(x @ a))
    return np.sum(x * x, axis=1) ** 11


def _rule7(case, p, c, h, vol):
    """Degree-7 rule value and |Q7 - Q5| of each region, node by node."""
    d = case["d"]
    a, u = p[:d], p[d:]
    l2, l3, l5 = math.sqrt(9 / 70), math.sqrt(9 / 10), math.sqrt(9 / 19)
    S = [np.zeros(len(c)) for _ in range(5)]

    def add(k, off):
        S[k] += _node_values(case["family"], a, u, c + np.asarray(off) * h)

    add(0, np.zeros(d))
    eye = np.eye(d)
    for i in range(d):
        for sg in (1.0, -1.0):
            add(1, sg * l2 * eye[i])
            add(2, sg * l3 * eye[i])
            for j in range(i):
                add(3, l3 * (sg * eye[i] + eye[j]))
                add(3, l3 * (sg * eye[i] - eye[j]))
    for m in range(1 << d):
        add(4, [l5 if m >> j & 1 else -l5 for j in range(d)])
    w = [(400 * d * d - 9120 * d + 12824) / 19683, 980 / 6561, (1820 - 400 * d) / 19683,
         200 / 19683, 6859 / 19683 / 2 ** d]
    v = [(950 * d * d - 16530 * d + 6859) / 19683, -4655 / 13122, (1900 * d - 3515) / 39366,
         -475 / 19683, w[4]]
    v[0] *= -1.0
    q = sum(x * s for x, s in zip(w, S))
    e = sum(x * s for x, s in zip(v, S))
    return vol * q, vol * np.abs(e)


def exact(case, seed):
    call = case["call"]
    if call == "batch":
        b = _batch(case, seed)
        return {"est": np.array([_closed(f, p)[0] for f, p in zip(b["families"], b["params"])]),
                "err": None, "status": None}
    p = _params(case, seed)
    if call == "regions":
        if case["rule"] != 0 or case["n"] * _nodes(case["d"], 0) * case["d"] > 2e8:
            return None
        c, h, lvl = W.random_regions(case["d"], case["n"], seed)
        q, e = _rule7(case, p, c, h, np.ldexp(1.0, -lvl))
        return {"est": q, "err": e, "axis": None}
    est, grad = _closed(case["family"], p)
    grad = None if grad is None else np.array(grad)
    if call == "autograd":
        return {"est": est, "grad": grad}
    if call == "grad":
        return {"est": est, "err": None, "grad": grad, "status": None}
    return {"est": est, "err": None, "status": None}
