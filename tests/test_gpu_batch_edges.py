"""Batches at the edges of the item kernels: item counts around a wavefront's 64
probes (chunk -> item search) and a commit workgroup's 256 items, more items than
one search step covers, groups that empty while others go on, and a shared
capacity that runs out.  Items of d <= 5 run the same rule kernels in a batch and
alone, and both add their regions in double-double: they differ by the last
rounding of I and E."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2511_01573_amd import gm, workloads as W

pytestmark = pytest.mark.gpu


def _items(n):
    out = []
    for k in range(n):
        fam, d = 1 + k % 6, 2 + (k // 6) % 4
        out.append((fam, W.family_params(fam, d, seed=31 * k + 5), np.zeros(d), np.ones(d),
                    (1e-3, 1e-5)[k % 2]))
    return out


def _batch(items, cap):
    fam, p, lo, hi, tol = zip(*items)
    _, est, err, st = gm.integrate_batch(fam, p, [len(x) for x in lo], lo, hi, tol,
                                         [1e-300] * len(items), cap)
    return est, err, st


@pytest.fixture
def small_partition():
    gm.set_option("init_log2_regions", 5)
    yield
    gm.set_option("init_log2_regions", 12)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 4097])
def test_item_counts(n, small_partition):
    items = _items(n)
    print(f"case batch of {n}", flush=True)
    I, E, st = _batch(items, 1 << 22)
    for k in range(0, n, max(1, n // 97)):
        fam, p, lo, hi, tol = items[k]
        i1, e1, s1 = gm.integrate(fam, p, lo, hi, tol, 1e-300, 1 << 20)
        assert st[k] == s1, k
        assert abs(I[k] - i1) <= 1e-14 * abs(i1) and abs(E[k] - e1) <= 1e-14 * e1, k


def test_capacity_runs_out(small_partition):
    items = [(4, W.family_params(4, 5, seed=k, difficulty=20.0), np.zeros(5), np.ones(5), 1e-9)
             for k in range(300)]
    print("case capacity", flush=True)
    I, E, st = _batch(items, 300 * 32)
    assert np.all(np.asarray(st) == gm.MAX_REGIONS) and np.all(np.isfinite(E)) and np.all(np.isfinite(I))


@pytest.mark.parametrize("fam", [1, 2, 4, 5, 6])
@pytest.mark.parametrize("d,lanes", [(8, 4), (8, 16), (9, 16), (10, 4), (10, 64)])
def test_tiles_of_several_lanes(fam, d, lanes):
    """A tile entry with several lanes per region, where the one-lane kernel of the
    dimension is the factored one: same statuses, and I to 1e-12 (the batch's bar)."""
    args = ([fam] * 3, [W.family_params(fam, d, seed=50 * fam + k, difficulty=2.0) for k in range(3)],
            [d] * 3, [np.zeros(d)] * 3, [np.ones(d)] * 3, [1e-3] * 3, [1e-300] * 3, 1 << 20)
    print(f"case tile fam={fam} d={d} lanes={lanes}", flush=True)
    _, i0, e0, s0 = gm.integrate_batch(*args)
    gm.set_tile(d, fam, lanes, 0)
    try:
        _, i1, e1, s1 = gm.integrate_batch(*args)
    finally:
        gm.set_tile(d, fam, 0, 0)
    assert np.array_equal(s0, s1)
    assert np.all(np.abs(i1 - i0) <= 1e-12 * np.abs(i0))
