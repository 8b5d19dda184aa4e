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
