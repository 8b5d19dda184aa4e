"""Kernels that a run's size selects, on either side of their lines, against the
chain form on every region and the oracle on a sample (test_gpu_factor's bar): the
degree-9 rule's 64 lanes or one per region at d = 9 and 10, one lane per region
above d = 10, and the bookkeeping in one workgroup or in kernels of its own."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2511_01573_amd import gm, workloads as W
from test_gpu_factor import FACTORED, _check, _stopped_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,iters,init_log2,lanes", [
    (9, 3, 9, 64), (9, 5, 9, 1),      # at most 2048 regions; 8192, the line is 5120
    (10, 2, 10, 64), (10, 4, 10, 1),  # 2048; 8192, the line is 6144
    (11, 2, 11, 64)])
@pytest.mark.parametrize("fam", FACTORED)
def test_degree9_lanes(fam, d, iters, init_log2, lanes):
    p = W.family_params(fam, d, seed=3100 + 10 * fam + d)
    lo, hi = W.unit_box(d)
    print(f"case degree 9 fam={fam} d={d} iters={iters}", flush=True)
    gm.set_option("graph_iters", 1)  # (none launched in vain: the mapping is the last set's)
    try:
        act, chain = _stopped_run(fam, p, lo, hi, iters, rule=2, init_log2=init_log2)
        used = gm.last_stats()["lanes_per_region"]
    finally:
        gm.set_option("graph_iters", 0)
    if iters == 5 or iters == 4:
        # (enough regions kept to pass the line, else the case shows nothing)
        assert (used == lanes) == (act["lvl"].size >= (5120 if d == 9 else 6144))
        if fam in (1, 2):
            assert used == lanes
    else:
        assert used == lanes
    _check(fam, p, lo, hi, act, chain, 2, f"degree 9 fam{fam} d{d} iters{iters}")


@pytest.mark.parametrize("d", [11, 12, 13, 14, 15, 16])
@pytest.mark.parametrize("fam", FACTORED)
def test_one_lane_above_ten_dimensions(fam, d):
    p = W.family_params(fam, d, seed=3300 + 10 * fam + d)
    lo, hi = W.unit_box(d)
    print(f"case one lane fam={fam} d={d}", flush=True)
    act, chain = _stopped_run(fam, p, lo, hi, 4 if d <= 12 else 3, lanes=1,
                              init_log2=3)
    _check(fam, p, lo, hi, act, chain, 0, f"one lane fam{fam} d{d}")


@pytest.mark.parametrize("fam,d,cap", [(4, 6, 70001), (3, 8, 66001), (1, 8, 99999), (2, 11, 81919)])
def test_bookkeeping_on_both_sides_of_its_line(fam, d, cap):
    """Active sets growing past 32768 regions, where one workgroup's bookkeeping
    gives way to a kernel per phase, in stores of odd capacities: estimate, error,
    counts and the last active set are the bits of the run with separate kernels
    throughout (timing = 2)."""
    p = W.family_params(fam, d, seed=3500 + d)
    lo, hi = W.unit_box(d)
    got = []
    for timing in (0, 2):
        print(f"case bookkeeping fam={fam} d={d} timing={timing}", flush=True)
        gm.set_option("timing", timing)
        try:
            r = gm.integrate(fam, p, lo, hi, 1e-9, 1e-300, cap)
            s = gm.last_stats()
            act = gm.last_active(d)
        finally:
            gm.set_option("timing", 0)
        got.append((r, [s[k] for k in ("iterations", "regions_evaluated", "max_active", "finished")],
                    act))
    assert got[0][1][2] > 32768, "the set did not pass the line"
    assert got[0][:2] == got[1][:2]
    for k in got[0][2]:
        assert np.array_equal(got[0][2][k], got[1][2][k]), k
