"""The last active set is that of the most recent single run, or none once another
call has used the workspace that held it."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2511_01573_amd import gm, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("other", ["batch", "regions"])
def test_no_set_is_reported_from_an_overwritten_workspace(other):
    d = 5
    p = W.family_params(4, d, seed=1)
    lo, hi = W.unit_box(d)
    print(f"case last active after {other}", flush=True)
    gm.integrate(4, p, lo, hi, 1e-6, 1e-16, 1 << 16)
    n = gm.last_active_count()
    assert n > 0 and gm.last_active(d)["lvl"].size == n
    if other == "batch":
        gm.integrate_batch([4, 5], [p, p], [d, d], [lo, lo], [hi, hi], [1e-3, 1e-3],
                           [1e-16, 1e-16], 1 << 14)
    else:
        gm.eval_regions(4, p, lo, hi, np.full((9, d), 0.5), np.full((9, d), 0.25), np.zeros(9))
    assert gm.last_active_count() == 0
    gm.integrate(4, p, lo, hi, 1e-6, 1e-16, 1 << 16)
    assert gm.last_active_count() == n
