"""What gm.integrate_batch takes for its items' families and arrays, without a
GPU: items of d = 11 are invalid in a batch, so a call with only such items ends
before any device work with GM_EINVAL per item -- after the binding has read
every argument."""
from __future__ import annotations

import enum

import numpy as np
import pytest

from paper_2511_01573_amd import gm


class Name(str):
    pass


class Kind(str, enum.Enum):
    GAUSSIAN = "gaussian"
    C0 = "c0"


@pytest.mark.parametrize("families", [
    ["gaussian", "c0"], np.array(["gaussian", "c0"]), [np.str_("gaussian"), np.str_("c0")],
    [Name("gaussian"), Name("c0")], [Kind.GAUSSIAN, Kind.C0], [4, 5], np.array([4, 5]),
    (np.int64(4), "c0")], ids=lambda f: f"{type(f).__name__}-{type(f[0]).__name__}")
def test_family_names(families):
    d = 11
    p, lo, hi = np.ones(2 * d), np.zeros(d), np.ones(d)
    rc, _, _, status = gm.integrate_batch(families, [p, p], [d, d], [lo, lo], [hi, hi],
                                          [1e-3, 1e-3], [1e-16, 1e-16], 1 << 16)
    assert rc == gm.OK and list(status) == [gm.EINVAL, gm.EINVAL]


def test_unknown_family_name():
    d = 11
    p, lo, hi = np.ones(2 * d), np.zeros(d), np.ones(d)
    with pytest.raises(KeyError):
        gm.integrate_batch([np.str_("gauss")], [p], [d], [lo], [hi], [1e-3], [1e-16], 1 << 16)
