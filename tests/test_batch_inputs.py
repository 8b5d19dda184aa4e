"""What gm.integrate_batch takes for its items' families and arrays, without a
GPU: items of d = 11 are invalid in a batch, so a call with only such items ends
before any device work with GM_EINVAL per item -- after the binding has read
every argument."""
from __future__ import annotations

import enum
import itertools
import warnings

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


DTYPES = ["bool", "i1", "u1", "i2", "u2", "i4", "u4", "i8", "u8", "f2", "f4", "f8", "g", "c8",
          "c16", "O", "U24"]


@pytest.mark.parametrize("pair", list(itertools.combinations_with_replacement(DTYPES, 2)),
                         ids=lambda p: "-".join(p))
def test_packed_arrays_of_mixed_types(pair):
    """Items of any two types are joined as the float64 values that each has by itself."""
    base = np.array([1, 0, 1, 0, 1])
    wide = np.array([2.0 ** 53 + 2, 0.1, 3.0, -7.25, 1e-9])
    items = []
    for k, t in enumerate(pair):
        x = base if t == "bool" else (base + 100 + k) if t[0] in "iu" else wide.astype("f4") if t == "f2" else wide
        if t in ("i8", "u8"):
            x = base + (2 ** 53 + 3)
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            items.append(x.astype(t))
    items.append([1.5, 2, 3])
    for some in (items[:2], items, [items[1], items[0]]):
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            want = np.concatenate([np.asarray(x, float) for x in some])
            got = gm._packed(some)
        assert got.dtype == np.float64 and np.array_equal(got, want, equal_nan=True)


@pytest.mark.parametrize("item", [list, np.array], ids=["lists", "arrays"])
def test_packed_takes_iterators(item):
    """Every item of an iterator arrives, whatever its items are."""
    rows = [[1.0, 2.0, 3.0], [4.0, 5.0, 6.0], [7.0, 8.0, 9.0]]
    got = gm._packed(item(r) for r in rows)
    assert np.array_equal(got, np.arange(1.0, 10.0))
