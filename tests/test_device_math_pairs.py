"""Accuracy of the sine-cosine pairs that the factored oscillatory kernels turn
with, with and without the reduced argument's tail, and of the reciprocal that the
corner peak's quotients take (paper_2511_01573_amd/csrc/gm_math.hpp), compiled for
the host from the same source, against 60-digit references.

Tolerances.  With the tail the reduction is that of cos and sin, 1.5 ulp of 1.
Without it the reduced argument |r| <= pi/2 is rounded, by at most 2^-53, which moves
either function by as much: 2 ulp of 1.  The reciprocal's estimate is good to 2^-22
(the host's is cut to that), its error enters as the cube, 2^-66, and only the last
operation rounds: 0.51 ulp."""
from __future__ import annotations

import ctypes as C
import os
import subprocess

import mpmath as mp
import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DP = C.POINTER(C.c_double)


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("pairs") / "libpairs.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared",
                           "-I", os.path.join(ROOT, "paper_2511_01573_amd", "csrc"),
                           os.path.join(ROOT, "tests", "math_pairs_harness.cpp"), "-o", so])
    L = C.CDLL(so)
    L.gm_test_sincos.argtypes = [DP, DP, DP, DP, C.c_long, C.c_int]
    L.gm_test_rcp3.argtypes = [DP, DP, C.c_long]
    return L


def _p(a):
    return a.ctypes.data_as(DP)


@pytest.mark.parametrize("tail", [True, False])
def test_sincos_pairs(harness, tail):
    mp.mp.dps = 60
    rng = np.random.default_rng(11)
    x = np.concatenate([rng.uniform(-10, 10, 2000), rng.uniform(-200, 200, 800),
                        rng.uniform(-1e5, 1e5, 300), np.arange(-20, 21) * (np.pi / 2),
                        [0.0, -0.0, 1e-300, 2e6, -3e7]])
    xl = rng.uniform(-1, 1, x.size) * np.abs(x) * 2.0 ** -53 if tail else np.zeros(x.size)
    s, c = np.zeros(x.size), np.zeros(x.size)
    harness.gm_test_sincos(_p(x), _p(xl), _p(s), _p(c), x.size, int(tail))
    angle = [mp.mpf(a) + mp.mpf(b) for a, b in zip(x, xl)]
    bound = (1.5 if tail else 2.0) * 2.0 ** -52
    es = np.array([float(abs(mp.mpf(v) - mp.sin(a))) for v, a in zip(s, angle)])
    ec = np.array([float(abs(mp.mpf(v) - mp.cos(a))) for v, a in zip(c, angle)])
    assert es.max() <= bound, (es.max() * 2.0 ** 52, x[np.argmax(es)])
    assert ec.max() <= bound, (ec.max() * 2.0 ** 52, x[np.argmax(ec)])


def test_quick_reciprocal(harness):
    mp.mp.dps = 60
    rng = np.random.default_rng(12)
    x = np.ldexp(rng.uniform(1.0, 2.0, 6000), rng.integers(-1000, 1000, 6000))
    x = np.concatenate([x, -x[:500], 2.0 ** np.arange(-1000, 1000, 37.0),
                        np.nextafter(2.0 ** np.arange(-990, 1000, 41.0), 0.0)])
    y = np.zeros(x.size)
    harness.gm_test_rcp3(_p(x), _p(y), x.size)
    err = np.array([float(abs(mp.mpf(a) * mp.mpf(b) - 1) * abs(1 / mp.mpf(b)) / mp.mpf(float(np.spacing(abs(a)))))
                    for a, b in zip(y, x)])
    assert err.max() <= 0.51, (err.max(), x[np.argmax(err)])
