"""Calls of libgm that fail half way leave nothing running: the host code of
libgm.so on a test double of the HIP runtime (tests/hip_double.cpp), on the CPU.  A
call that returns with launches that no synchronisation has followed would leave
kernels working on a workspace, a leaf store or status slots that the caller or
the next call may free or use."""
from __future__ import annotations

import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes as C, json, sys
root, double, spec = sys.argv[1], sys.argv[2], json.loads(sys.argv[3])
sys.path.insert(0, root)
D = C.CDLL(double, mode=C.RTLD_GLOBAL)      # before libgm.so: its names are found first
import numpy as np
from paper_2511_01573_amd import gm
D.double_reset.argtypes = [C.c_int, C.c_int, C.c_int64, C.c_int]
SEQ = 27  # words of the status block (gm_common.hpp Status), then the number
out = []
def call(kind, fail_malloc=0, fail_launch=0, stop=6):
    stop = {"grad": stop, "integrate": -stop, "regions": 0, "batch": 0}[kind]
    D.double_reset(fail_malloc, fail_launch, stop, SEQ)
    d, n = 3, 20000
    box = ("gaussian", np.ones(2 * d), np.zeros(d), np.ones(d))
    try:
        if kind == "batch":
            k = 300
            gm.integrate_batch(["gaussian"] * k, [box[1]] * k, [d] * k, [box[2]] * k, [box[3]] * k,
                               [1e-9] * k, [1e-300] * k, 1 << 21, stream=0)
        elif kind == "regions":
            gm.eval_regions(*box, np.zeros((n, d)), np.ones((n, d)), np.zeros(n), stream=0)
        else:
            fn = gm.integrate_grad if kind == "grad" else gm.integrate
            fn(*box, 1e-9, 1e-300, 1 << 15, stream=0)
        rc = 0
    except gm.GMError as e:
        rc = e.code
    return [rc, D.double_pending(), D.double_launches(), D.double_events()]
for k, v in spec["options"].items():
    gm.set_option(k, v)
if spec["call"] == "batch":  # (the double ends no batch)
    out = [[0, 0], call("batch", **spec["fail"]), [0, 0]]
else:
    out.append(call(spec["call"], stop=2))  # makes workspace, slots and a small leaf store
    out.append(call(spec["call"], **spec["fail"]))
    out.append(call(spec["call"]))
print("RESULT " + json.dumps(out))
"""


@pytest.fixture(scope="module")
def double(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("double") / "libhipdouble.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared",
                           os.path.join(ROOT, "tests", "hip_double.cpp"), "-o", so])
    return so


@pytest.mark.parametrize("call,fail,options,rc", [
    ("grad", {"fail_malloc": 1}, {}, -2),   # the leaf store cannot grow: 20000 + 15000 k regions
    ("grad", {"fail_launch": 9}, {}, -3),
    ("grad", {"fail_launch": 21}, {}, -3),  # the second adjoint launch
    ("integrate", {"fail_launch": 6}, {}, -3),
    ("integrate", {"fail_launch": 7}, {"timing": 1}, -3),
    ("regions", {"fail_launch": 3}, {}, -3),  # the layout of a long list's axes
    ("batch", {"fail_launch": 5}, {}, -3),
    ("batch", {"fail_launch": 5}, {"timing": 1}, -3),
])
def test_failed_call_leaves_nothing_running(double, call, fail, options, rc):
    spec = json.dumps({"call": call, "fail": fail, "options": options})
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, double, spec], capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, (r.stdout[-300:], r.stderr[-1500:])
    good, failed, after = json.loads(r.stdout.split("RESULT ")[1])
    assert good[:2] == [0, 0] and after[:2] == [0, 0], (good, after)
    assert failed[0] == rc
    assert failed[1] == 0, f"{failed[1]} launches pending after the failed call"
    assert failed[3] == 0, f"{failed[3]} events left"
