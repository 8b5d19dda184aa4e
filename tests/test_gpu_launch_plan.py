"""Which kernels a run launches, and so the last bits of its estimate and error,
follow from the run alone: gm_integrate_noalloc as the first call of a process
(which has no pinned status slots yet), gm_integrate, the same with "timing",
gm_integrate_noalloc afterwards, and gm_integrate with two, three and eight iterations
in flight give the same bits.  Dimensions, rules and
families with more than one rule-kernel mapping, on sets that grow and shrink
across the lines between them."""
from __future__ import annotations

import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu

CHILD = r"""
import json, sys
sys.path.insert(0, sys.argv[1])
import numpy as np
from paper_2511_01573_amd import gm, workloads as W
fam, d, rule, tau, log2cap, init, flight = json.loads(sys.argv[2])
gm.set_option("rule", rule)
gm.set_option("init_log2_regions", init)
gm.set_option("graph_iters", flight)
p = W.family_params(fam, d, seed=40 + d)
lo, hi = W.unit_box(d)
out = []
for call in ("noalloc", "integrate", "timing", "noalloc", 2, 3, 8):
    print("call", call, flush=True)
    gm.set_option("timing", call == "timing")
    if call in (2, 3, 8):  # as many in flight
        gm.set_option("graph_iters", call)
    fn = gm.integrate_noalloc if call == "noalloc" else gm.integrate
    I, E, st = fn(fam, p, lo, hi, tau, 1e-16, 1 << log2cap)
    s = gm.last_stats()
    act = gm.last_active(d)
    out.append([I.hex(), E.hex(), st, s["iterations"], s["regions_evaluated"], s["max_active"],
                act["Q"].tobytes().hex()[-4096:], act["err"].tobytes().hex()[-4096:],
                act["c"].tobytes().hex()[-4096:]])
print("RESULT " + json.dumps(out))
"""


@pytest.mark.parametrize("fam,d,rule,tau,log2cap,init,flight", [
    (4, 6, 0, 1e-7, 16, 12, 0),   # chain form, four lanes or one
    (7, 6, 0, 1e-9, 17, 9, 0),
    (3, 8, 0, 1e-6, 17, 12, 0),   # corner peak, 16 lanes, four or one
    (3, 8, 0, 1e-6, 17, 12, 3),   # ... with a number in flight of the caller's
    (3, 10, 0, 1e-5, 16, 12, 0),
    (2, 12, 0, 1e-4, 17, 12, 0),  # factored, 64 lanes to one
    (1, 11, 0, 1e-5, 17, 12, 0),
    (3, 7, 2, 1e-8, 17, 7, 0),    # degree 9, 64 lanes or the dimension's own number
    (4, 10, 2, 1e-7, 16, 12, 0),  # degree 9 factored, 64 lanes or one
    (4, 5, 0, 1e-7, 16, 12, 0),   # one mapping only
])
def test_first_call_of_a_process(fam, d, rule, tau, log2cap, init, flight):
    case = json.dumps([fam, d, rule, tau, log2cap, init, flight])
    print("case", case, flush=True)
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, case], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, (r.stdout[-500:], r.stderr[-1500:])
    first, *rest = json.loads(r.stdout.split("RESULT ")[1])
    print(first[:6], flush=True)
    assert len(rest) == 6
    for name, got in zip(("gm_integrate", "gm_integrate with timing", "a second noalloc", "two in flight",
                          "three", "eight"), rest):
        assert got == first, (name, got[:6], first[:6])
