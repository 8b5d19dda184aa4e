"""A process that asked HIP to block while it waits (hipDeviceScheduleBlockingSync)
gets a call that does: the run loop's reading of the iterations' status leaves the
core to others, with the results of a process that spins."""
from __future__ import annotations

import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu

CHILD = r"""
import ctypes, json, sys, time
sys.path.insert(0, sys.argv[1])
import torch
from paper_2511_01573_amd import gm, workloads as W
gm.lib()
hip = ctypes.CDLL([l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l][0])
assert hip.hipSetDeviceFlags(ctypes.c_uint(int(sys.argv[2]))) == 0
gm.set_option("rule", 1)
gm.set_option("init_log2_regions", 3)
p = W.family_params(5, 6, seed=91, difficulty=9.0)
lo, hi = W.unit_box(6)
out = []
for _ in range(3):   # a few iterations of tens of milliseconds
    w, c = time.perf_counter(), time.process_time()
    I, E, st = gm.integrate(5, p, lo, hi, 1e-6, 1e-16, 1 << 14, stream=0)
    out = [time.perf_counter() - w, time.process_time() - c, I.hex(), E.hex(), st]
print("RESULT " + json.dumps(out))
"""


def _run(flags):
    print("case flags", flags, flush=True)
    r = subprocess.run([sys.executable, "-c", CHILD, ROOT, str(flags)], capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, (r.stdout[-300:], r.stderr[-1500:])
    return json.loads(r.stdout.split("RESULT ")[1])


def test_blocking_wait_leaves_the_core():
    wall, cpu, *blocking = _run(4)
    print("wall", wall, "cpu", cpu, flush=True)
    assert wall > 0.05, "too short to tell"
    assert cpu < 0.3 * wall
    assert blocking == _run(0)[2:]
