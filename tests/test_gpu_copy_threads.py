"""The serving engine copies large requests on at most as many threads as the
process has CPUs, the caller among them, and gives the same results on any
number of them."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import json, os, sys
sys.path.insert(0, {root!r})
cpus = sorted(os.sched_getaffinity(0))[:{cpus}]
os.sched_setaffinity(0, cpus)
from paper_1503_08366_amd import pogs as P, workloads as W
p = W.lasso(9001, 300, seed=2)
eng = P.BatchEngine()
t = eng.submit(p)
eng.wait_all()
r = eng.poll(t)
names = [open("/proc/self/task/%s/comm" % k).read().strip() for k in os.listdir("/proc/self/task")]
print(json.dumps([len(cpus), names.count("pogs-copy"), r.iters, r.optval, float(abs(r.x).sum())]), flush=True)
eng.close()
"""


def test_copy_threads_fit_the_cpus():
    got = {}
    for cpus in (1, 3, 64):
        out = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT, cpus=cpus)], capture_output=True, text=True,
                             timeout=100)
        assert out.returncode == 0, out.stderr[-2000:]
        have, threads, *result = json.loads(out.stdout.strip().splitlines()[-1])
        # the uploader's own three copy threads, where this request started them
        assert threads in (min(7, have - 1), min(7, have - 1) + 3), (have, threads)
        got[cpus] = result
    assert got[1] == got[3] == got[64]
