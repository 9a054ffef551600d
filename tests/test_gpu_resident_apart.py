"""Resident solves where the GPU keeps their workgroups apart: a stream with half
of the compute units, of which the solve's launch needs more."""
import contextlib
import ctypes as C
import time

import numpy as np
import pytest

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu


def _hip():
    import torch
    torch.cuda.init()
    P.load()
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return C.CDLL(path)


@contextlib.contextmanager
def _masked_stream(units):
    hip, s = _hip(), C.c_void_p()
    words = (C.c_uint32 * 8)(*[(1 << min(32, max(0, units - 32 * i))) - 1 for i in range(8)])
    assert hip.hipExtStreamCreateWithCUMask(C.byref(s), 8, words) == 0
    try:
        yield s.value
    finally:
        assert hip.hipStreamDestroy(s) == 0


def _problem():
    return W.lasso(8000, 1000, seed=3, dtype=np.float32)  # 200 workgroups


def test_workgroups_kept_apart_give_up_soon():
    """The wait for workgroups that cannot arrive is 7 ms (0.7 s before a
    launch's first exchange had a bound of its own); a solve with one launch
    per step takes 2 ms."""
    p = _problem()
    with _masked_stream(128) as s, P.Context(p.A, stream=s) as ctx, P.Context(p.A, stream=s) as steps:
        steps.set_resident_wait(-1)
        want = steps.solve(p.f, p.g)
        ctx.set_resident_wait(P.POGS_RESIDENT_WAIT - 1)
        for i in (1, 2):
            t0 = time.perf_counter()
            r = ctx.solve(p.f, p.g)
            assert time.perf_counter() - t0 < 0.2
            assert (ctx.route().resident_last, ctx.route().resident_give_ups) == (0, i)
            for k in ("x", "y", "mu", "nu"):
                np.testing.assert_array_equal(getattr(r, k), getattr(want, k))


@pytest.mark.parametrize("units,resident", [(256, 1), (255, 0), (128, 0)])
def test_restricted_stream_runs_one_launch_per_step(units, resident):
    """A context on a stream that leaves out compute units does not wait for
    workgroups at all; a mask of all units is no restriction."""
    p = _problem()
    with _masked_stream(units) as s:
        for _ in range(2):  # contexts made one after another: nothing is learned from the first
            with P.Context(p.A, stream=s) as ctx:
                assert ctx.solve(p.f, p.g).converged
                r = ctx.route()
                assert (r.resident_workgroups, r.resident_last, r.resident_give_ups) == (200, resident, 0)
