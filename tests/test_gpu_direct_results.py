"""Results in host memory of at most 256 KB are written there by the last
kernel; larger ones are copied, and device results stay on the device.  The
three routes return the same bits: at the smallest size, odd sizes, either
side of the limit, and from two threads at once."""
import threading

import numpy as np
import pytest

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd.workloads import Fn

pytestmark = pytest.mark.gpu


def _solve(ctx, f, g, device):
    r = ctx.solve(f, g, device_out=device)
    return [np.asarray(getattr(r, k).cpu() if device else getattr(r, k)) for k in ("x", "y", "mu", "nu")] + [
        np.array([r.optval, r.iters])]


@pytest.mark.parametrize("m,n,dt", [(1, 1, np.float32), (67, 33, np.float64), (32704, 64, np.float32),
                                    (32705, 64, np.float32), (16320, 64, np.float64), (16321, 64, np.float64)])
def test_host_results_equal_device_results(m, n, dt):
    rng = np.random.default_rng(m)
    A = rng.normal(size=(m, n)).astype(dt) / np.sqrt(n).astype(dt)
    f, g = Fn("square", m, b=rng.normal(size=m)), Fn("abs", n, c=0.2)
    with P.Context(A, P.default_params(max_iter=12)) as ctx:
        ref = _solve(ctx, f, g, True)
        for a, b in zip(_solve(ctx, f, g, False), ref):
            np.testing.assert_array_equal(a, b)


def test_threads_have_results_of_their_own():
    rng = np.random.default_rng(5)
    probs = [(rng.normal(size=(300, 80)).astype(np.float32), rng.normal(size=300)) for _ in range(2)]
    fg = [(Fn("square", 300, b=b), Fn("abs", 80, c=0.1)) for _, b in probs]
    alone, got = [], [[], []]
    for (A, _), (f, g) in zip(probs, fg):
        with P.Context(A) as ctx:
            alone.append(_solve(ctx, f, g, False))

    def work(i):
        with P.Context(probs[i][0]) as ctx:
            for _ in range(8):
                got[i].append(_solve(ctx, *fg[i], False))
    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for i in range(2):
        assert len(got[i]) == 8
        for r in got[i]:
            for a, b in zip(r, alone[i]):
                np.testing.assert_array_equal(a, b)
