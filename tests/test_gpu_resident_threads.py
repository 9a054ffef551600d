"""More threads than the process has hardware queues, each solving on a context
and stream of its own: every solve has the bits of a solve alone, and together
they take no longer than with one launch per step."""
import threading
import time

import numpy as np
import pytest

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu
THREADS, SOLVES = 8, 12


def _run(p, polls):
    out, errors = [], []
    bar = threading.Barrier(THREADS + 1)

    def work():
        try:
            with P.Context(p.A) as ctx:
                ctx.set_resident_wait(polls)
                ctx.solve(p.f, p.g)
                bar.wait(timeout=60)
                rs = [ctx.solve(p.f, p.g) for _ in range(SOLVES)]
                bar.wait(timeout=60)
                assert ctx.route().resident_give_ups == 0 and ctx.route().resident_last == int(polls > 0)
                out.extend(rs)
        except Exception as e:  # reported by the main thread
            errors.append(e)
            bar.abort()

    threads = [threading.Thread(target=work) for _ in range(THREADS)]
    for t in threads:
        t.start()
    bar.wait(timeout=60)
    t0 = time.perf_counter()
    bar.wait(timeout=60)
    dt = time.perf_counter() - t0
    for t in threads:
        t.join()
    assert not errors, errors
    return dt, out


@pytest.mark.parametrize("kind,m,n,dt", [("lasso", 3000, 700, np.float64), ("logistic", 1999, 503, np.float32)])
def test_many_threads(kind, m, n, dt):
    p = getattr(W, kind)(m, n, seed=3, dtype=dt)
    with P.Context(p.A) as ctx:
        alone = ctx.solve(p.f, p.g)
    resident, rs = _run(p, P.POGS_RESIDENT_WAIT)
    for r in rs:
        assert r.iters == alone.iters
        for k in ("x", "y", "mu", "nu"):
            np.testing.assert_array_equal(getattr(r, k), getattr(alone, k))
    steps, _ = _run(p, -1)
    assert resident < 1.1 * steps
