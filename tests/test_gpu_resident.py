"""The resident solve (a chunk of iterations per launch, workgroups exchanging
vectors in memory) at the edges of its kernels and of the rule that takes it:
one row or column, the last row that a number of rows per wave serves and the
next one, the row lengths where a lane's pieces grow, square, tall and wide, the
largest matrix it takes and the first one past it.

Against the FP64 oracle after a fixed number of iterations with a constant rho
(both sides run the same count).  The iteration is non-expansive, so the
difference grows at most linearly: 30 iterations times a few roundings, with
the K^-1 product as the largest, bounded by 3e-5 in float32 (30 x 16 x 6e-8) and
1e-11 in float64 (30 x 16 x 1.1e-16 is 5e-14; K^-1's own rounding adds cond(K) ~ 100)
relative to the vector."""
import threading

import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu
ITERS = 30


def _both(m, n, dt, problem="lasso"):
    prob = getattr(W, problem)(m, n, seed=m + 3 * n, dtype=dt)
    prm = P.default_params(eps_abs=0.0, eps_rel=0.0, max_iter=ITERS)
    with P.Context(prob.A, prm) as ctx:
        r = ctx.solve(prob.f, prob.g, prm)
    ref = O.solve(prob.A.astype(np.float64), prob.f, prob.g,
                  O.Params(eps_abs=0.0, eps_rel=0.0, max_iter=ITERS, eps_cmp=float(np.finfo(dt).eps)))
    return r, ref


@pytest.mark.parametrize("m,n,dt", [
    (1, 1, np.float32), (1, 9, np.float64), (9, 1, np.float32),
    (4096, 256, np.float32), (4097, 256, np.float32), (256, 4097, np.float32), (3000, 257, np.float32),
    (1023, 1024, np.float32), (1025, 1024, np.float32), (2048, 513, np.float32),
    (1300, 128, np.float64), (128, 4099, np.float64), (1030, 129, np.float64), (1025, 512, np.float64),
    (700, 769, np.float64), (1100, 1024, np.float64),
    (40960, 100, np.float32), (40961, 100, np.float32),
])
def test_resident_matches_oracle(m, n, dt):
    r, ref = _both(m, n, dt)
    assert r.iters == ref.iters == ITERS
    tol = 3e-5 if dt == np.float32 else 1e-11
    for name in ("x", "y", "nu"):
        got, want = getattr(r, name).astype(np.float64), getattr(ref, name)
        assert np.linalg.norm(got - want) <= tol * max(np.linalg.norm(want), 1e-3), name


@pytest.mark.parametrize("m,n,dt", [(900, 300, np.float32), (300, 2000, np.float64)])
def test_launch_length_and_company_change_no_bit(m, n, dt):
    """Launches of 2 or 64 iterations, with rho changing, and solves on other
    threads' streams at the same time give the same bits."""
    prob = W.lasso(m, n, seed=4, dtype=dt)

    def solve(chunk):
        with P.Context(prob.A) as ctx:
            r = ctx.solve(prob.f, prob.g, P.default_params(chunk_iters=chunk))
            again = ctx.solve(prob.f, prob.g, P.default_params(chunk_iters=chunk))
        np.testing.assert_array_equal(r.x, again.x)
        return r

    one = solve(20)
    assert one.converged
    got = {}
    threads = [threading.Thread(target=lambda c=c: got.__setitem__(c, solve(c))) for c in (2, 64, 6, 20)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for r in got.values():
        assert r.iters == one.iters
        for k in ("x", "y", "mu", "nu"):
            np.testing.assert_array_equal(getattr(r, k), getattr(one, k))
    assert len(got) == 4
