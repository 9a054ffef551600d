"""The steps of a grouped iteration pick a body by each problem's shape (tall
or wide, 16 or 64 lanes per row of A and of the solve).  Every combination in
one group, at the edges of the row tiles, against the problem alone (the same
bits: its arithmetic does not depend on its group) and against the FP64 oracle
(objective to 1e-3 of its size, the tolerance of the stop test)."""
import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu
FLT_EPS = float(np.finfo(np.float32).eps)
SHAPES = [(65, 64), (705, 448), (545, 513), (64, 65), (63, 449), (17, 513), (520, 577), (1, 70), (70, 1)]


@pytest.fixture(scope="module")
def mixed():
    probs = [W.lasso(m, n, 40 + i) for i, (m, n) in enumerate(SHAPES)]
    return probs, P.pogs_solve_batch(probs)


@pytest.mark.parametrize("i", range(len(SHAPES)), ids=["%dx%d" % s for s in SHAPES])
def test_each_body_in_a_mixed_group(mixed, i):
    prob, r = mixed[0][i], mixed[1][i]
    alone = P.pogs_solve_batch([prob])[0]
    assert alone.iters == r.iters
    for k in ("x", "y", "mu", "nu"):
        np.testing.assert_array_equal(getattr(alone, k), getattr(r, k))
    ref = O.solve(prob.A.astype(np.float64), prob.f, prob.g,
                  O.Params(eps_abs=prob.eps_abs, eps_rel=prob.eps_rel, max_iter=prob.max_iter, eps_cmp=FLT_EPS))
    if ref.converged:
        assert abs(r.optval - ref.optval) <= 1e-3 * max(abs(ref.optval), 1.0)
