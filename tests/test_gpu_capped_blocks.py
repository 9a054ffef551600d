"""Above 262144 elements a side the CGLS prox step and the unscale step take
several elements per thread.  At the edge and past it: x against a float64
context after 3 iterations of exactly 4 CG steps (3e-5 in the relative 2-norm:
about 50 float32 roundings grown at most tenfold), and the objective against
its value at the returned float32 x and y (1e-6: their rounding, 6e-8, enters
each term at most twice)."""
import numpy as np
import pytest

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W
from paper_1503_08366_amd.workloads import Fn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [262144, 262145, 530001])
def test_prox_and_objective_past_the_cap(m):
    n = 700
    rng = np.random.default_rng(m)
    A = W.sparse_matrix(m, n, 2, rng, np.float32).tocsr()
    b = rng.normal(size=m)
    f, g = Fn("square", m, b=b), Fn("abs", n, c=0.3)
    out = []
    for dt in (np.float32, np.float64):
        pr = P.default_params(eps_abs=0.0, eps_rel=0.0, max_iter=3, cg_max_iter=4, cg_tol=1e-30,
                              eps_cmp=float(np.finfo(np.float32).eps))
        with P.SparseContext(A.astype(dt), pr) as ctx:
            out.append(ctx.solve(f, g, pr))
    a, e = out
    x = a.x.astype(np.float64)
    assert np.linalg.norm(x - e.x) <= 3e-5 * np.linalg.norm(e.x)
    obj = 0.5 * np.sum((a.y.astype(np.float64) - b) ** 2) + 0.3 * np.abs(x).sum()
    assert abs(a.optval - obj) <= 1e-6 * abs(obj)
