"""The CGLS passes that read A once, at the edges of their kernels: one row per
wave and fewer rows than waves, the row lengths where a lane's pieces grow (256,
512, 1024 entries), rows shared by four waves (1025 to 2048 entries) from the
first row count that takes them and the last that does not, ragged groups of rows,
and a direct context (larger partial sums than its own passes) solving by CGLS.

A fixed number of ADMM iterations, so the oracle does the same work: float32
rounding of 8 iterations of at most 10 CG steps each (a few roundings per step,
contracting towards the projection), bounded by 5e-5 relative to the vector.
The step counts are not compared: at this tolerance the float32 normal residual
stalls above the threshold that float64 reaches (9001 x 256: 58 steps against 52,
with one pass or two)."""
import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu
ITERS = 8


@pytest.mark.parametrize("m,n,setup", [
    (5, 3, "cgls"), (33, 20, "cgls"), (9001, 256, "cgls"), (8200, 257, "cgls"), (1200, 513, "direct"),
    (1100, 1024, "cgls"), (2559, 1030, "cgls"), (2561, 1025, "cgls"), (2700, 2048, "direct"), (4001, 1500, "cgls"),
])
def test_cgls_one_pass_matches_oracle(m, n, setup):
    prob = W.lasso(m, n, seed=m + n)
    prm = P.default_params(eps_abs=1e-6, eps_rel=1e-6, max_iter=ITERS, projection="cgls")
    with P.Context(prob.A, P.default_params(projection=setup)) as ctx:
        r = ctx.solve(prob.f, prob.g, prm)
    ref = O.solve(prob.A.astype(np.float64), prob.f, prob.g,
                  O.Params(eps_abs=1e-6, eps_rel=1e-6, max_iter=ITERS, projection="cgls",
                           eps_cmp=float(np.finfo(np.float32).eps)))
    assert r.iters == ref.iters
    assert r.cg_steps > 0
    for name in ("x", "y", "nu"):
        got, want = getattr(r, name).astype(np.float64), getattr(ref, name)
        assert np.linalg.norm(got - want) <= 5e-5 * max(np.linalg.norm(want), 1e-3), name
