"""Equilibration of tall narrow float64 matrices (two passes over A per sweep:
rows of fewer than 224 entries, more than 6144 of them) on both sides of the
rule, and where the number of workgroups of the one-pass sweep changes, against
the float64 oracle (1e-10 relative: ten sweeps of float64 sums in another order,
about 100 roundings of 1e-16 each, grown at most a thousandfold).  Every entry of
D and E is finite and positive, so that none can match by being infinite on both
sides; the smallest matrix has a nonzero entry."""
import time

import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P

pytestmark = pytest.mark.gpu
NO_FACTOR = dict(projection="cgls")


@pytest.mark.parametrize("m,n,dt", [
    (1, 1, np.float64), (1, 1, np.float32), (6144, 223, np.float64), (6145, 223, np.float64), (6145, 224, np.float64),
    (16384, 225, np.float64), (16385, 225, np.float64), (16385, 512, np.float64), (30001, 3, np.float64),
    (30001, 64, np.float32)])
def test_scaling_matches_oracle(m, n, dt):
    rng = np.random.default_rng(m + n)
    A = rng.normal(size=(m, n))
    A[rng.random((m, n)) < 0.2] = 0.0
    A[0, 0] = 1.5
    A = A.astype(dt)
    with P.Context(A, P.default_params(**NO_FACTOR)) as ctx:
        D, E = ctx.scaling()
    Dr, Er = O.equilibrate(A.astype(np.float64), float(np.finfo(dt).eps), 10)
    for got, want in ((D, Dr), (E, Er)):
        assert np.isfinite(got).all() and np.isfinite(want).all() and (got > 0).all()
        np.testing.assert_allclose(got, want, rtol=1e-10)


@pytest.mark.parametrize("m,n,ms", [(400000, 50, 1.7), (1000000, 64, 4.5)])
def test_setup_time_of_narrow_matrices(m, n, ms):
    """0.9 and 2.3 ms; with one pass per sweep 2.8 and 7.5."""
    import torch
    A = torch.randn(m, n, device="cuda", dtype=torch.float64)
    best = 1e9
    for _ in range(10):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        with P.Context(A, P.default_params(autotune=0, **NO_FACTOR)):
            best = min(best, time.perf_counter() - t0)
    assert best * 1e3 < ms
