"""The prox of e^u for large arguments and small curvatures (the equilibration
scales arguments by 1 / D, so they reach hundreds in ordinary problems): against
a bisection in extended precision, and a problem that needs it against the
oracle.

Bars: the last Newton step and the value it comes from carry a few roundings of
max(1, |u|) (the sums e^u and r (u - z) cancel, and their difference is divided by
at least the larger one's slope): 1e-14 in float64, 1e-6 in float32 (__expf adds
its own 2 ulp + |u| / 16 of them).  The problem's objective as in the parity
tests, 1e-3 relative, and the iteration count within 2 of the oracle's."""
import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu
L = np.longdouble


def _exact(z, r):
    z, r = z.astype(L), L(r)
    lo = np.where(z <= 0, z - 2 * np.exp(np.minimum(z, 0)) / r - L(1e-15) * (1 + np.abs(z)),
                  np.minimum(np.log(r) - 100, -1))
    hi = z.copy()
    for _ in range(200):
        u = (lo + hi) / 2
        right = np.exp(u) + r * (u - z) > 0
        hi, lo = np.where(right, u, hi), np.where(right, lo, u)
    return (lo + hi) / 2


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("rho", [1e-8, 1e-4, 0.01, 1.0, 100.0, 1e4, 1e8])
def test_exp_prox_over_arguments(rho, dt):
    rng = np.random.default_rng(0)
    z = np.concatenate([rng.uniform(-20, 20, 2000), rng.uniform(0, 2, 1000), np.exp(rng.uniform(0, 9, 3000)),
                        [1.0, np.nextafter(1.0, 2.0), 80.0, 88.8, 700.0, 709.9]]).astype(dt)
    got = P.pogs_prox(W.Fn("exp", len(z)), z, float(dt(rho))).astype(L)
    want = _exact(z.astype(np.float64), float(dt(rho)))
    assert (np.abs(got - want) / np.maximum(1, np.abs(want))).max() <= (1e-6 if dt == np.float32 else 1e-14)


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("m,n", [(1000, 300), (100, 60)])
def test_exp_problem_matches_oracle(m, n, dt):
    rng = np.random.default_rng(0)
    A = rng.normal(size=(m, n)).astype(dt)
    f, g = W.Fn("exp", m, b=rng.normal(size=m) * 0.1), W.Fn("square", n, c=0.1)
    ref = O.solve(A.astype(np.float64), f, g, O.Params(max_iter=500, eps_cmp=float(np.finfo(dt).eps)))
    with P.Context(A) as ctx:
        for polls in (P.POGS_RESIDENT_WAIT, -1):
            ctx.set_resident_wait(polls)
            r = ctx.solve(f, g, P.default_params(max_iter=500))
            assert ref.converged and r.converged and abs(r.iters - ref.iters) <= 2
            assert abs(r.optval - ref.optval) <= 1e-3 * abs(ref.optval)


def test_exp_problem_in_a_batch_and_on_a_path():
    from types import SimpleNamespace
    rng = np.random.default_rng(0)
    m, n = 1000, 300
    A = rng.normal(size=(m, n)).astype(np.float32)
    f = W.Fn("exp", m, b=rng.normal(size=m) * 0.1)
    gs = [W.Fn("square", n, c=c) for c in (0.1, 1.0)]
    prm = P.default_params(max_iter=500)
    refs = [O.solve(A.astype(np.float64), f, g, O.Params(max_iter=500, eps_cmp=float(np.finfo(np.float32).eps))) for g in gs]
    batch = P.pogs_solve_batch([SimpleNamespace(A=A, f=f, g=g, m=m, n=n) for g in gs], prm)
    with P.Context(A) as ctx:
        path = ctx.solve_path([f, f], gs, prm)
    for rs in (batch, path):
        for r, ref in zip(rs, refs):
            assert ref.converged and r.converged and abs(r.iters - ref.iters) <= 2
            assert abs(r.optval - ref.optval) <= 1e-3 * abs(ref.optval)
