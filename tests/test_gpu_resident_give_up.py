"""Resident solves whose workgroups give up waiting for each other, and the
rule that takes the route.  A wait bound of zero polls makes every workgroup end
at its first wait; the solve then starts over with one launch per step, and has
to return the bits of a context that runs so from the start (both run the same
launches on the same state, so there is no tolerance), cold and warm-started,
host and device outputs.  Against the FP64 oracle: 30 iterations of constant
rho, 3e-5 in float32 and 1e-11 in float64 (the tolerances that the resident
launches are held to; the launches per step form the same sums in float64)."""
import ctypes as C

import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu
KEYS = ("x", "y", "mu", "nu")
DEFAULT_POLLS = 1 << 20


@pytest.fixture(autouse=True)
def _no_pause_left():
    """A give-up keeps contexts from trying for a while; a solve with a bound of
    its own that gets through ends that."""
    yield
    p = W.lasso(64, 32, seed=1)
    with P.Context(p.A) as ctx:
        ctx.set_resident_wait(DEFAULT_POLLS)
        ctx.solve(p.f, p.g)
        assert ctx.route().resident_last == 1


def _bits(a, b):
    assert a.iters == b.iters and a.status == b.status
    for k in KEYS:
        u, v = getattr(a, k), getattr(b, k)
        if not isinstance(u, np.ndarray):
            u, v = u.cpu().numpy(), v.cpu().numpy()
        np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("m,n,dt", [(1, 1, np.float32), (900, 300, np.float32), (300, 900, np.float32),
                                    (700, 300, np.float64), (100, 400, np.float64)])
def test_given_up_solve_is_the_launch_per_step_solve(m, n, dt):
    p = W.lasso(m, n, seed=m + n, dtype=dt)
    prm = P.default_params(eps_abs=0.0, eps_rel=0.0, max_iter=30, chunk_iters=6)
    ref = O.solve(p.A.astype(np.float64), p.f, p.g,
                  O.Params(eps_abs=0.0, eps_rel=0.0, max_iter=30, eps_cmp=float(np.finfo(dt).eps)))
    with P.Context(p.A) as ctx, P.Context(p.A) as steps:
        steps.set_resident_wait(-1)
        ctx.set_resident_wait(0)
        for kw in ({}, {"device_out": True}, {"x0": ref.x, "nu0": ref.nu}, {"nu0": ref.nu},
                   {"x0": ref.x, "nu0": ref.nu, "device_out": True}):
            a, b = ctx.solve(p.f, p.g, prm, **kw), steps.solve(p.f, p.g, prm, **kw)
            _bits(a, b)
            if not kw:
                tol = 3e-5 if dt == np.float32 else 1e-11
                for k in ("x", "y", "nu"):
                    want = getattr(ref, k)
                    assert np.linalg.norm(getattr(a, k) - want) <= tol * max(np.linalg.norm(want), 1e-3), k
        r, s = ctx.route(), steps.route()
        assert (r.resident_last, r.resident_give_ups) == (0, 5) and r.resident_workgroups > 0
        assert (s.resident_last, s.resident_give_ups) == (0, 0) and s.resident_workgroups > 0


def test_solves_after_a_give_up_are_resident_again():
    """A give-up costs its own solve only: with the bound back the same
    context's next solve is resident, with the bits of a fresh context."""
    p = W.lasso(900, 300, seed=5)
    with P.Context(p.A) as fresh:
        want = fresh.solve(p.f, p.g)
        assert fresh.route().resident_last == 1
    with P.Context(p.A) as ctx:
        for _ in range(3):
            ctx.set_resident_wait(0)
            assert ctx.solve(p.f, p.g).converged and ctx.route().resident_last == 0
            ctx.set_resident_wait(DEFAULT_POLLS)
            _bits(ctx.solve(p.f, p.g), want)
            assert ctx.route().resident_last == 1
        assert ctx.route().resident_give_ups == 3


@pytest.mark.parametrize("m,n,dt,taken", [
    (1, 1, np.float32, True), (40960, 100, np.float32, True), (40961, 100, np.float32, False),
    (1024, 1024, np.float32, True), (1025, 1025, np.float32, False), (1025, 1025, np.float64, False),
    (1100, 1024, np.float64, True), (100, 40960, np.float32, True)])
def test_shapes_that_are_resident(m, n, dt, taken):
    p = W.lasso(m, n, seed=7, dtype=dt)
    with P.Context(p.A) as ctx:
        ctx.solve(p.f, p.g, P.default_params(max_iter=4))
        r = ctx.route()
        assert (r.resident_workgroups > 0) == taken and r.resident_last == int(taken) and r.resident_give_ups == 0
        for prm in (P.default_params(max_iter=4, stop_rule="gap"), P.default_params(max_iter=4, projection="cgls")):
            ctx.solve(p.f, p.g, prm)
            assert ctx.route().resident_last == 0
    with P.Context(p.A, P.default_params(projection="cgls")) as ctx:
        assert ctx.route().resident_workgroups == 0


def test_rejects_null():
    lib = P.load()
    assert lib.pogs_get_route(None, C.byref(P.pogs_route())) == P.POGS_EINVAL
    assert lib.pogs_set_resident_wait(None, 0) == P.POGS_EINVAL


@pytest.mark.parametrize("m,n,dt", [(8000, 1000, np.float32), (300, 900, np.float64)])
def test_profile_after_a_give_up_times_launches_per_step(m, n, dt):
    """A profile whose resident launches gave up reports the iteration that ran
    instead: five launches, none under 2 us, and not the launches that returned."""
    p = W.lasso(m, n, seed=9, dtype=dt)
    with P.Context(p.A) as ctx:
        want = ctx.solve(p.f, p.g)
        ctx.set_resident_wait(-1)
        steps = min(ctx.profile_iteration(100)["iteration"] for _ in range(3))
        ctx.set_resident_wait(0)
        given_up = min(ctx.profile_iteration(100)["iteration"] for _ in range(3))
        assert ctx.route().resident_give_ups == 3
        assert given_up > 0.01 and 0.7 * steps < given_up < 1.4 * steps
        ctx.set_resident_wait(DEFAULT_POLLS)
        assert ctx.profile_iteration(100)["iteration"] < 0.9 * steps
        _bits(ctx.solve(p.f, p.g), want)
        assert ctx.route().resident_last == 1 and ctx.route().resident_give_ups == 3
