"""What one solve's give-up means for the next ones on the same GPU: for a while
no context tries resident launches (each try would wait again), then they do."""
import time

import pytest

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu


def _give_up(ctx, p):
    ctx.set_resident_wait(0)
    ctx.solve(p.f, p.g)
    ctx.set_resident_wait(P.POGS_RESIDENT_WAIT)


def test_contexts_pause_after_a_give_up_and_try_again():
    p = W.lasso(500, 200, seed=8)
    with P.Context(p.A) as kept, P.Context(p.A) as other:
        try:
            _give_up(kept, p)
            _give_up(kept, p)  # in a row: at least 0.2 s
            t0 = time.perf_counter()
            kept.solve(p.f, p.g)
            other.solve(p.f, p.g)
            with P.Context(p.A) as new:
                new.solve(p.f, p.g)
                assert time.perf_counter() - t0 < 0.2
                assert [c.route().resident_last for c in (kept, other, new)] == [0, 0, 0]
                assert [c.route().resident_give_ups for c in (kept, other, new)] == [2, 0, 0]
                # a bound of its own makes a context try all the same
                new.set_resident_wait(1 << 20)
                new.solve(p.f, p.g)
                assert new.route().resident_last == 1
            # and its getting through ends the pause
            kept.solve(p.f, p.g)
            assert kept.route().resident_last == 1
            _give_up(kept, p)
            time.sleep(0.15)  # the first of a row: 0.1 s
            kept.solve(p.f, p.g)
            other.solve(p.f, p.g)
            assert (kept.route().resident_last, other.route().resident_last) == (1, 1)
        finally:  # leave no pause behind
            other.set_resident_wait(1 << 20)
            other.solve(p.f, p.g)
