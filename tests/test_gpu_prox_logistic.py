"""The logistic prox over its range of curvatures: Newton steps end the loop at
rho = 100, saturated elements bisect at rho = 0.05, and the arguments reach both
tails.  Same bars as the other base functions: float64 relative 1e-12, float32
|gpu - ref| <= 1e-5 max(1, |ref|) on the same rounded inputs."""
import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("rho", [0.05, 1.0, 100.0])
def test_logistic_prox_over_curvatures(rho, dt):
    rng = np.random.default_rng(5)
    v = np.concatenate([np.linspace(-40.0, 40.0, 801), rng.normal(0, 2, 1000), [0.0]]).astype(dt)
    d = -(rng.random(v.size) < 0.5).astype(np.float64)
    F = W.Fn("logistic", v.size, d=d)
    got = P.pogs_prox(F, v, rho).astype(np.float64)
    ref = O.prox_param(F, v.astype(np.float64), float(dt(rho)))
    if dt == np.float64:
        np.testing.assert_allclose(got, ref, rtol=1e-12, atol=1e-12)
    else:
        assert (np.abs(got - ref) / np.maximum(1.0, np.abs(ref))).max() <= 1e-5
