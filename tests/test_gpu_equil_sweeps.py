"""A Sinkhorn-Knopp sweep reads A once where a workgroup holds a row's columns in
registers: up to 6144 columns in float32, 3072 in float64, in steps of 1024 and
512.  Either side of each step, rows that do not fill the last workgroup, and
the first sizes past the range, against the float64 oracle: D and E to 1e-10
relative (ten sweeps of float64 sums in another order; about 100 roundings of
1e-16 each, grown at most a thousandfold)."""
import numpy as np
import pytest

from oracle import pogs_oracle as O
from paper_1503_08366_amd import pogs as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,dt", [
    (1, 1, np.float64), (5, 511, np.float64), (2049, 513, np.float64), (203, 1025, np.float64), (97, 1537, np.float64),
    (50, 2049, np.float64), (4101, 3072, np.float64), (70, 3073, np.float64),
    (3, 4096, np.float32), (1023, 4097, np.float32), (2051, 6144, np.float32), (70, 6145, np.float32)])
def test_sweeps_match_oracle(m, n, dt):
    rng = np.random.default_rng(m * 7 + n)
    A = (rng.normal(size=(m, n)) * (rng.random((m, n)) < 0.7)).astype(dt)
    with P.Context(A, P.default_params(projection="cgls")) as ctx:
        D, E = ctx.scaling()
    Dr, Er = O.equilibrate(A.astype(np.float64), float(np.finfo(dt).eps), 10)
    np.testing.assert_allclose(D, Dr, rtol=1e-10)
    np.testing.assert_allclose(E, Er, rtol=1e-10)
