"""Which sparse float32 matrices are kept in pieces: by size on both sides of each
limit (uniform rows), and by the rows' lengths.  A row of a piece is added up by
one lane, so matrices with many entries a row, rows sorted by length, or frequent
columns side by side ran up to 37 times slower in pieces than on the plain
passes (CG step 730 -> 26996 us), and have to stay with those; a CG step of a
matrix that is kept in pieces may not take much longer than on the plain passes."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd.workloads import Fn

pytestmark = pytest.mark.gpu


def _csr(cols, lens, n, seed):
    ptr = np.concatenate([[0], np.cumsum(lens)])
    vals = np.random.default_rng(seed).normal(size=len(cols)).astype(np.float32)
    return sp.csr_matrix((vals, cols.astype(np.int32), ptr), shape=(len(lens), n))


def _uniform(m, n, nnz):
    lens = np.full(m, nnz // m)
    lens[:nnz - lens.sum()] += 1
    return _csr(np.random.default_rng(m).integers(0, n, nnz), lens, n, 1)


def _zipf(m, n, k, shift, mixed):
    """Column frequencies 1 / (rank + shift), frequent ones first or in random order."""
    rng = np.random.default_rng(2)
    c = (shift * ((n + shift) / shift) ** rng.random(m * k) - shift).astype(np.int64).clip(0, n - 1)
    if mixed:
        c = rng.permutation(n)[c]
    return _csr(c, np.full(m, k), n, 3)


def _rows_by_length(m, n, k, shift):
    w = 1.0 / (np.arange(m) + shift)
    lens = np.maximum(1, (w / w.sum() * m * k).astype(np.int64)).clip(0, n)
    return _csr(np.random.default_rng(4).integers(0, n, lens.sum()), lens, n, 5)


def _pieces(A, **kw):
    with P.SparseContext(A, P.default_params(**kw)) as ctx:
        return ctx.route().sparse_pieces


@pytest.mark.parametrize("m,n,nnz,pieces", [
    (98304, 12288, 1 << 20, 1), (98303, 12288, 1 << 20, 0), (98304, 12287, 1 << 20, 0), (98304, 12288, (1 << 20) - 1, 0),
    (2100000, 12289, 2100000, 1), (150000, 64256, 300000 * 4, 1), (600000, 64257, 600000 * 3 - 1, 0)])
def test_size_limits(m, n, nnz, pieces):
    A = _uniform(m, n, nnz)
    assert _pieces(A) == pieces
    assert _pieces(A, sparse_segment=16384) == 0
    assert _pieces(A.astype(np.float64)) == 0


@pytest.mark.parametrize("name,pieces", [
    ("uniform-15", 1), ("uniform-100", 0), ("zipf-sorted", 0), ("zipf-mild-mixed", 1), ("rows-by-length", 0),
    ("zipf-past-16-bits", 0), ("bias", 1)])
def test_rows_lengths_decide_and_no_step_is_slower(name, pieces):
    m, n = 300000, 30000
    if name == "uniform-15":
        A = _uniform(m, n, 15 * m)
    elif name == "uniform-100":
        A = _uniform(100000, 20000, 100 * 100000)
    elif name == "zipf-sorted":
        A = _zipf(m, n, 15, 100, False)
    elif name == "zipf-mild-mixed":
        A = _zipf(m, n, 15, 10000, True)
    elif name == "rows-by-length":
        A = _rows_by_length(m, n, 15, 1000)
    elif name == "zipf-past-16-bits":
        A = _zipf(m, n, 15, 3, False)
    else:
        A = _uniform(m, n, 9 * m)
        A.indices[A.indptr[:-1]] = 0  # every row's first entry
    f, g = Fn("square", A.shape[0], b=1.0), Fn("abs", A.shape[1], c=0.1)
    us = {}
    for seg in (0, A.shape[0]):
        prm = P.default_params(max_iter=2, sparse_segment=seg)
        with P.SparseContext(A, prm) as ctx:
            assert ctx.route().sparse_pieces == (pieces if seg == 0 else 0)
            ctx.solve(f, g, prm)
            us[seg] = min(ctx.profile_iteration(10)["cg_step"] for _ in range(3)) * 1e3
    assert us[0] < 1.2 * us[A.shape[0]] + 5.0, us
