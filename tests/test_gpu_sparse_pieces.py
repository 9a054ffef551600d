"""Large sparse float32 matrices are kept in pieces whose part of the vector
fits in LDS (at least 2^20 entries, 98304 rows and 12288 columns).  Against the
plain row passes, which a segment length in the parameters keeps (all outputs),
and a float64 context (x; nu of a row without entries is a difference that
float32 state cannot resolve on either route): 3 iterations of exactly 4 CG steps each (no tolerance stops them), at ragged tiles and
segments, with unsorted rows, repeated entries, empty rows and columns, a full
column and a long row (many times the 256 entries a wave takes at once).

Tolerance 3e-5 in the relative 2-norm: about 50 roundings of float32 state
(6e-8 each), grown at most tenfold by the steps between.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd.workloads import Fn

pytestmark = pytest.mark.gpu


def _matrix(m, n, per_row, kind):
    rng = np.random.default_rng(m + n)
    nnz = m * per_row
    ptr = np.arange(0, nnz + 1, per_row)
    cols = rng.integers(0, n, nnz)  # unsorted, some repeated within a row
    vals = rng.normal(size=nnz).astype(np.float32)
    A = sp.csr_matrix((vals, cols, ptr), shape=(m, n))
    if kind == "full":  # 6 full columns side by side: more entries in 64 rows of A^T and one segment than 16 bits count
        full = sp.csr_matrix(rng.normal(size=(m, 6)).astype(np.float32) * 0.1)
        A = sp.hstack([full, A.tocsc()[:, 6:]], format="csr").astype(np.float32)
    if kind == "gaps":  # empty rows (whole groups of 64) and columns, a full column, a long row
        A = A.tocoo()
        keep = ~((A.row >= 640) & (A.row < 900)) & (A.col != 11) & (A.row != m - 1)
        r = np.concatenate([A.row[keep], np.arange(m), np.full(n, 5)])
        c = np.concatenate([A.col[keep], np.full(m, 7), np.arange(n)])
        v = np.concatenate([A.data[keep], np.full(m, 0.01), rng.normal(size=n) * 0.1]).astype(np.float32)
        order = np.argsort(r, kind="stable")
        ptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=m))])
        A = sp.csr_matrix((v[order], c[order], ptr), shape=(m, n))
    return A


@pytest.mark.parametrize("m,n,per_row,kind", [
    (98304, 12288, 11, "plain"), (100003, 32129, 12, "plain"), (98305, 13001, 12, "gaps"), (98305, 13001, 12, "full"),
    (2100000, 12289, 1, "plain")])
def test_pieces_match_plain_passes(m, n, per_row, kind):
    A = _matrix(m, n, per_row, kind)
    rng = np.random.default_rng(1)
    f, g = Fn("square", m, b=rng.normal(size=m)), Fn("abs", n, c=0.1)
    out = []
    for dt, seg in ((np.float32, 0), (np.float32, 16384), (np.float64, 0)):
        pr = P.default_params(eps_abs=0.0, eps_rel=0.0, max_iter=3, cg_max_iter=4, cg_tol=1e-30,
                              eps_cmp=float(np.finfo(np.float32).eps), sparse_segment=seg)
        same = sp.csr_matrix((A.data.astype(dt), A.indices, A.indptr), shape=A.shape)  # astype merges repeated entries
        with P.SparseContext(same, pr) as ctx:
            out.append(ctx.solve(f, g, pr))
    a, plain, b = out
    assert a.iters == plain.iters == b.iters and a.cg_steps == plain.cg_steps == b.cg_steps == 12
    pairs = [(getattr(a, k), getattr(plain, k)) for k in ("x", "y", "mu", "nu")] + [(a.x, b.x)]
    for u, v in pairs:
        u, v = u.astype(np.float64), v.astype(np.float64)
        assert np.linalg.norm(u - v) <= 3e-5 * np.linalg.norm(v)
