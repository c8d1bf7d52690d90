"""Residuals and norms of the Ritz vectors, formed for several columns at once,
against NumPy on the vectors the library returned: every SpMV layout, real
and complex pairs, group boundaries inside and between pairs, empty rows, rows
longer than one batch of loads, and a last row that is empty.

Bar: a row's product and the residual's two further terms are sums of at most
L + 3 FP64 terms, so ||r|| moves by at most (L + 3) u (||A||x||| + 2 |lam| ||x||)
and its own summation by n u ||r||, with L the longest row (u = 2^-53)."""
import numpy as np
import pytest
import scipy.sparse as sp

import paper_2508_05400_amd as P

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _matrix(n, seed, distinct):
    """Random pattern, a skew part for complex pairs, empty rows and one full-ish row."""
    rng = np.random.default_rng(seed)
    L = rng.integers(0, 9, size=n)
    L[[0, n // 2, n - 1]] = 0
    L[n // 3] = min(n - 1, 150)
    rows = np.repeat(np.arange(n), L)
    cols = np.concatenate([rng.choice(n, size=k, replace=False) for k in L if k])
    vals = rng.choice([-1.5, 0.25, 1.0], size=rows.size) if distinct else rng.standard_normal(rows.size)
    A = sp.csr_matrix((vals, (rows, cols)), shape=(n, n))
    A.sort_indices()
    return A


@pytest.mark.parametrize("layout", ["rows", "sliced", "column_blocks"])
@pytest.mark.parametrize("n,k,distinct", [(257, 9, True), (1031, 17, False), (64, 7, False), (5003, 33, True)])
def test_residuals_of_ritz_pairs(lib, cuda, layout, n, k, distinct):
    A = _matrix(n, n + k, distinct)
    m = min(2 * k + 6, n - 4)
    ctx = P.rks_create(A.indptr, A.indices, A.data, n, k, m, min(n, 2 * m + 3), "LM", 1e-10,
                       P.rks_opts_default(sketch_seed=3, max_restarts=1, spmv_layout=layout, keep=-1))
    try:
        P.rks_solve(ctx)
        ke = P.rks_num_pairs(ctx)
        re, im, res = np.empty(ke), np.empty(ke), np.empty(ke)
        X = cuda.empty((ke, n), dtype=cuda.float64, device="cuda")
        P.rks_eigpairs(ctx, re, im, X, res)
        X = X.cpu().numpy().T
    finally:
        P.rks_destroy(ctx)
    assert (im != 0).any()
    norm1 = abs(A).sum(0).max()
    longest = np.diff(A.indptr).max()
    i = 0
    while i < ke:
        pair = im[i] != 0 and i + 1 < ke
        x = X[:, i] + 1j * X[:, i + 1] if pair else X[:, i]
        lam = re[i] + 1j * im[i] if pair else re[i]
        assert abs(np.linalg.norm(x) - 1.0) <= (n + 8) * U
        r = np.linalg.norm(A @ x - lam * x) / norm1
        bar = (longest + 3) * U * (np.linalg.norm(abs(A) @ abs(x)) + 2 * abs(lam)) / norm1 + n * U * r
        assert abs(res[i] - r) <= 2 * bar
        if pair:
            assert res[i + 1] == res[i]
        i += 2 if pair else 1
