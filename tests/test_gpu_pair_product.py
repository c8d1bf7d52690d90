"""The pair basis at a restart: the column after the kept ones is u_{m+1}
scaled by 1 / beta, split from the product before its rounding to FP64.

The stored u_{m+1} follows from the returned (scaled and rounded) column as the
pair nearest to it times beta; a b - round(a b) is exact by Dekker's product."""
import numpy as np
import pytest

import paper_2508_05400_amd as P
from oracle.rks import fx16_pair
from workloads import convdiff2d

pytestmark = pytest.mark.gpu


def _halves(a):
    c = 134217729.0 * a
    hi = c - (c - a)
    return hi, a - hi


def test_scaled_column_is_split_from_the_product(lib, cuda):
    A = convdiff2d(512, (2.0, 1.0))
    k, m, d = 3, 12, 40
    opts = dict(sketch_seed=1, start_seed=3, precision="fp32+fx16", max_restarts=0, keep=0)
    B, U, V = np.zeros((m + 1, m), order="F"), *(np.zeros((A.n, m + 1), order="F") for _ in range(2))
    ctx = P.rks_create(A.row_ptr, A.col, A.val, A.n, k, m, d, "LM", 1e-10, P.rks_opts_default(**opts))
    try:
        P.rks_arnoldi(ctx)
        P.rks_get_state(ctx, B, None, U)
        P.rks_solve(ctx)  # the same extension, then one contraction
        ke = P.rks_get_state(ctx, None, None, V) - 1
    finally:
        P.rks_destroy(ctx)
    beta = B[m, m - 1]
    s = 1.0 / beta
    hi, q, step = fx16_pair(U[:, m] * beta)
    v = hi + q * step
    p = v * s
    assert np.array_equal(p, U[:, m])  # v is the stored column
    (vh, vl), (sh, sl) = _halves(v), _halves(s)
    e = ((vh * sh - p) + vh * sl + vl * sh) + vl * sl  # v s = p + e
    hi, q, step = fx16_pair(p)
    q1 = np.rint(((p - hi) + e) / step)
    assert np.array_equal(V[:, ke], hi + q1 * step)
    assert (q1 != q).any()  # splitting the rounded product would differ
