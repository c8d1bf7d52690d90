"""A Gaussian embedding that a context evaluates instead of storing it (over
4 GiB), in the extension's own kernel, which sketches w and the pending column
together: d = 1000, whose 500 pairs leave lanes of the last wave without one.

Bars: S = Omega U is a sum of n FP64 products per entry, compared in norm at
1e-12; a stored column is off by the unit roundoff of its storage, so the
sketched basis is orthonormal to a small multiple of that (five columns)."""
import numpy as np
import pytest

import paper_2508_05400_amd as P
from workloads import convdiff2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,eps", [("fp64", 2.0**-53), ("fp32+fx16", 2.0**-39), ("fp32", 2.0**-24),
                                      ("bf16", 2.0**-9)])
def test_embedding_over_4_gib(lib, cuda, prec, eps):
    A = convdiff2d(735, (2.0, 1.0))
    k, m, d, seed = 2, 4, 1000, 9
    assert A.n * (d // 2) * 16 > 1 << 32
    ctx = P.rks_create(A.row_ptr, A.col, A.val, A.n, k, m, d, "LM", 1e-10,
                       P.rks_opts_default(sketch_kind="gauss", sketch_seed=seed, start_seed=1, precision=prec))
    try:
        P.rks_arnoldi(ctx)
        S, U = np.zeros((d, m + 1), order="F"), np.zeros((A.n, m + 1), order="F")
        assert P.rks_get_state(ctx, None, S, U) == m + 1
    finally:
        P.rks_destroy(ctx)
    z = cuda.empty(d, dtype=cuda.float64, device="cuda")
    for t in range(m + 1):
        P.rks_sketch_noalloc(A.n, d, "gauss", 8, seed, cuda.from_numpy(U[:, t].copy()).cuda(), z)
        cuda.cuda.synchronize()
        assert np.linalg.norm(z.cpu().numpy() - S[:, t]) < 1e-12, t
    assert np.linalg.norm(S.T @ S - np.eye(m + 1)) < 20 * (m + 1) * eps + 1e-12
