"""A Gaussian embedding over FP32 and BF16 bases (w in FP32, the pending column
in the basis type) against the oracle with the same storage rounding.  Bars as
for the sparse embedding in test_gpu_parity.py: the identities of the GPU's own
output, and B and the stored columns over the first six steps, where the two
sides differ by the order of the binary32 product's sums."""
import numpy as np
import pytest
import scipy.sparse as sp

import paper_2508_05400_amd as P
from oracle.rks import RKSOracle
from oracle.sketch import sketch_matrix
from workloads import convdiff2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("omega", ["auto", "evaluate"])
@pytest.mark.parametrize("prec,u_low,b_bar", [("fp32", 2.0**-24, 1e-6), ("bf16", 2.0**-8, 3e-4)])
def test_extension_matches_oracle(lib, cuda, prec, u_low, b_bar, omega):
    A = convdiff2d(45, (20.0, 10.0))
    k, m, d = 8, 30, 90
    ctx = P.rks_create(A.row_ptr, A.col, A.val, A.n, k, m, d, "LR", 1e-10,
                       P.rks_opts_default(sketch_kind="gauss", sketch_seed=2, precision=prec, omega=omega))
    try:
        P.rks_arnoldi(ctx, None)
        B, S, U = (np.zeros(s, order="F") for s in ((m + 1, m), (d, m + 1), (A.n, m + 1)))
        P.rks_get_state(ctx, B, S, U)
    finally:
        P.rks_destroy(ctx)
    OU = np.asarray(sketch_matrix(A.n, d, "gauss", 2) @ U)
    assert np.linalg.norm(OU - S) < 1e-12
    assert np.abs(np.diag(OU.T @ OU) - 1).max() < 1e-13
    Sp = sp.csr_matrix((A.val, A.col, A.row_ptr), shape=(A.n, A.n))
    nA = abs(Sp).sum(axis=0).max()
    assert np.linalg.norm(Sp @ U[:, :m] - U @ B) < 50 * u_low * nA * np.linalg.norm(U[:, :m])
    o = RKSOracle(A, k, m, d, "LR", 1e-10, sketch="gauss", sketch_seed=2, start_seed=1, store=prec)
    o.start(None)
    o.extend()
    assert np.abs(B[:7, :6] - o.B[:7, :6]).max() <= b_bar * nA
    if prec == "fp32":
        for j in range(7):
            assert np.linalg.norm(U[:, j] - o.U[:, j]) <= 16 * u_low * np.linalg.norm(o.U[:, j])
