"""A context's stored Gaussian Omega and the evaluated one give the same sums
to the bit: rks_sketch and rks_spmv_sketch (stored) against rks_sketch_noalloc
(evaluated), at sizes around the 64-entry groups of rows, the four waves of a
block and odd sketch sizes."""
import numpy as np
import pytest

import paper_2508_05400_amd as P
from workloads import convdiff2d, start_vector_normal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d", [(12, 21), (16, 33), (91, 127), (91, 130), (181, 64), (200, 257)])
def test_stored_omega_is_the_evaluated_one(lib, cuda, N, d):
    A = convdiff2d(N, (2.0, 1.0))
    ctx = P.rks_create(A.row_ptr, A.col, A.val, A.n, 2, 20, d, "LM", 1e-10,
                       P.rks_opts_default(sketch_kind="gauss", sketch_seed=N))
    try:
        x = cuda.from_numpy(start_vector_normal(A.n, d)).cuda()
        w, z1, z2, z3, z4 = (cuda.full((s,), float("nan"), dtype=cuda.float64, device="cuda")
                             for s in (A.n, d, d, d, d))
        P.rks_sketch(ctx, x, z1)
        P.rks_spmv_sketch(ctx, x, w, z2)
        P.rks_sketch_noalloc(A.n, d, "gauss", 8, N, x, z3)
        P.rks_sketch_noalloc(A.n, d, "gauss", 8, N, w, z4)
        cuda.cuda.synchronize()
        assert np.array_equal(z1.cpu().numpy(), z3.cpu().numpy())
        assert np.array_equal(z2.cpu().numpy(), z4.cpu().numpy())
    finally:
        P.rks_destroy(ctx)
