"""The generated start vector is rounded to FP64 before it is rounded to the
basis precision: a decomposition from the seed equals, to the bit, the one from
the same vector passed in.  (Splitting the unrounded product of the Box-Muller
pair into the pair basis moves about one entry in 2^15 by a pair step.)"""
import numpy as np
import pytest

import paper_2508_05400_amd as P
from oracle.philox import TAG_START, _key, _split, philox4x32_10, uniform01
from workloads import convdiff2d

pytestmark = pytest.mark.gpu


def box_muller_on_device(torch, n, seed):
    lo, hi = _split(np.arange(n, dtype=np.uint64))
    w = philox4x32_10(lo, hi, 0, TAG_START, *_key(seed))
    u1, u2 = (torch.from_numpy(uniform01(w[i], w[i + 1])).cuda() for i in (0, 2))
    return torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * np.pi * u2)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16", "fp32+fx16"])
def test_generated_start_is_the_given_one(lib, cuda, prec):
    A = convdiff2d(512, (2.0, 1.0))
    k, m, d, seed = 2, 4, 16, 3
    states = []
    for u0 in (None, box_muller_on_device(cuda, A.n, seed)):
        ctx = P.rks_create(A.row_ptr, A.col, A.val, A.n, k, m, d, "LM", 1e-10,
                           P.rks_opts_default(sketch_seed=1, start_seed=seed, precision=prec))
        try:
            P.rks_arnoldi(ctx, u0)
            U = np.zeros((A.n, m + 1), order="F")
            P.rks_get_state(ctx, None, None, U)
            states.append(U)
        finally:
            P.rks_destroy(ctx)
    assert int((states[0][:, 0] != states[1][:, 0]).sum()) == 0
    assert np.array_equal(states[0], states[1])
