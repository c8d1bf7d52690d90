"""The per-kernel times of a Gaussian context (rks_opts.profile) hold the pass
over Omega: on 160,000 rows with d = 600 it reads 768 MB, some 150 us of a step
of 200, so without it the kernels make up less than half of the step.  Bar:
0.7 of the step timed as a whole, which adds launch gaps and its events, some
20 us."""
import pytest

import paper_2508_05400_amd as P
from workloads import convdiff2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("omega", ["auto", "evaluate"])
def test_kernel_times_hold_the_sketch(lib, cuda, omega):
    A = convdiff2d(400, (50.0, 30.0))
    with P.Solver.from_csr(A, k=6, m=24, d=600, which="SR", tol=1e-10, sketch_kind="gauss", sketch_seed=2,
                           start_seed=1, max_restarts=3, keep=-1, profile=1, omega=omega) as s:
        s.solve()
        st = s.stats.as_dict()
    per = [st[q] / st["n_timed_steps"] for q in ("t_spmv", "t_reduce", "t_update")]
    whole = st["t_step"] / st["n_timed_whole"]
    assert 0.7 * whole <= sum(per) <= 1.1 * whole, (per, whole)
