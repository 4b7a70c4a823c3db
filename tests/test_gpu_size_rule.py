"""The size rule of precision 32 as the header states it, options included."""
import pytest

import workloads as W
from gpu_util import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


@pytest.mark.parametrize("option,value,most", [("prefetch", 1, 587), ("prefetch", 3, 447), ("chunk_rows", 256, 483),
                                               ("chunk_rows", 512, 345)])
def test_precision_32(P, option, value, most):
    for nr in (most, most + 1):
        p = W.SMALL.with_sizes(nr, 4, 513)
        say("size rule", p.shape, option, value)
        plan = P.Plan.for_problem(p, precision=32, max_cycles=2)
        rho = dev(W.blob_charge(p, 7))
        plan.set_option(option, value)
        if nr == most:
            plan.solve(rho, tol=1e-30, allow=(P.NOT_CONVERGED,))
        else:
            with pytest.raises(P.CylPoissonError, match=f"size rule.*{option}.* {nr} radial nodes"):
                plan.solve(rho, tol=1e-30, allow=(P.NOT_CONVERGED,))
