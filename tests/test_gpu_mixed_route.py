"""Which inner cycles of the mixed-precision solve run merged: the launches counted
by the option "timing"."""
import pytest

import workloads as W
from gpu_util import dev, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


@pytest.mark.parametrize("options,merged", [({}, 3), ({"inner_cycles": 3}, 4), ({"inner_cycles": 1}, 0), ({"merge": 0}, 0),
                                            ({"groups": 2}, 0), ({"nu1": 3}, 0), ({"direct": 0}, 3)], ids=str)
def test_merged_passes_are_launched(P, options, merged):
    """Six inner cycles: one merged pass between each two of a refinement."""
    p = W.SMALL.with_sizes(129, 4, 131)
    say("mixed route", p.shape, options)
    plan = P.Plan.for_problem(p, precision=32, max_cycles=6, timing=1, **options)
    _, st = plan.solve(dev(W.blob_charge(p, 7)), tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
    assert st["cycles"] == 6
    assert st["kernel_launches"]["fine_merged"] == merged
