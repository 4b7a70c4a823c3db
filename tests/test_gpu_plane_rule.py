"""Which planes run all cycles between two checks in one launch: the rule on both
sides of each of its limits, and the two ways bitwise the same there (the same
node arithmetic, so the tolerance is zero)."""
import ctypes

import pytest

import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


def one_launch(P, plan) -> bool:
    """cp::plane_active of the plan: what every cycle loop asks."""
    f = P.library()._ZN2cp12plane_activeEPK15cylpoisson_plan
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_void_p]
    return bool(f(plan.handle))


# one column pair a thread, two, three (never); two with level 1 up to 32
# interior nodes each way (256 planes) and beyond (64 planes); a level 1 that one
# workgroup does not solve; LDS
RULE = [((33, 16, 33), True), ((33, 512, 33), True), ((18, 100, 129), True), ((65, 256, 65), True), ((65, 257, 65), False),
        ((65, 4, 65), True), ((66, 4, 63), True), ((66, 4, 68), False), ((35, 64, 120), True), ((35, 65, 120), False),
        ((72, 64, 56), True), ((72, 65, 56), False), ((35, 3, 122), True), ((35, 3, 123), False), ((9, 4, 300), False), ((129, 8, 129), False)]


@pytest.mark.parametrize("shape,expected", RULE, ids=lambda s: "x".join(map(str, s)) if isinstance(s, tuple) else str(s))
def test_rule(P, shape, expected):
    p = W.SMALL.with_sizes(*shape)
    say("plane rule", shape)
    rho = dev(W.blob_charge(p, 7))
    out = []
    for timing in (0, 1):  # the option "timing" takes the passes apart
        plan = P.Plan.for_problem(p, max_cycles=3, timing=timing)
        assert one_launch(P, plan) == (expected and not timing)
        phi, st = plan.solve(rho, tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
        assert st["cycles"] == 3
        out.append(host(phi).copy())
    assert (out[0] == out[1]).all()
    for off in ({"merge": 0}, {"direct": 0}, {"fused": 0}, {"nu1": 1}):
        assert not one_launch(P, P.Plan.for_problem(p, **off))
