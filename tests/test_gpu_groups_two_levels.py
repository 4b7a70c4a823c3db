"""Plane groups on a hierarchy of two levels, whose coarsest level is the bottom
kernel's first: each group's streams touch that group's planes alone, so the
iterates are bitwise those of one stream."""
import pytest
import torch

import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


@pytest.mark.parametrize("shape", [(9, 3, 18), (9, 16, 18), (11, 7, 15)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("options", [{}, {"fmg": 1}, {"masks": 1}, {"bottom": 0, "groups": 1}], ids=str)
def test_groups_stay_with_their_planes(P, shape, options):
    p = W.SMALL.with_sizes(*shape)
    say("groups on two levels", p.shape, options)
    rho = dev(W.blob_charge(p, 7))
    one = P.Plan.for_problem(p, direct=0, merge=0, max_cycles=6, **{**options, "groups": 1, "bottom": 1})
    assert one.info()["levels"] == 2 and one.info()["bottom_level"] == 1
    phi, st = one.solve(rho, tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
    a = host(phi).copy()
    plan = P.Plan.for_problem(p, direct=0, merge=0, max_cycles=6, **{"groups": 3, **options})
    for _ in range(8):
        phi = torch.full_like(rho, float("nan"))
        phi, sb = plan.solve(rho, tol=1e-30, phi=phi, allow=(P.OK, P.NOT_CONVERGED))
        assert (host(phi) == a).all()
        assert sb["cycles"] == st["cycles"]
