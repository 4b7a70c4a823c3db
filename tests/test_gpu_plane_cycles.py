"""Small planes' cycles in one launch, bitwise against the per-step kernels (the
same node arithmetic and the same exact solve, so the tolerance is zero)."""
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


# level 1 of up to 16, 32 and 64 interior nodes each way; one and two column
# pairs a thread, full and not; odd and even counts; one direction coarsened;
# the last shape the limit admits and the first beyond it
SHAPES = [(11, 3, 12), (33, 4, 33), (34, 5, 35), (33, 2, 34), (50, 3, 47), (65, 4, 65), (66, 4, 63), (35, 3, 120),
          (18, 4, 129), (129, 3, 18), (9, 4, 100), (64, 1, 34), (67, 4, 67)]


def solve(P, p, rho, **options):
    plan = P.Plan.for_problem(p, **options)
    phi = torch.zeros(p.shape, dtype=torch.float64, device="cuda")
    _, st = plan.solve(rho, phi=phi, tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
    return host(phi), st


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("options", [{}, {"fmg": 1}, {"nu1": 1, "nu2": 3}, {"nu1": 3, "nu2": 3}, {"graph": 1},
                                     {"warm_start": 1}, {"max_cycles": 1}], ids=str)
def test_cycles_in_one_launch(P, shape, options):
    p = W.SMALL.with_sizes(*shape)
    say("plane cycles", p.shape, options)
    rho = dev(W.blob_charge(p, 7))
    options = {"max_cycles": 5, **options}
    a, sa = solve(P, p, rho, **options)
    # the passes (the option "timing" takes them apart) and, from the same
    # start, the per-step kernels
    b, sb = solve(P, p, rho, timing=1, **{k: v for k, v in options.items() if k != "graph"})
    assert (a == b).all()
    assert sa["cycles"] == sb["cycles"]
    assert sa["rel_residual"] == pytest.approx(sb["rel_residual"], rel=1e-9)
    if "fmg" not in options and "graph" not in options:
        c, _ = solve(P, p, rho, fused=0, **options)
        assert (a == c).all()


@pytest.mark.parametrize("shape", [(33, 8, 33), (65, 6, 65)], ids=lambda s: "x".join(map(str, s)))
def test_masks(P, shape):
    """Frozen planes keep their iterate."""
    p = W.SMALL.with_sizes(*shape)
    say("plane masks", p.shape)
    rho = dev(W.blob_charge(p, 7))
    out = []
    for timing in (0, 1):
        phi, st = P.Plan.for_problem(p, masks=1, timing=timing).solve(rho, tol=1e-10)
        assert st["status"] == P.OK
        out.append(host(phi).copy())
    assert (out[0] == out[1]).all()
