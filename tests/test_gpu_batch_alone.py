"""A plan's solves in a batch and alone do not leave each other anything but
answers: what is bitwise the same alone stays so."""
import pytest

import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
# sizes at which a pass beside others is cut into other chunks than alone
SHAPES = [(129, 64, 129), (101, 48, 190)]


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


@pytest.mark.parametrize("merge", [0, 1])
def test_captured_graphs_of_a_batch_stay_with_the_batch(P, merge):
    """Replayed cycles have the launch shapes of the solve they serve: residual
    norms, whose sums depend on them, are those of a plan that was never in a batch."""
    probs = [W.SMALL.with_sizes(*s) for s in SHAPES]
    say("graphs of a batch", SHAPES, merge)
    rhos = [dev(W.blob_charge(p, 7)) for p in probs]
    fresh = [P.Plan.for_problem(p, graph=1, merge=merge) for p in probs]
    plans = [P.Plan.for_problem(p, graph=1, merge=merge) for p in probs]
    for _ in range(2):  # the second solve's checks follow the first's
        [f.solve(r, tol=1e-12) for f, r in zip(fresh, rhos)]
        P.solve_plans(plans, rhos, tol=1e-12)
    for _ in range(2):
        for f, p, r in zip(fresh, plans, rhos):
            a, sa = f.solve(r, tol=1e-12)
            a = host(a).copy()
            b, sb = p.solve(r, tol=1e-12)
            assert (host(b) == a).all()
            assert sb["history"] == sa["history"]


@pytest.mark.parametrize("options", [{}, {"merge": 0}, {"fmg": 1}, {"precision": 32}, {"masks": 1}, {"nu1": 3, "nu2": 3}], ids=str)
def test_a_batch_solves_as_alone(P, options):
    """Each problem exactly as alone: iterates, residual norms, checks and cycles."""
    probs = [W.SMALL.with_sizes(*s) for s in SHAPES]
    say("batch as alone", SHAPES, options)
    rhos = [dev(W.blob_charge(p, 7)) for p in probs]
    alone = [P.Plan.for_problem(p, **options) for p in probs]
    plans = [P.Plan.for_problem(p, **options) for p in probs]
    for _ in range(2):
        phis, sts = P.solve_plans(plans, rhos, tol=1e-12)
        for f, r, phi, sb in zip(alone, rhos, phis, sts):
            a, sa = f.solve(r, tol=1e-12)
            assert (host(phi) == host(a)).all()
            assert (sb["cycles"], sb["checks"], sb["history"]) == (sa["cycles"], sa["checks"], sa["history"])
