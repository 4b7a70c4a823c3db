"""A batch's lanes: more problems than lanes, in every order, repeated, against
each problem solved alone (bitwise: chunks change no node's arithmetic)."""
import pytest
import torch

import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
SHAPES = [(33, 4, 35), (129, 6, 70), (17, 3, 19), (70, 8, 129), (65, 4, 65), (40, 5, 33), (101, 2, 66)]


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


@pytest.mark.parametrize("count", [1, 2, 3, 4, 7])
def test_batch_of_uneven_problems(P, count):
    probs = [W.SMALL.with_sizes(*s) for s in SHAPES[:count]]
    say("batch lanes", [p.shape for p in probs])
    rhos = [dev(W.blob_charge(p, 7)) for p in probs]
    alone = [host(P.Plan.for_problem(p, fmg=1).solve(r, tol=1e-12)[0]).copy() for p, r in zip(probs, rhos)]
    plans = [P.Plan.for_problem(p, fmg=1) for p in probs]
    side = torch.cuda.Stream()
    for turn in range(3):
        order = [(i + turn) % count for i in range(count)]  # another plan leads
        phis = [torch.full_like(rhos[i], float("nan")) for i in order]
        stream = None
        if turn == 2:
            side.wait_stream(torch.cuda.current_stream())
            stream = side
        status, sts = P.solve_batch([plans[i].handle for i in order], [rhos[i] for i in order], phis, tol=1e-12,
                                    stream=stream)
        assert status == P.OK and all(s == P.OK for s in sts)
        for i, phi in zip(order, phis):
            assert (host(phi) == alone[i]).all()
    # the leader of the first turn goes; the others' streams are their own
    lead = plans.pop(0)
    lead.close()
    if plans:
        phis = [torch.empty_like(r) for r in rhos[1:]]
        status, _ = P.solve_batch([p.handle for p in plans], rhos[1:], phis, tol=1e-12)
        assert status == P.OK
        assert all((host(f) == a).all() for f, a in zip(phis, alone[1:]))
