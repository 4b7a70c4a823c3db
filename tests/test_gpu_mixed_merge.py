"""The mixed-precision solve's inner cycles: the merged finest pass against the
separate ones (bitwise), and the exact coarse solve on FP32 levels."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, host, rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


def plan_for(P, p, growing, **options):
    if not growing:
        return P.Plan.for_problem(p, precision=32, **options)
    r = np.linspace(0.02, 0.05, p.nr - 1)
    w = 1.01 ** np.arange(p.nz - 2)
    z = 0.05 * np.concatenate([[0.0], np.cumsum(w) / w.sum()])
    return P.Plan.from_mesh(r, z, p.ntheta, P.CELL, p.bc, precision=32, **options)


# one and several strips; the exact solve in one workgroup a plane (up to 64
# interior nodes) and in two kernels; equal rows and a table of rows
@pytest.mark.parametrize("shape", [(65, 6, 65), (127, 4, 130), (129, 4, 131), (257, 4, 200)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("growing", [False, True])
@pytest.mark.parametrize("options", [{}, {"inner_cycles": 3}, {"direct": 0}, {"direct": 2}], ids=str)
def test_merged_inner_cycles(P, shape, growing, options):
    p = W.SMALL.with_sizes(*shape)
    say("merged inner cycles", p.shape, growing, options)
    rho = dev(W.blob_charge(p, 7))
    out = []
    for merge in (1, 0):
        plan = plan_for(P, p, growing, merge=merge, max_cycles=6, **options)
        phi, st = plan.solve(rho, tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
        assert st["cycles"] == 6
        out.append(host(phi).copy())
    assert (out[0] == out[1]).all()


@pytest.mark.parametrize("nr", [18, 34, 65, 66, 67, 130, 131, 200])
@pytest.mark.parametrize("direct", [0, 1, 2])
def test_exact_coarse_solve(P, nr, direct):
    """Every stop of the inner cycles leads to the FP64 answer (to the tolerance and its amplification)."""
    p = W.SMALL.with_sizes(nr, 5, nr + 9)
    say("inner stop", p.shape, direct)
    rho = dev(W.blob_charge(p, 7))
    a, _ = P.Plan.for_problem(p).solve(rho, tol=1e-13)
    a = host(a).copy()
    b, st = P.Plan.for_problem(p, precision=32, direct=direct).solve(rho, tol=1e-13)
    assert st["status"] == P.OK
    assert rel_l2(host(b), a) <= 1e-11
