"""The exact solve of a coarse level at the edges of its 16 x 16 tiles, groups
of eigenvectors and elimination segments, against the oracle."""
import numpy as np
import pytest

import workloads as W
from gpu_util import INTERIOR, dev, host, rel_l2, say
from oracle import fv, solvers

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


# (radial, axial) interior nodes of level 1: one workgroup of 1, 4 or 16
# wavefronts a plane, a tile more and less; the two-kernel form with an odd and
# an even number of groups, one node past a group, the largest; few rows
@pytest.mark.parametrize("n", [(15, 16), (16, 17), (17, 16), (32, 31), (33, 32), (32, 33), (64, 63), (63, 64), (65, 64),
                               (64, 65), (80, 96), (97, 81), (113, 112), (112, 113), (128, 127), (127, 128), (90, 20),
                               (20, 90)], ids=lambda n: "x".join(map(str, n)))
@pytest.mark.parametrize("nt", [1, 3, 10])
def test_solve_matches_oracle(P, n, nt):
    nr, nz = 2 * n[0] + 3, 2 * n[1] + 3
    dr = 0.03 / (nr - 1)
    # square cells, so that both directions are coarsened
    p = W.Problem(nr, nt, nz, 0.02, 0.05, dr)
    say("direct level", n, nt)
    plan = P.Plan.for_problem(p)
    info = plan.info()
    assert info["direct_level"] == 1 and info["level_shapes"][1] == (n[0] + 2, n[1] + 2)
    rho = W.blob_charge(p, 5)
    phi, st = plan.solve(dev(rho), tol=1e-14, allow=(P.OK, P.NOT_CONVERGED))
    got = host(phi)
    ref = solvers.solve_separable(fv.Grid.of(p), rho, p.bc)
    # the answer to the bar of every FP64 solve; an exact coarse correction
    # contracts each cycle by far more than 0.2
    assert rel_l2(got, ref, INTERIOR) <= 1e-12
    h = [x for x in st["history"] if x is not None]
    assert h[-1] <= 0.2 ** (len(st["history"]) - 2), st["history"]
    assert np.isfinite(got).all()
