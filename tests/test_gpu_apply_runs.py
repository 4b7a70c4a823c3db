"""The operator at the edges of its runs of planes and blocks of rows, and in place."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import dev, host, say
from oracle import fv

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps
INTERIOR = (slice(None), slice(1, -1), slice(1, -1))


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


# one plane (its own neighbour), two (one neighbour on both sides), runs of
# eight planes with a whole and a partial last one, odd counts; blocks of four
# rows with one to four in the last
@pytest.mark.parametrize("nt", [1, 2, 3, 8, 9, 16, 17, 41])
@pytest.mark.parametrize("nz", [3, 6, 7, 8, 9])
@pytest.mark.parametrize("nr", [7, 130])
@pytest.mark.parametrize("in_place", [False, True])
def test_apply_runs(P, nt, nz, nr, in_place):
    p = W.SMALL.with_sizes(nr, nt, nz)
    say("apply runs", p.shape, in_place)
    phi = np.random.Generator(np.random.PCG64(nt * nz)).standard_normal(p.shape)
    plan = P.Plan.for_problem(p)
    x = dev(phi)
    out = x if in_place else torch.full_like(x, float("nan"))
    P.apply(plan.handle, x, out)
    got = host(out)
    ref = fv.charge_from_potential(fv.Grid.of(p, np.longdouble), phi.astype(np.longdouble)).astype(np.float64)
    g = fv.Grid.of(p)
    # the row's terms sum to at most twice its diagonal times the largest value;
    # each is rounded three times, as are their ten sums
    largest = 2 * (2 * g.theta_coupling() + g.D0) * np.abs(phi).max()
    bound = 16 * EPS * largest * fv.EPS0 / g.s_eps0
    assert (np.abs(got[INTERIOR] - ref[INTERIOR]) <= bound).all()
    assert (got[:, [0, -1], :] == 0).all() and (got[:, :, [0, -1]] == 0).all()
