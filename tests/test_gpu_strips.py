"""The fused passes' strips and chunks at their edges, bitwise against the
per-step kernels (the same node arithmetic, so the tolerance is zero)."""
import pytest

import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


def both(P, p, **options):
    """The iterate after three cycles by the fused passes and by the per-step kernels."""
    rho = dev(W.blob_charge(p, 7))
    out = []
    for fused in (1, 0):
        plan = P.Plan.for_problem(p, max_cycles=3, fused=fused, **options)
        phi, _ = plan.solve(rho, tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
        out.append(host(phi))
        if fused:
            assert plan.info()["fused_levels"] >= 1
    return out


# radial nodes: one strip up to 128 (two more with an open edge each side of it),
# 237 and 344 / 345 where four merged sweeps take one strip more, one column more
# and less; even and odd; a level of a single interior column
@pytest.mark.parametrize("nr", [3, 4, 127, 128, 129, 130, 236, 237, 238, 344, 345, 513, 514, 700])
def test_strip_edges(P, nr):
    # a plane of more unknowns than the coarsest level keeps (64), so that there are two levels
    p = W.SMALL.with_sizes(nr, 4, 200 if nr < 10 else 70)
    say("strip edges", p.shape)
    a, b = both(P, p)
    assert (a == b).all()


# cells flat enough that the first level is coarsened along one direction only,
# with even and odd node counts, and chunks of one to a few rows
@pytest.mark.parametrize("shape", [(65, 4, 301), (66, 3, 300), (301, 4, 65), (300, 3, 66), (130, 8, 401)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("chunk", [0, 1, 7])
def test_levels_coarsened_in_one_direction(P, shape, chunk):
    p = W.SMALL.with_sizes(*shape)
    say("one direction", p.shape, chunk)
    a, b = both(P, p, chunk_rows=chunk, chunk_rows_coarse=chunk, chunk_rows_merge=chunk)
    assert (a == b).all()


def test_ring_entries_of_a_plane_right_hand_side_are_not_read(P):
    """solve_planes ignores the ring of b: NaN there changes nothing."""
    import torch

    p = W.SMALL.with_sizes(131, 4, 66)
    say("ring of b", p.shape)
    b = dev(W.blob_charge(p, 9))
    bad = b.clone()
    bad[:, 0, :] = bad[:, -1, :] = float("nan")
    bad[:, :, 0] = bad[:, :, -1] = float("nan")
    out = []
    for rhs in (b, bad):
        plan = P.Plan.for_problem(p)
        u = torch.zeros_like(b)
        P.solve_planes(plan.handle, rhs, u, 1e-12)
        out.append(host(u))
    assert (out[0] == out[1]).all()
