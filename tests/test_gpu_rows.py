"""The single sweeps over a level's rows (operator, plane norms, the mixed
solve's refinement, the finest right-hand side's restriction) at the edges of
their strips and chunks."""
import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import dev, host, rel_l2, say
from oracle import fv

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps
INTERIOR = (slice(None), slice(1, -1), slice(1, -1))

# radial nodes: one strip up to 128, two up to 252, three beyond; the last
# column pair whole and half; a single interior column
EDGES = [3, 4, 5, 126, 127, 128, 129, 130, 251, 252, 253, 254, 255]


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


@pytest.mark.parametrize("nr", EDGES)
@pytest.mark.parametrize("nz", [3, 4, 5, 31])
def test_apply(P, nr, nz):
    """Against the oracle in extended precision, within rounding of the terms that cancel."""
    p = W.SMALL.with_sizes(nr, 3, nz)
    say("apply", p.shape)
    phi = W.manufactured_potential(p, 3)
    out = torch.full(p.shape, float("nan"), dtype=torch.float64, device="cuda")
    plan = P.Plan.for_problem(p)
    P.apply(plan.handle, dev(phi), out)
    got = host(out)
    ref = fv.charge_from_potential(fv.Grid.of(p, np.longdouble), phi.astype(np.longdouble)).astype(np.float64)
    g = fv.Grid.of(p)
    ab = np.abs(phi)
    scale = abs(fv.assemble(g)) @ ab[INTERIOR].ravel() + fv.rhs(g, np.zeros(g.shape), ab).ravel()
    scale = scale.reshape(g.interior_shape) * fv.EPS0 / g.s_eps0
    bound = 64 * EPS * scale.max(axis=0)[None] * p.ntheta
    assert (np.abs(got[INTERIOR] - ref[INTERIOR]) <= bound).all()
    assert (got[:, [0, -1], :] == 0).all() and (got[:, :, [0, -1]] == 0).all()


def test_a_solve_after_apply_is_the_one_before(P):
    """The operator's scratch is no state of the next solve."""
    p = W.SMALL.with_sizes(130, 4, 70)
    rho = dev(W.blob_charge(p, 7))
    say("solve after apply")
    plan = P.Plan.for_problem(p, warm_start=0)
    a = host(plan.solve(rho, tol=1e-12)[0]).copy()
    bad = torch.full_like(rho, float("nan"))
    P.apply(plan.handle, bad, torch.empty_like(bad))
    assert (host(plan.solve(rho, tol=1e-12)[0]) == a).all()


# the right-hand side's norm: alone, with the residual's (warm start), with the
# refinement of the mixed solve, with the restriction of the full-multigrid start
@pytest.mark.parametrize("nr", [n for n in EDGES if n > 5])
@pytest.mark.parametrize("nz", [70, 131])
@pytest.mark.parametrize("options", [{"fmg": 0}, {"warm_start": 1}, {"precision": 32}, {"fmg": 1}], ids=str)
def test_right_hand_side_norm(P, nr, nz, options):
    p = W.SMALL.with_sizes(nr, 4, nz)
    say("norm", p.shape, options)
    rho = W.blob_charge(p, 7)
    g = fv.Grid.of(p)
    # the planes carry 1 / N each, so their weighted squares sum to ||b||^2 / N
    ref = np.linalg.norm(fv.rhs(g, rho, fv.boundary_values(g, p.bc))) / np.sqrt(p.ntheta)
    plan = P.Plan.for_problem(p, max_cycles=1, **options)
    phi = torch.zeros(p.shape, dtype=torch.float64, device="cuda")
    _, st = plan.solve(dev(rho), phi=phi, tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
    # a sum of n squares, each from a transform of four values: n/2 + 8 roundings at most
    n = (nr - 2) * (nz - 2)
    assert st["initial_residual_norm"] == pytest.approx(ref, rel=(n + 16) * EPS)


@pytest.mark.parametrize("nr", [n for n in EDGES if n > 5])
@pytest.mark.parametrize("nz", [66, 67])
def test_residual_norm_of_a_guess(P, nr, nz):
    """With zero faces nine tenths of the answer leave a tenth of the right-hand side."""
    p = W.SMALL.with_sizes(nr, 4, nz)
    say("guess", p.shape)
    rho = dev(W.blob_charge(p, 7))
    bc = (0.0, 0.0, 0.0, 0.0)
    plan = P.Plan(p.nr, p.ntheta, p.nz, p.r_in, p.r_out, p.dz, bc, warm_start=1)
    phi = torch.zeros(p.shape, dtype=torch.float64, device="cuda")
    phi, st = plan.solve(rho, phi=phi, tol=1e-12)
    guess = 0.9 * phi
    _, st = plan.solve(rho, phi=guess, tol=0.5)
    assert st["cycles"] == 0
    # the answer's own residual, and the rounding of its terms (below it)
    assert st["rel_residual"] == pytest.approx(0.1, abs=2e-12)


@pytest.mark.parametrize("nr", [n for n in EDGES if n > 5])
@pytest.mark.parametrize("nz", [70, 131])
def test_mixed_solve(P, nr, nz):
    p = W.SMALL.with_sizes(nr, 4, nz)
    say("mixed", p.shape)
    rho = dev(W.blob_charge(p, 7))
    a, _ = P.Plan.for_problem(p).solve(rho, tol=1e-13)
    a = host(a).copy()
    b, st = P.Plan.for_problem(p, precision=32).solve(rho, tol=1e-13)
    assert st["status"] == P.OK
    assert rel_l2(host(b), a) <= 1e-11


# Both of the following compare two ways to the same iterate after one cycle
# from the full-multigrid start.  They differ by the rounding of right-hand
# sides (a few EPS of the largest) and of sums in another order, which one
# cycle and the solves below it (condition at most the nodes of a plane) carry
# into the answer: 1e-11 of it at these sizes.
def one_cycle(P, p, rho, bc):
    plan = P.Plan(p.nr, p.ntheta, p.nz, p.r_in, p.r_out, p.dz, bc, max_cycles=1, fmg=1)
    phi, _ = plan.solve(dev(rho), tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
    return host(phi)


@pytest.mark.parametrize("nr", [n for n in EDGES if n > 5])
@pytest.mark.parametrize("nz", [70, 131])
def test_start_from_faces_or_charge(P, nr, nz):
    """Face values enter as the charge that gives the nodes next to them the same right-hand side."""
    p = W.SMALL.with_sizes(nr, 4, nz)
    say("faces as charge", p.shape)
    rho = W.blob_charge(p, 7)
    g = fv.Grid.of(p)
    bc = (10.0, -5.0, 20.0, 30.0)
    same = rho.copy()
    same[INTERIOR] += fv.rhs(g, np.zeros(g.shape), fv.boundary_values(g, bc)) * fv.EPS0 / g.s_eps0
    assert rel_l2(one_cycle(P, p, rho, bc), one_cycle(P, p, same, (0.0, 0.0, 0.0, 0.0))) <= 1e-11


@pytest.mark.parametrize("nr", [126, 129, 254])
@pytest.mark.parametrize("nz", [65, 129, 131])
def test_start_upside_down(P, nr, nz):
    """An odd count of rows is coarsened, coloured and chunked the same from either end up to the chunks' edges."""
    p = W.SMALL.with_sizes(nr, 4, nz)
    say("upside down", p.shape)
    rho = W.blob_charge(p, 7)
    a = one_cycle(P, p, rho, (10.0, -5.0, 20.0, 30.0))
    b = one_cycle(P, p, rho[:, ::-1], (10.0, -5.0, 30.0, 20.0))
    assert rel_l2(b[:, ::-1], a) <= 1e-11
