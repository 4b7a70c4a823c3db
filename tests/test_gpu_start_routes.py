"""The full-multigrid start formed by the first down passes as they stream, bitwise
against the start written out by the interpolation kernel and read by the plain
down passes (the same node arithmetic, so the tolerance is zero)."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
BC = (10.0, -5.0, 0.0, 30.0)


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


def streams(P, plan, level) -> bool:
    """cp::fused_down_pro_ok of the plan: what the start and the first cycle ask."""
    f = P.library()._ZN2cp17fused_down_pro_okEPK15cylpoisson_plani
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_int]
    return bool(f(plan.handle, level))


def compare(P, make, rho, **options):
    """One and two cycles from the start, formed and written out."""
    for cycles in (1, 2):
        out = []
        for prefetch in (1, 2):
            plan = make(fmg=1, prefetch=prefetch, max_cycles=cycles, **options)
            assert plan.info()["fused_levels"] >= 1
            assert streams(P, plan, 0) == (prefetch == 1)
            phi = torch.full(plan.shape, float("nan"), dtype=torch.float64, device="cuda:0")
            phi, st = plan.solve(rho, tol=1e-30, phi=phi, allow=(P.OK, P.NOT_CONVERGED))
            assert st["cycles"] == cycles
            out.append((host(phi).copy(), st["history"]))
        assert np.isfinite(out[0][0]).all()
        assert (out[0][0] == out[1][0]).all()
        assert out[0][1] == out[1][1]


# one, two and three strips, the last pair of columns whole and half; one and
# two levels above the exact solve; one direction coarsened alone; a plane whose
# cycles run in one launch
@pytest.mark.parametrize("shape", [(33, 4, 35), (128, 4, 131), (131, 3, 70), (254, 3, 60), (257, 8, 300), (400, 2, 260),
                                   (65, 4, 401), (401, 4, 65)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("options", [{}, {"chunk_rows": 5, "chunk_rows_coarse": 3}, {"nu1": 3}, {"direct": 0}], ids=str)
def test_uniform(P, shape, options):
    p = W.SMALL.with_sizes(*shape)
    say("start routes", p.shape, options)
    compare(P, lambda **o: P.Plan.for_problem(p, **o), dev(W.blob_charge(p, 7)), **options)


# rows outside the band of equal rows: two (the half-cells at the faces), four,
# five, and all
@pytest.mark.parametrize("kind", ["cells", "wide2", "wide3", "growing"])
@pytest.mark.parametrize("options", [{}, {"chunk_rows": 5, "chunk_rows_coarse": 3}, {"nu1": 3}], ids=str)
def test_meshes(P, kind, options):
    nz = 290
    w = 1.01 ** np.arange(nz - 2) if kind == "growing" else np.ones(nz - 2)
    if kind.startswith("wide"):
        w[:int(kind[4:])] = 1.5 + 0.1 * np.arange(int(kind[4:]))
    z = 0.05 * np.concatenate([[0.0], np.cumsum(w) / w.sum()])
    r = np.linspace(0.02, 0.05, 270)
    say("start routes mesh", kind, options)
    t = np.arange(3 * nz * 271, dtype=np.float64).reshape(3, nz, 271)
    compare(P, lambda **o: P.Plan.from_mesh(r, z, 3, P.CELL, BC, **o), dev(1e-8 * np.sin(0.37 * t) + 1e-8), **options)
