"""The fused passes where a level's axial spacing is not one band of equal rows,
bitwise against the per-step kernels (the same node arithmetic, so the
tolerance is zero)."""
import numpy as np
import pytest

import workloads as W
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu
BC = (10.0, -5.0, 0.0, 30.0)


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


def axial_cells(n, kind):
    """Cell widths: equal but for `kind` wider ones at the first face, the last or both, or growing."""
    w = np.ones(n)
    if kind == "growing":
        return 1.01 ** np.arange(n)
    where, count = kind
    for k in range(count):
        if where in ("first", "both"):
            w[k] = 1.5 + 0.1 * k
        if where in ("last", "both"):
            w[n - 1 - k] = 1.7 + 0.1 * k
    return w


# rows outside the band: two (the half-cells next to the faces) to nine, on
# either side of the four up to which the band's coefficients stay in registers;
# chunks shorter than the rows a wavefront holds, and sweep counts whose merged
# pass has five sweeps and whose up pass three
@pytest.mark.parametrize("kind", [("first", 0), ("first", 1), ("last", 1), ("both", 1), ("last", 5), ("both", 3),
                                  "growing"], ids=str)
@pytest.mark.parametrize("nz", [70, 131])
@pytest.mark.parametrize("options", [{}, {"chunk_rows": 5, "chunk_rows_coarse": 3, "chunk_rows_merge": 4},
                                     {"merge": 0}, {"nu2": 3}], ids=str)
def test_rows_outside_the_band(P, kind, nz, options):
    w = axial_cells(nz - 2, kind)
    z = 0.05 * np.concatenate([[0.0], np.cumsum(w) / w.sum()])
    r = np.linspace(0.02, 0.05, 137 - 1)
    say("rows outside the band", kind, nz, options)
    out = []
    for fused in (1, 0):
        plan = P.Plan.from_mesh(r, z, 4, P.CELL, BC, max_cycles=3, fused=fused, **options)
        shape = plan.shape
        if not out:
            t = np.arange(np.prod(shape), dtype=np.float64).reshape(shape)
            rho = dev(1e-8 * np.sin(0.37 * t) + 1e-8)
        phi, _ = plan.solve(rho, tol=1e-30, allow=(P.OK, P.NOT_CONVERGED))
        out.append(host(phi))
        if fused:
            assert plan.info()["fused_levels"] >= 1
    assert (out[0] == out[1]).all()
