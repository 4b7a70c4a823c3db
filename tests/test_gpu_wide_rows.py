"""Rows too long for 32-bit offsets within a few of them (45 million radial nodes
and more in a plane of three rows): the single sweeps serve them as they serve
any other, so a plane with the same nodes and such a pitch gives the same results.
"""
import ctypes

import pytest
import torch

import paper_2609_07172_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu

VP, I, D = ctypes.c_void_p, ctypes.c_int, ctypes.c_double


class Level(ctypes.Structure):
    """cp::DeviceLevel: its LevelView, and nothing else that these sweeps read."""
    _fields_ = [("nr", I), ("nz", I), ("pitch", I), ("pad", I), ("pstride", ctypes.c_longlong), ("tables", VP * 7),
                ("rest", ctypes.c_char * 512)]


def dev(n, seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return torch.rand(n, generator=g, device="cuda:0", dtype=torch.float64) + 0.5


def level(nr, nz, pitch, tables):
    return Level(nr, nz, pitch, 0, nz * pitch, (VP * 7)(*[t.data_ptr() for t in tables]), b"")


def spread(x, pitch):
    """The same nodes at another pitch (what lies between is left as allocated)."""
    nt, nz, nr = x.shape
    y = torch.empty(nt * nz * pitch + 2, dtype=torch.float64, device="cuda:0")
    v = torch.as_strided(y, (nt, nz, nr), (nz * pitch, pitch, 1))
    v.copy_(x)
    return y, v


# three strips of columns; a row is 0.36 GB (blocks of six rows pass 2 GB) and
# 0.8 GB (three rows do)
@pytest.mark.parametrize("pitch", [45_000_000, 100_000_000])
def test_same_as_at_an_ordinary_pitch(pitch):
    nt, nz, nr = 2, 5, 300
    say("wide rows", pitch)
    L = P.library()
    apply = L._ZN2cp12launch_applyERKNS_11DeviceLevelEidPKdS4_PdP12ihipStream_t
    apply.restype, apply.argtypes = I, [ctypes.POINTER(Level), I, D, VP, VP, VP, VP]
    norms = L._ZN2cp12launch_normsERKNS_11DeviceLevelEiPKdS4_S4_PdS5_S5_P12ihipStream_t
    norms.restype, norms.argtypes = I, [ctypes.POINTER(Level), I] + [VP] * 7
    tables = [dev(nr, k) for k in range(4)] + [dev(nz, k) for k in range(4, 7)]
    u, f, inv_s = (dev(nt * nz * nr, k).view(nt, nz, nr) for k in (8, 9, 10))
    lam = dev(nt, 11)
    out = []
    for q in (nr, pitch):
        lv = level(nr, nz, q, tables)
        (ub, _), (fb, _), (sb, _) = spread(u, q), spread(f, q), spread(inv_s[:1], q)
        ob, ov = spread(torch.full_like(u, float("nan")), q)
        partial, rn, bn = (torch.zeros(nt * 256, dtype=torch.float64, device="cuda:0") for _ in range(3))
        assert apply(lv, nt, 0.1, ub.data_ptr(), sb.data_ptr(), ob.data_ptr(), None) == 0
        r = []
        for r_ptr, b_ptr in ((rn.data_ptr(), bn.data_ptr()), (rn.data_ptr(), None), (None, bn.data_ptr())):
            assert norms(lv, nt, lam.data_ptr(), ub.data_ptr(), fb.data_ptr(), partial.data_ptr(), r_ptr, b_ptr, None) == 0
            torch.cuda.synchronize()
            r += [rn[:nt].cpu().tolist(), bn[:nt].cpu().tolist()]
        out.append((ov.cpu(), torch.tensor(r)))
    assert torch.isfinite(out[0][0]).all() and (out[0][0] == out[1][0]).all()
    # the order of the sums differs with the shape: 64 bits' rounding of 3000 terms
    assert torch.allclose(out[0][1], out[1][1], rtol=3000 * 2.3e-16, atol=0)
    del ub, fb, sb, ob, ov
    torch.cuda.empty_cache()  # tens of gigabytes
