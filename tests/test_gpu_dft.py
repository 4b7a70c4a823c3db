"""The folded DFT products on the matrix cores, for numbers of azimuths at the
edges of their tiles and k-blocks, against the oracle's explicit sums."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, say
from oracle import spectral

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


# 16 results a tile and four azimuths a k-block of N // 2 + 1 modes: one mode, a
# block more and less, a tile more and less, the steps of the larger register
# blocks (17, 18, 23, 28, 33), the largest N and the first beyond it; 35 columns
# leave a wavefront's columns part empty
@pytest.mark.parametrize("nt", [1, 2, 3, 6, 7, 8, 29, 30, 31, 32, 61, 62, 63, 64, 97, 128, 133, 134, 135, 136, 141,
                                142, 181, 182, 221, 222, 223, 255, 256, 257])
def test_planes_and_back(P, nt):
    say("dft products", nt)
    plan = P.Plan(7, nt, 5, 0.02, 0.05, 0.01, fft=0)
    x = np.random.default_rng(nt).standard_normal((nt, 5, 7))
    xd = dev(x)
    planes, back = torch.empty_like(xd), torch.empty_like(xd)
    P.dft_forward(plan.handle, xd, planes)
    # N products of weight <= 1 / N, added up on each side: N eps sum|x| / N each
    # for the sums and the weights' own rounding
    bound = 4 * EPS * np.abs(x).sum(axis=0)[None] + 1e-300
    assert (np.abs(host(planes) - spectral.forward(x)) <= bound).all()
    P.dft_inverse(plan.handle, planes, back)
    bound = 8 * nt * EPS * np.abs(host(planes)).sum(axis=0)[None] + 1e-300
    assert (np.abs(host(back) - spectral.inverse(host(planes))) <= bound).all()


def test_solve_scales_the_planes(P):
    """The right-hand side scale of the forward transform: a solve with the
    products against one with the register FFT, both at the residual's tolerance."""
    import workloads as W

    p = W.SMALL
    say("dft products in a solve", p.shape)
    rho = dev(W.blob_charge(p))
    a, _ = P.Plan.for_problem(p, fft=0).solve(rho, tol=1e-13)
    b, _ = P.Plan.for_problem(p, fft=1).solve(rho, tol=1e-13)
    a, b = host(a), host(b)
    assert np.linalg.norm(a - b) <= 1e-11 * np.linalg.norm(b)
