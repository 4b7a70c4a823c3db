"""The network's streaming forward and its backward kernel where strips, row
chunks and tiles end, against the CPU oracle.

Tolerances as in the network's other tests: operands are rounded to BF16 alike,
so only an activation within FP32 rounding of a BF16 tie can differ (about 1 in
4e4 entries, by 2^-8): 1e-4 on outputs, 5e-4 on gradients.
"""
import numpy as np
import pytest
import torch

from gpu_util import say
from oracle import nn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2609_07172_amd as P

    P.library()
    return P


def unflat(w):
    out, o = [], 0
    for ci, co in nn.SHAPES:
        n = 9 * ci * co
        out.append(w[o:o + n].astype(np.float64).reshape(9, ci, co))
        o += n
    return out


def rel(a, b):
    n = np.linalg.norm(np.ravel(b))
    d = np.linalg.norm(np.ravel(a) - np.ravel(b))
    return float(d / n) if n else float(d)


# widths: strips of 26, 42 and 58 pixels, one pixel more, two strips and one
# more; heights: chunks of eight rows, one more and less; tiles of 16 x 32
@pytest.mark.parametrize("shape", [(3, 7, 26), (2, 8, 27), (2, 9, 42), (1, 17, 43), (2, 33, 58), (1, 16, 59),
                                   (1, 8, 116), (1, 25, 117), (130, 8, 33), (300, 16, 32), (1, 70, 31)],
                         ids=lambda s: "x".join(map(str, s)))
def test_forward_and_gradients(P, shape):
    B, H, W = shape
    say("network", shape)
    rng = np.random.Generator(np.random.PCG64(B + 7 * H + 31 * W))
    net = P.Net(seed=1)
    net.set_weights(np.concatenate([p.astype(np.float32).ravel() for p in nn.init_params(9)]))
    params = unflat(net.get_weights())
    x = rng.standard_normal((B, H, W, 4)).astype(np.float32)
    t = rng.standard_normal((B, H, W, 2)).astype(np.float32)
    # images start anywhere: only a float's alignment is given
    buf = torch.zeros(x.size + 1, dtype=torch.float32, device="cuda:0")
    xd = buf[1:].view(B, H, W, 4)
    xd.copy_(torch.from_numpy(x))
    y = net.forward(xd).cpu().numpy()
    ref, _ = nn.forward(params, x.astype(np.float64), rounding=True)
    assert rel(y, ref) <= 1e-4, rel(y, ref)
    loss = net.loss_grad(xd, torch.from_numpy(t).to("cuda:0"))
    ref_loss, ref_grads = nn.loss_and_grads(params, x.astype(np.float64), t.astype(np.float64), rounding=True)
    assert loss == pytest.approx(ref_loss, rel=1e-4)
    g = unflat(net.get_grads())
    for l in range(3):
        assert rel(g[l], ref_grads[l]) <= 5e-4, (l, rel(g[l], ref_grads[l]))
    # the packed copies that a step leaves are those of its weights
    net.adam_step(1e-2)
    stepped = net.get_weights()
    y1 = net.forward(xd).cpu().numpy()
    net.set_weights(stepped)
    assert (y1 == net.forward(xd).cpu().numpy()).all()


def test_no_inner_pixels(P):
    """An image narrower than the loss's border: zero loss, zero gradients."""
    net = P.Net(seed=2)
    x = torch.ones((2, 6, 9, 4), device="cuda:0")
    assert net.loss_grad(x, torch.zeros((2, 6, 9, 2), device="cuda:0")) == 0.0
    assert (net.get_grads() == 0).all()
