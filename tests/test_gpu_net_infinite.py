"""Infinite values in the network: each one reaches exactly the results whose
taps it belongs to.  Products with the zero weights and zero gradients that only
pad an operand would turn it into NaN.

Weights and inputs are positive, so that sums of infinities stay infinite; the
finite entries' tolerances are those of the network's other tests (BF16 ties
decided by FP32 rounding): 1e-4 on outputs, 5e-4 on gradients.
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


def positive_net(P):
    rng = np.random.Generator(np.random.PCG64(3))
    params = [rng.uniform(0.01, 0.1, (9, ci, co)).astype(np.float32) for ci, co in nn.SHAPES]
    net = P.Net(seed=1)
    net.set_weights(np.concatenate([w.ravel() for w in params]))
    return net, [w.astype(np.float64) for w in params], rng


def same(got, ref, tol):
    got, ref = np.asarray(got, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    assert (np.isnan(got) == np.isnan(ref)).all(), (np.isnan(got).sum(), np.isnan(ref).sum())
    assert (got[np.isinf(ref)] == ref[np.isinf(ref)]).all()
    ok = np.isfinite(ref)
    assert np.isfinite(got[ok]).all()
    assert np.linalg.norm(got[ok] - ref[ok]) <= tol * np.linalg.norm(ref[ok])


# one strip of each width, and two strips with the value on either side of their border
@pytest.mark.parametrize("shape", [(9, 26), (9, 42), (9, 58), (20, 70)], ids=lambda s: "x".join(map(str, s)))
def test_forward(P, shape):
    H, W = shape
    say("infinite input", shape)
    net, params, rng = positive_net(P)
    where = [(0, 0), (H - 1, W - 1), (4, 5), (H // 2, W // 2), (5, min(W - 1, 57)), (6, min(W - 1, 58))]
    x = rng.uniform(0.1, 1.0, (len(where), H, W, 4)).astype(np.float32)
    for b, (i, j) in enumerate(where):
        x[b, i, j, b % 4] = np.inf
    ref, _ = nn.forward(params, x.astype(np.float64))
    assert np.isinf(ref).any() and not np.isnan(ref).any()
    same(net.forward(torch.from_numpy(x).to("cuda:0")).cpu().numpy(), ref, 1e-4)


def weight_grad(x, g):
    """nn.weight_grad with every product formed (a zero gradient under an infinite activation is NaN)."""
    B, H, W, c = x.shape
    xp = np.pad(x, ((0, 0), (1, 1), (1, 1), (0, 0)))
    out = []
    for dy, dx in nn.TAPS:
        xs = xp[:, 1 + dy:1 + dy + H, 1 + dx:1 + dx + W].reshape(-1, c, 1)
        out.append((xs * g.reshape(-1, 1, g.shape[3])).sum(axis=0))
    return np.array(out)


def gradients(params, x, target):
    """The oracle's gradients with those products."""
    y, acts = nn.forward(params, x)
    inner = nn.inner_mask(*y.shape[1:3])[None, :, :, None] > 0
    g = np.where(inner, y - target, 0.0) / (y.shape[0] * inner.sum() * 2)
    grads = [None] * 3
    for l in (2, 1, 0):
        g = nn.bf16(g)
        grads[l] = weight_grad(acts[l], g)
        if l:
            g = np.where(acts[l] > 0.0, nn.conv_adjoint(g, nn.bf16(params[l])), 0.0)
    return grads


def check_gradients(P, x, target, net, params):
    with np.errstate(invalid="ignore"):
        ref = gradients(params, x.astype(np.float64), target.astype(np.float64))
    net.loss_grad(torch.from_numpy(x).to("cuda:0"), torch.from_numpy(target).to("cuda:0"))
    got, at = net.get_grads(), 0
    for l, (ci, co) in enumerate(nn.SHAPES):
        n = 9 * ci * co
        same(got[at:at + n], ref[l].ravel(), 5e-4)
        at += n
    return ref


def test_infinite_target(P):
    """Every gradient through the one infinite pixel of the output is infinite, none is NaN."""
    H, W = 16, 32
    say("infinite target", (H, W))
    net, params, rng = positive_net(P)
    x = rng.uniform(0.1, 1.0, (2, H, W, 4)).astype(np.float32)
    target = rng.uniform(0.1, 1.0, (2, H, W, 2)).astype(np.float32)
    target[0, 8, 11, 1] = np.inf
    ref = check_gradients(P, x, target, net, params)
    assert np.isinf(ref[0]).all() and np.isinf(ref[1]).all()


# images that end inside a tile of 16 x 32 pixels, in the first tile and in the second
@pytest.mark.parametrize("shape", [(13, 29), (20, 40)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("edge", ["corner", "row", "column"])
def test_infinite_edge_activation(P, shape, edge):
    """The weight gradients sum over the image's pixels: beside its last row and
    column lie tile positions outside it, with zero gradients, which add nothing."""
    H, W = shape
    say("infinite edge", shape, edge)
    net, params, rng = positive_net(P)
    x = rng.uniform(0.1, 1.0, (2, H, W, 4)).astype(np.float32)
    target = rng.uniform(0.1, 1.0, (2, H, W, 2)).astype(np.float32)
    x[(0, *{"corner": (H - 1, W - 1), "row": (H - 1, 10), "column": (8, W - 1)}[edge], 1)] = np.inf
    ref = check_gradients(P, x, target, net, params)
    assert np.isinf(ref[0]).sum() == 528
