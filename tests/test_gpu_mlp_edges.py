"""The score network's FP32 kernels at the edges of their tiles (16, 32), of the
four-way split of K and of the batch size up to which dout is formed in LDS (1024).

Tolerance: a sum of K <= 2048 FP32 products carries about sqrt(K) 6e-8 = 3e-6 of
its terms' norm, and three layers follow one another: 1e-5 of the gradient's norm.
"""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ffk():
    from paper_2212_12737_amd import ffk as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def ctx(ffk):
    return ffk.create(0)


@pytest.mark.parametrize("D,H,B", [(1, 64, 1), (3, 64, 15), (17, 64, 17), (16, 128, 33), (210, 256, 256), (31, 192, 1024),
                                   (36, 128, 1025), (861, 256, 2048)])
def test_gradient_at_tile_edges(ffk, ctx, D, H, B):
    print("mlp", D, H, B, flush=True)
    rng = np.random.default_rng(D + H + B)
    theta = (rng.normal(size=omlp.n_params(D, H)) / np.sqrt(max(D, 8))).astype(np.float32)
    X = rng.normal(size=(B, D)).astype(np.float32)
    y = rng.normal(size=B).astype(np.float32)
    net = ffk.mlp_create(ctx, D, H, 1)
    dev = lambda a: torch.as_tensor(a, device="cuda")
    ffk.mlp_set_params(ctx, net, dev(theta))
    out = ffk.mlp_forward(ctx, net, dev(X), prec=ffk.FP32).cpu().numpy().astype(np.float64)
    ref = omlp.forward(theta.astype(np.float64), X.astype(np.float64), D, H)
    assert np.linalg.norm(out - ref) <= 1e-5 * np.linalg.norm(ref)
    loss, grad = ffk.mlp_grad(ctx, net, dev(X), dev(y))
    L, g = omlp.backward(theta.astype(np.float64), X.astype(np.float64), y.astype(np.float64), D, H)
    assert abs(loss.item() - L) <= 1e-5 * L
    err = grad.cpu().numpy().astype(np.float64) - g
    assert np.linalg.norm(err) <= 1e-5 * np.linalg.norm(g)
