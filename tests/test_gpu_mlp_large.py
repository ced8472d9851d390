"""The score network's FP32 forward pass on both sides of the rule that sends large
layers through LDS (two 128-wide tiles a CU, one with a deep first layer, the 64-wide
tile for H = 64 and between three and four tiles a CU), against the oracle, and the time
of a large one.

Tolerance: a sum of K <= 600 FP32 products carries about sqrt(K) 6e-8 = 1.5e-6 of its
terms' norm, and three layers follow one another: 1e-5 of the output's norm.
"""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


@pytest.mark.parametrize("D,H,B", [(7, 64, 65408), (7, 64, 65409), (7, 192, 32641), (9, 448, 16300), (511, 64, 32769),
                                   (513, 64, 32641), (600, 320, 10753), (5, 128, 98305), (5, 128, 131100)])
def test_forward_around_the_rule(ctx, D, H, B):
    print("forward", D, H, B, flush=True)
    rng = np.random.default_rng(D + H + B)
    theta = (rng.normal(size=omlp.n_params(D, H)) / np.sqrt(max(D, 8))).astype(np.float32)
    X = rng.normal(size=(B, D)).astype(np.float32)
    net = ffk.mlp_create(ctx, D, H, 1)
    ffk.mlp_set_params(ctx, net, torch.as_tensor(theta, device="cuda"))
    out = ffk.mlp_forward(ctx, net, torch.as_tensor(X, device="cuda"), prec=ffk.FP32).cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(200), rng.integers(0, B, size=1500), np.arange(B - 300, B)]))
    ref = omlp.forward(theta.astype(np.float64), X[rows].astype(np.float64), D, H)
    assert np.isfinite(out).all()
    assert np.linalg.norm(out[rows] - ref) <= 1e-5 * np.linalg.norm(ref)


def test_time_of_a_large_forward_pass(ctx):
    """D = 1770, H = 1024: 2048 rows take 290 us and 8192 took 1060, 600 through LDS."""
    net = ffk.mlp_create(ctx, 1770, 1024, 1)
    X = torch.randn(8192, 1770, generator=torch.Generator().manual_seed(1)).cuda()

    def ms(B):
        t = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ffk.mlp_forward(ctx, net, X[:B])
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return float(np.median(t[2:]))

    few, many = ms(2048), ms(8192)
    print("2048 rows %.3f ms, 8192 rows %.3f ms" % (few, many), flush=True)
    assert many < 2.8 * few
