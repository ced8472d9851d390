"""Prediction and the FP64 product at the edges of prediction's tiles (16 or 32
test geometries, 16 or 64 training ones, batches of 512), of the small
coefficient tiles (16, up to 1024 padded rows) and of the column means (512
rows), against the oracle: 1e-10 norm-wise, the bound of the FP64 operators.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok
from oracle import symmetry as osym

pytestmark = pytest.mark.gpu

SIGMA = 10.0


@pytest.fixture(scope="module")
def ffk():
    from paper_2212_12737_amd import ffk as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def ctx(ffk):
    return ffk.create(0)


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), device="cuda")


def relerr(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def geometries(M, N, seed):
    return synth.make_system(M, N, 0.08, True, 1000 + M, seed, 7).R


@pytest.mark.parametrize("M,N,T", [(3, 1, 1), (4, 15, 2), (5, 17, 16), (6, 63, 17), (7, 65, 33), (12, 300, 1), (9, 130, 48),
                                   (5, 1400, 400), (4, 70, 513), (3, 3, 1030), (30, 40, 5), (3, 5000, 200),
                                   (4, 2200, 500), (3, 1700, 700)])
def test_prediction_at_tile_edges(ffk, ctx, M, N, T):
    print("predict", M, N, T, flush=True)
    R, Rt = geometries(M, N, 1), geometries(M, T, 2)
    alpha = synth.random_vectors(3 * M * N, 3)
    train, test = (ffk.descriptor_build(ctx, dev(r), SIGMA) for r in (R, Rt))
    F = ffk.kernel_predict(ctx, train, test, dev(alpha)).cpu().numpy()
    assert relerr(F, ok.kernel_mvm(Rt, R, alpha, SIGMA)) <= 1e-10


def test_prediction_of_a_symmetrized_model(ffk, ctx):
    R, Rt = geometries(6, 50, 4), geometries(6, 21, 5)
    perms = np.array([[0, 1, 2, 3, 4, 5], [1, 0, 2, 3, 4, 5], [0, 1, 2, 3, 5, 4], [1, 0, 2, 3, 5, 4]])
    alpha = synth.random_vectors(3 * 6 * 50, 6)
    train, test = (ffk.descriptor_build(ctx, dev(r), SIGMA) for r in (R, Rt))
    ffk.set_symmetries(ctx, train, perms)
    F = ffk.kernel_predict(ctx, train, test, dev(alpha)).cpu().numpy()
    assert relerr(F, osym.sym_kernel_mvm(R, perms, alpha, SIGMA, Rt)) <= 1e-10


@pytest.mark.parametrize("M,N", [(3, 16), (3, 17), (4, 511), (3, 513), (3, 1024), (4, 1030), (16, 1281)])
def test_product_at_coefficient_and_mean_edges(ffk, ctx, M, N):
    print("product", M, N, flush=True)
    R = geometries(M, N, 8)
    v = synth.random_vectors(3 * M * N, 9)
    S = ffk.descriptor_build(ctx, dev(R), SIGMA)
    y = ffk.kernel_mvm(ctx, S, dev(v), prec=ffk.FP64).cpu().numpy()
    assert relerr(y, ok.kernel_mvm(R, R, v, SIGMA)) <= 1e-10
