"""The kernel clocks tick for every path of the dense steps: predictions by their own
kernel (and its reduction) and by the GEMMs, FP64 products of few geometries and of many."""
import numpy as np
import pytest
import torch

from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


def geometries(M, N, seed):
    grid = 1.5 * np.stack(np.unravel_index(np.arange(M), (5, 5, 4)), axis=1)
    return torch.from_numpy(grid + 0.08 * np.random.Generator(np.random.PCG64(seed)).normal(size=(N, M, 3))).cuda()


def ticks(ctx, call):
    call()
    ffk.clock_enable(ctx, 1)
    call()
    clk = ffk.clock_read(ctx)
    ffk.clock_enable(ctx, 0)
    for name, (ms, count) in clk.items():
        assert (ms > 0.0) == (count > 0), name
    return {name: count for name, (ms, count) in clk.items() if count}


@pytest.mark.parametrize("M,N,T,expect", [
    (9, 100, 1, {"fused": 1, "gemm2_reduce": 1}),
    (21, 2000, 200, {"fused": 1, "gemm2_reduce": 1}),
    (100, 131, 6300, {"gemm1": 2, "gemm2": 2}),   # two batches of 512 MB
])
def test_clocks_of_a_prediction(ctx, M, N, T, expect):
    S = ffk.descriptor_build(ctx, geometries(M, N, 1), 10.0)
    Te = ffk.descriptor_build(ctx, geometries(M, T, 2), 10.0)
    alpha = torch.from_numpy(np.random.Generator(np.random.PCG64(3)).normal(size=S.n)).cuda()
    assert ticks(ctx, lambda: ffk.kernel_predict(ctx, S, Te, alpha)) == expect


@pytest.mark.parametrize("N,dense", [(100, {"fused": 1}), (1500, {"gemm1": 1, "gemm2": 1})])
def test_clocks_of_an_fp64_product(ctx, N, dense):
    S = ffk.descriptor_build(ctx, geometries(21, N, 1), 10.0)
    v = torch.from_numpy(np.random.Generator(np.random.PCG64(3)).normal(size=S.n)).cuda()
    assert ticks(ctx, lambda: ffk.kernel_mvm(ctx, S, v)) == dict({"jv": 1, "colsum": 1, "jtg": 1}, **dense)
