"""A large prediction reads padded copies of the model's descriptor that a product may have
formed: on another stream, whose work is still queued, or at the same time from another
thread (each prediction by itself takes its turn).  Every result is that of a model of
its own, bit for bit."""
import threading

import numpy as np
import pytest
import torch

from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0
M, N, T = 60, 1500, 1600   # T N D = 4.2e9 at D = 1770: by the GEMMs


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


def geometries(n, seed):
    grid = 1.5 * np.stack(np.unravel_index(np.arange(M), (4, 4, 4)), axis=1)
    return torch.from_numpy(grid + 0.08 * np.random.Generator(np.random.PCG64([n, seed])).normal(size=(n, M, 3))).cuda()


def test_prediction_beside_a_product_on_another_stream(ctx):
    R, Rt = geometries(N, 1), geometries(T, 2)
    v = torch.from_numpy(np.random.Generator(np.random.PCG64(3)).normal(size=3 * M * N)).cuda()
    S, Te = ffk.descriptor_build(ctx, R, SIGMA), ffk.descriptor_build(ctx, Rt, SIGMA)
    busy, other = torch.cuda.Stream(), torch.cuda.Stream()
    a = torch.randn(8192, 8192, device="cuda")
    y = torch.empty(S.n, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        for _ in range(30):   # a quarter of a second
            b = a @ a
        ffk.kernel_mvm(ctx, S, v, y, stream=busy)
    with torch.cuda.stream(other):
        F = ffk.kernel_predict(ctx, S, Te, v, stream=other)
    torch.cuda.synchronize()
    S2 = ffk.descriptor_build(ctx, R, SIGMA)
    ref = ffk.kernel_predict(ctx, S2, Te, v)
    print("difference %.1e" % (F - ref).abs().max().item(), flush=True)
    assert torch.equal(F, ref)
    assert torch.equal(y, ffk.kernel_mvm(ctx, S2, v))
    del b


def test_predictions_and_columns_from_several_threads(ctx):
    R, Rt = geometries(N, 1), geometries(T, 2)
    v = torch.from_numpy(np.random.Generator(np.random.PCG64(3)).normal(size=3 * M * N)).cuda()
    cols = torch.arange(0, 3 * M * N, 2711, dtype=torch.int64, device="cuda")
    S, Te = ffk.descriptor_build(ctx, R, SIGMA), ffk.descriptor_build(ctx, Rt, SIGMA)
    torch.cuda.synchronize()
    out, streams = [None] * 6, [torch.cuda.Stream() for _ in range(6)]

    def work(i):
        with torch.cuda.stream(streams[i]):
            if i % 2:
                out[i] = ffk.kernel_columns(ctx, S, cols, stream=streams[i])
            else:
                out[i] = ffk.kernel_predict(ctx, S, Te, v, stream=streams[i])
            streams[i].synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    S2 = ffk.descriptor_build(ctx, R, SIGMA)
    ref = ffk.kernel_predict(ctx, S2, Te, v), ffk.kernel_columns(ctx, S2, cols)
    for i in range(6):
        assert torch.equal(out[i], ref[i % 2]), i
