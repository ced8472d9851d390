"""Predictions of many geometries from small models, whose batches are as large as 16 MB
of parts allow (512 before), against the oracle: batches at the limits, tiles of test
geometries beyond the places of an XCD with one chunk of training ones, one and two
batches, up to four and more chunks in the reduction.  FP64 operators: 1e-10 relative,
norm-wise.
"""
import numpy as np
import pytest
import torch

from oracle import kernel as ok
from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


def geometries(M, N, seed):
    grid = 1.5 * np.stack(np.unravel_index(np.arange(M), (3, 3, 3)), axis=1)
    return grid + 0.08 * np.random.Generator(np.random.PCG64([M, N, seed])).normal(size=(N, M, 3))


@pytest.mark.parametrize("M,N,T", [(3, 1, 513), (3, 5, 9000), (3, 5, 32769), (3, 5, 40000), (5, 64, 8193), (5, 65, 8225),
                                   (9, 100, 1537), (9, 257, 7000), (21, 40, 9100), (12, 1000, 2050)])
def test_many_tests_of_a_small_model(ctx, M, N, T):
    R, Rt = geometries(M, N, 1), geometries(M, T, 2)
    alpha = np.random.Generator(np.random.PCG64(N)).normal(size=3 * M * N)
    S = ffk.descriptor_build(ctx, torch.from_numpy(R).cuda(), SIGMA)
    Te = ffk.descriptor_build(ctx, torch.from_numpy(Rt).cuda(), SIGMA)
    F = ffk.kernel_predict(ctx, S, Te, torch.from_numpy(alpha).cuda()).cpu().numpy()
    rng = np.random.Generator(np.random.PCG64(T))
    rows = np.unique(np.concatenate([np.arange(20), rng.integers(0, T, size=300), np.arange(T - 40, T)]))
    ref = ok.kernel_mvm(Rt[rows], R, alpha, SIGMA).reshape(len(rows), -1)
    err = np.linalg.norm(F.reshape(T, -1)[rows] - ref) / np.linalg.norm(ref)
    print("prediction", M, N, T, "%.2e" % err, flush=True)
    assert np.isfinite(F).all() and err <= 1e-10


def test_time_of_many_tests(ctx):
    """M = 3, N = 5: 500 tests take 36 us, 4000 took 161 in eight batches, 48 in one."""
    S = ffk.descriptor_build(ctx, torch.from_numpy(geometries(3, 5, 1)).cuda(), SIGMA)
    Te = {T: ffk.descriptor_build(ctx, torch.from_numpy(geometries(3, T, 2)).cuda(), SIGMA) for T in (500, 4000)}
    alpha = torch.from_numpy(np.random.Generator(np.random.PCG64(1)).normal(size=45)).cuda()

    def us(T):
        t = []
        for _ in range(40):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ffk.kernel_predict(ctx, S, Te[T], alpha)
            b.record()
            b.synchronize()
            t.append(1000 * a.elapsed_time(b))
        return float(np.median(t[5:]))

    few, many = us(500), us(4000)
    print("500 tests %.1f us, 4000 tests %.1f us" % (few, many), flush=True)
    assert many < 3 * few
