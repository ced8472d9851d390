"""Coefficients of a system's pairs at the line between the small tiles and the pipelined
engine (2048^2 pairs for short rows, 1536^2 for longer ones): products against the oracle
on some of the rows, FP64 1e-10 relative, norm-wise; and below the line a system that
has not multiplied holds no padded copy of its descriptor.
"""
import numpy as np
import pytest
import torch

from oracle import kernel as ok
from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0
MB = 1 << 20


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


def geometries(M, N, seed=0):
    grid = 1.5 * np.stack(np.unravel_index(np.arange(M), (4, 4, 4)), axis=1)
    return grid + 0.08 * np.random.Generator(np.random.PCG64([M, N, seed])).normal(size=(N, M, 3))


@pytest.mark.parametrize("M,N", [(3, 1025), (30, 2048), (30, 2049), (31, 1536), (31, 1537), (17, 1793), (40, 1281)])
def test_product_rows(ctx, M, N):
    R = geometries(M, N)
    S = ffk.descriptor_build(ctx, torch.from_numpy(R).cuda(), SIGMA)
    v = np.random.Generator(np.random.PCG64(N)).normal(size=S.n)
    rows = np.unique(np.concatenate([np.arange(17), np.random.Generator(np.random.PCG64(M)).integers(0, N, size=32),
                                     np.arange(N - 17, N)]))
    ref = ok.kernel_mvm(R[rows], R, v, SIGMA).reshape(len(rows), -1)
    y = ffk.kernel_mvm(ctx, S, torch.from_numpy(v).cuda()).cpu().numpy().reshape(N, -1)
    err = np.linalg.norm(y[rows] - ref) / np.linalg.norm(ref)
    print("product", M, N, "%.2e" % err, flush=True)
    assert np.isfinite(y).all() and err <= 1e-10


@pytest.mark.parametrize("M,N", [(30, 2048), (60, 1536)])
def test_no_padded_copy_before_a_product(ctx, M, N):
    R = torch.from_numpy(geometries(M, N)).cuda()
    D = M * (M - 1) // 2

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    kept = [ffk.descriptor_build(ctx, R, SIGMA) for _ in range(2)]   # memory that the runtime keeps is in use then
    before = free()
    kept += [ffk.descriptor_build(ctx, R, SIGMA) for _ in range(4)]
    used = (before - free()) / 4
    need = 8 * (R.numel() + 2 * N * D + 2 * N ** 2)   # geometries, descriptor, its centred copy, two coefficient matrices
    padded = 8 * N * (D + 63) // 64 * 64
    print("held: %.1f MB, needed %.1f MB, padded copy %.1f MB" % (used / MB, need / MB, padded / MB), flush=True)
    assert used <= need + padded / 2
