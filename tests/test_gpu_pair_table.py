"""The pair table (32 bytes a pair and geometry) is formed when columns ask for it, and
not where it would be a large part of the free memory: a system that only multiplies
does not carry it, and columns and selections of a system without it are the same."""
import numpy as np
import pytest
import torch

from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0
MB = 1 << 20


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


def geometries(M, N):
    rng = np.random.Generator(np.random.PCG64([M, N]))
    grid = 1.5 * np.stack(np.unravel_index(np.arange(M), (4, 4, 4)), axis=1) + rng.uniform(-0.2, 0.2, size=(M, 3))
    return torch.from_numpy(grid + 0.08 * rng.normal(size=(N, M, 3))).cuda()


def free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_a_built_system_holds_no_pair_table(ctx):
    M, N = 60, 2000
    D, table = M * (M - 1) // 2, 32 * N * M * (M - 1) // 2
    R = geometries(M, N)
    ffk.descriptor_build(ctx, R[:4], SIGMA)
    before = free()
    S = ffk.descriptor_build(ctx, R, SIGMA)
    used = before - free()
    # geometries, descriptor, its centred copy and that padded, two coefficient matrices
    need = 8 * (R.numel() + 2 * N * D + 2048 * 1792 + 2 * 2048 ** 2)
    print("built: %d MB, needed %d MB, table %d MB" % (used // MB, need // MB, table // MB), flush=True)
    assert used <= need + 24 * MB < need + table
    before = free()
    ffk.set_symmetries(ctx, S, [list(range(M)), list(range(M - 2)) + [M - 1, M - 2]])
    used = before - free()
    need = 2 * 2 * 8 * (R.numel() + 2 * N * D) + 8 * R.numel()   # two copies and their stack, and a work vector
    print("symmetrized: %d MB, needed %d MB" % (used // MB, need // MB), flush=True)
    assert used <= need + 48 * MB < need + 4 * table


def test_columns_and_pivots_without_the_table(ctx):
    M, N, k = 60, 3000, 150
    table = 32 * N * M * (M - 1) // 2
    R = geometries(M, N)
    cols = torch.from_numpy(np.random.Generator(np.random.PCG64(1)).permutation(3 * M * N)[:70].copy()).cuda()
    out = []
    for short in (False, True):
        S = ffk.descriptor_build(ctx, R, SIGMA)
        torch.cuda.empty_cache()
        hog = torch.empty(free() - 14 * table, dtype=torch.uint8, device="cuda") if short else None
        print("free %d MB, table %d MB" % (free() // MB, table // MB), flush=True)
        before = free()
        C = ffk.kernel_columns(ctx, S, cols).t().clone()
        formed = before - free() > table + 2 * 8 * C.numel()
        assert not (short and formed)
        out.append((C.cpu().numpy(), ffk.nystrom_select(ctx, S, "pivchol", k).cpu().numpy()))
        del C, S, hog
        torch.cuda.empty_cache()
    err = np.abs(out[0][0] - out[1][0]).max() / np.abs(out[0][0]).max()
    print("columns differ by %.2e" % err, flush=True)
    assert err <= 1e-14   # FP64 sums of M = 60 terms in another order: 60 * 2^-53
    assert (out[0][1] == out[1][1]).all()
