"""Few kernel columns (a wave per target and column) against the oracle and against
many (64 columns a wave): both sides of the rule that chooses, 4 to 24 columns, at
molecules around it, one and several waves of atoms, a permuted source, and the most
columns of a target block.  FP64 operators: 1e-10 relative, norm-wise.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok
from oracle import symmetry as osym
from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


def system(M, N):
    return synth.make_system(M, N, 0.08, True, 700 + M, 701 + M, 702 + M)


@pytest.mark.parametrize("M,N", [(3, 1), (3, 14), (7, 9), (8, 9), (9, 13), (21, 5), (66, 2)])
def test_columns_on_both_sides_of_the_rule(ctx, M, N):
    s = system(M, N)
    K = ok.dense_kernel(s.R, SIGMA)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    rng = np.random.Generator(np.random.PCG64([M, N]))
    for k in (1, 2, 4, 5, 12, 13, 16, 17, 24, 25, 32, 33, 48, 49):
        cols = rng.integers(0, S.n, size=k)
        C = ffk.kernel_columns(ctx, S, torch.from_numpy(cols)).cpu().numpy()
        err = np.linalg.norm(C - K[:, cols]) / np.linalg.norm(K[:, cols])
        print("columns", M, N, k, "%.2e" % err, flush=True)
        assert err <= 1e-10


@pytest.mark.parametrize("k", [1, 4, 16, 17])
def test_columns_of_a_symmetrized_kernel(ctx, k):
    s = system(9, 11)
    perms = np.array([[0, 1, 2, 3, 4, 5, 6, 7, 8], [0, 1, 2, 3, 4, 5, 7, 8, 6], [0, 1, 2, 3, 4, 5, 8, 6, 7]])
    K = osym.dense_sym_kernel(s.R, perms, SIGMA)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    ffk.set_symmetries(ctx, S, perms)
    cols = np.random.Generator(np.random.PCG64(k)).integers(0, S.n, size=k)
    C = ffk.kernel_columns(ctx, S, torch.from_numpy(cols)).cpu().numpy()
    assert np.linalg.norm(C - K[:, cols]) <= 1e-10 * np.linalg.norm(K[:, cols])


def test_one_column_costs_less_than_a_tile_of_them(ctx):
    """One column used to cost what 64 do (304 and 381 us at this size); 80 us now."""
    M, N = 30, 5000
    rng = np.random.Generator(np.random.PCG64(5))
    grid = 1.5 * np.stack(np.unravel_index(np.arange(M), (4, 4, 2)), axis=1)
    S = ffk.descriptor_build(ctx, torch.from_numpy(grid + 0.05 * rng.normal(size=(N, M, 3))).cuda(), SIGMA)

    def seconds(k):
        cols = torch.from_numpy(rng.permutation(S.n)[:k].copy()).cuda()
        t = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ffk.kernel_columns(ctx, S, cols)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return float(np.median(t[2:]))

    one, tile = seconds(1), seconds(64)
    print("one column %.3f ms, 64 columns %.3f ms" % (one, tile), flush=True)
    assert one < 0.6 * tile
