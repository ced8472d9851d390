"""A preconditioner is built where its factor and core fit the memory: the pieces of the
core's Gram product, several times the core's size, are then made in one piece a tile.

The core's sums come in another order then.  With lambda = 1 its condition is at most 1 +
trace(K) (some 1e4), so that z agrees to 1e4 eps sqrt(n) = 4e-10; the bound is 1e-9.
"""
import numpy as np
import pytest
import torch

from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0
MB = 1 << 20


def test_build_with_little_memory_left():
    M, N, k = 21, 600, 4000
    n, kp = 3 * M * N, 4096
    rng = np.random.Generator(np.random.PCG64(3))
    grid = 1.5 * np.stack(np.unravel_index(np.arange(M), (3, 3, 3)), axis=1)
    ctx = ffk.create(0)
    S = ffk.descriptor_build(ctx, torch.from_numpy(grid + 0.08 * rng.normal(size=(N, M, 3))).cuda(), SIGMA)
    idx = torch.from_numpy(rng.permutation(n)[:k].copy()).cuda()
    r = torch.from_numpy(rng.normal(size=n)).cuda()
    trace = float(ffk.kernel_diag(ctx, S).sum())
    assert trace < 1e4
    z = []
    for short in (False, True):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        # the factor (its columns padded to 128), the core, and 300 MB, less than the pieces of 528 tiles in
        # eight ranges (554 MB) and more than one of each (69 MB) or the core's inverse and its transpose
        need = 8 * ((n + 63) // 64 * 64 * kp + k * 4032) + 300 * MB
        hog = []
        while short and torch.cuda.mem_get_info()[0] > need + 16 * MB and len(hog) < 8:
            hog.append(torch.empty(torch.cuda.mem_get_info()[0] - need, dtype=torch.uint8, device="cuda"))
            torch.cuda.synchronize()
        print("free %d MB" % (torch.cuda.mem_get_info()[0] // MB), flush=True)
        P = ffk.precond_build(ctx, S, idx, 1.0)
        z.append(ffk.precond_apply(ctx, P, r).cpu().numpy())
        print("k_eff", P.k_eff, flush=True)
        del P, hog
    torch.cuda.empty_cache()
    err = np.linalg.norm(z[1] - z[0]) / np.linalg.norm(z[0])
    print("z differs by %.2e, trace %.0f" % (err, trace), flush=True)
    assert err <= 1e-9
