"""Exact leverage scores of systems of one to three 64-wide blocks (the inverse of one
block is a kernel by itself; of two, the first level of pairs; of three, an odd one out)
and preconditioners with as small a core, against the oracle.

tau = 1 - lambda |F^-1 e_c|^2 with K + lambda I of condition below 1e2 / 1e-4: 1e6 eps =
2e-10, bound 1e-9.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok
from oracle import select as osel
from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0
LAM = 1e-4


@pytest.fixture(scope="module")
def ctx():
    return ffk.create(0)


@pytest.mark.parametrize("M,N", [(3, 1), (5, 1), (7, 3), (21, 1), (3, 7), (22, 1), (3, 8), (42, 1), (43, 1), (9, 6)])
def test_labels_of_one_to_three_blocks(ctx, M, N):
    s = synth.make_system(M, N, 0.08, True, 600 + M, 601 + M, 602 + M)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    K = ok.dense_kernel(s.R, SIGMA)
    assert np.linalg.eigvalsh(K)[-1] < 1e2
    tau = ffk.exact_rls(ctx, S, LAM).cpu().numpy()
    err = np.abs(tau - osel.exact_ridge_leverage(K, LAM)).max()
    print("labels", M, N, "%.2e" % err, flush=True)
    assert err <= 1e-9


@pytest.mark.parametrize("k", [1, 2, 63, 64, 65, 129])
def test_preconditioner_of_one_to_three_blocks(ctx, k):
    s = synth.make_system(9, 30, 0.08, True, 650, 651, 652)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    idx = np.random.Generator(np.random.PCG64(k)).permutation(S.n)[:k]
    P = ffk.precond_build(ctx, S, torch.from_numpy(idx), LAM)
    L = ffk.precond_export(ctx, P, S.n).cpu().numpy()
    r = np.random.Generator(np.random.PCG64(1)).normal(size=S.n)
    z = ffk.precond_apply(ctx, P, torch.from_numpy(r).cuda()).cpu().numpy()
    ref = (r - L @ np.linalg.solve(L.T @ L + LAM * np.eye(P.k_eff), L.T @ r)) / LAM
    assert np.linalg.norm(z - ref) <= 1e-9 * np.linalg.norm(ref)
