"""The dense FP64 factorizations at the edges of their blocks (16, 64, 256) and
with odd orders: exact leverage scores (Cholesky and triangular inverse) and
the incomplete Cholesky factor, against the FP64 oracle.

Tolerances.  Scores: 1 - lambda |F^-1 e_c|^2 of a matrix of condition number
kappa carries an error of order n eps kappa at worst; lambda = 1e-3 keeps
kappa below 1e4, and the repository's bound for FP64 operators at moderate
conditioning, 1e-10, holds with two digits to spare.  Factor: 1e-10 of its norm.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok
from oracle import select as osel

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


def system(ffk, ctx, M, N, seed):
    s = synth.make_system(M, N, 0.08, True, seed, seed + 1, seed + 2)
    return s.R, ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)


# n = 9, 36, 63, 189, 255, 261, 513, 765, 774, 1287
@pytest.mark.parametrize("M,N", [(3, 1), (4, 3), (7, 3), (9, 7), (5, 17), (3, 29), (9, 19), (5, 51), (6, 43), (11, 39)])
def test_exact_leverage_scores_at_block_edges(ffk, ctx, M, N):
    print("rls", M, N, flush=True)
    R, S = system(ffk, ctx, M, N, 900 + M)
    lam = 1e-3
    tau = ffk.exact_rls(ctx, S, lam).cpu().numpy()
    ref = osel.exact_ridge_leverage(ok.dense_kernel(R, SIGMA), lam)
    assert np.abs(tau - ref).max() <= 1e-10


@pytest.mark.parametrize("M,N,k", [(5, 17, 1), (5, 17, 15), (5, 17, 17), (7, 21, 63), (7, 21, 65), (9, 41, 129),
                                   (9, 41, 255), (9, 41, 257), (8, 60, 321)])
def test_incomplete_factor_at_panel_edges(ffk, ctx, M, N, k):
    print("icd", M, N, k, flush=True)
    R, S = system(ffk, ctx, M, N, 930 + M)
    idx = np.random.default_rng(k).permutation(S.n)[:k].astype(np.int64)
    P = ffk.precond_build(ctx, S, torch.as_tensor(idx, device="cuda"), 1e-6)
    assert P.k_eff == k
    L = ffk.precond_export(ctx, P, S.n).cpu().numpy()
    K = ok.dense_kernel(R, SIGMA)
    ref = osel.incomplete_cholesky(lambda c: K[:, c], np.diag(K), k, order=idx)[0]
    assert np.linalg.norm(L - ref) <= 1e-10 * np.linalg.norm(ref)
