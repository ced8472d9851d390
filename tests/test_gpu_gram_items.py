"""The Gram matrix of the preconditioner's factor where its items change: one
range of K and eight (n from 3900 to 4400), one tile and several, pieces of a
tile (one to sixteen), against the oracle's Woodbury form: 1e-9 norm-wise, the
applied preconditioner's bound at these condition numbers (lambda = 1e-2).
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ffk():
    from paper_2212_12737_amd import ffk as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def ctx(ffk):
    return ffk.create(0)


@pytest.mark.parametrize("M,N,k", [(9, 151, 60), (9, 152, 60), (10, 150, 129), (9, 160, 300), (6, 70, 140)])
def test_applied_preconditioner(ffk, ctx, M, N, k):
    print("gram", M, N, k, flush=True)
    R = synth.make_system(M, N, 0.08, True, 1200 + M, 1, 7).R
    S = ffk.descriptor_build(ctx, torch.as_tensor(R, device="cuda"), 10.0)
    lam = 1e-2
    idx = np.random.default_rng(k).permutation(S.n)[:k].astype(np.int64)
    P = ffk.precond_build(ctx, S, torch.as_tensor(idx, device="cuda"), lam)
    L = ffk.precond_export(ctx, P, S.n).cpu().numpy()
    r = synth.random_vectors(S.n, 5)
    z = ffk.precond_apply(ctx, P, torch.as_tensor(r, device="cuda")).cpu().numpy()
    ref = (r - L @ np.linalg.solve(lam * np.eye(L.shape[1]) + L.T @ L, L.T @ r)) / lam
    assert np.linalg.norm(z - ref) <= 1e-9 * np.linalg.norm(ref)
