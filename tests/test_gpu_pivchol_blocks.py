"""Pivoted-Cholesky selection in blocks of pivots against Algorithm 1 of the oracle.

Sizes where the blocks can go wrong: fewer rows than candidates, one column,
more columns than one block or one 32-wide panel accepts, odd n, exact ties
(repeated geometries), more columns than the numerical rank, a symmetrized
kernel.  Every pivot has to be the largest remaining diagonal of the oracle's own
elimination with the pivots so far, to 1e-9 relative (a near-tie, where rounding
decides) and the rounding that both sides' diagonals carry after m steps, 4 m eps
max diag K (each step rounds a diagonal at most twice).
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok
from oracle import symmetry as osym

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


def check_greedy(K, piv, k):
    """Every pivot is a largest remaining diagonal of K given the ones before it."""
    n = K.shape[0]
    d = np.diag(K).copy()
    thr, slack = 1e-12 * d.max(), 4 * max(len(piv), 1) * 2.0 ** -53 * d.max()
    L = np.zeros((n, len(piv)))
    free = np.ones(n, bool)
    for m, p in enumerate(piv):
        best = d[free].max()
        assert free[p] and d[p] > thr - slack
        assert d[p] >= best - 1e-9 * best - slack, (m, p, d[p], best)
        if m == 0:
            assert p == int(np.argmax(d))
        col = (K[:, p] - L[:, :m] @ L[p, :m]) / np.sqrt(d[p])
        col[~free] = 0.0
        L[:, m] = col
        d -= col * col
        free[p] = False
    if len(piv) < k:
        assert d[free].max() <= thr + slack


@pytest.mark.parametrize("M,N,k", [(3, 1, 1), (4, 5, 40), (5, 41, 1), (5, 41, 33), (7, 61, 127), (7, 61, 129),
                                   (9, 80, 300), (12, 57, 500), (6, 30, 520)])
def test_blocked_pivots_are_greedy(ffk, ctx, M, N, k):
    print("pivchol", M, N, k, flush=True)
    s = synth.make_system(M, N, 0.08, True, 960 + M, 961 + M, 962 + M)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    piv = ffk.nystrom_select(ctx, S, "pivchol", min(k, S.n)).cpu().numpy()
    assert len(piv) <= k and len(set(piv.tolist())) == len(piv)
    check_greedy(ok.dense_kernel(s.R, SIGMA), piv, min(k, S.n))


def test_exact_ties_take_the_lower_index(ffk, ctx):
    s = synth.make_system(6, 12, 0.08, True, 980, 981, 982)
    R = np.concatenate([s.R, s.R, s.R])          # every diagonal three times
    S = ffk.descriptor_build(ctx, torch.as_tensor(R, device="cuda"), SIGMA)
    piv = ffk.nystrom_select(ctx, S, "pivchol", 60).cpu().numpy()
    first = len(s.R) * 18
    assert (piv[:20] < first).all()
    check_greedy(ok.dense_kernel(R, SIGMA), piv, 60)


def test_symmetrized_kernel(ffk, ctx):
    s = synth.make_system(6, 20, 0.08, True, 985, 986, 987)
    perms = np.array([[0, 1, 2, 3, 4, 5], [0, 1, 2, 3, 5, 4]])
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    ffk.set_symmetries(ctx, S, perms)
    piv = ffk.nystrom_select(ctx, S, "pivchol", 150).cpu().numpy()
    check_greedy(osym.dense_sym_kernel(s.R, perms, SIGMA), piv, 150)


@pytest.mark.parametrize("M,N,k", [(21, 3, 17), (22, 3, 16), (22, 5, 33), (43, 2, 31)])
def test_single_pivots_of_large_molecules(ffk, ctx, M, N, k):
    """Rows of one to three waves a geometry, columns of L around a batch of sixteen."""
    print("pivchol singles", M, N, k, flush=True)
    s = synth.make_system(M, N, 0.08, True, 990 + M, 991 + M, 992 + M)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    piv = ffk.nystrom_select(ctx, S, "pivchol", k).cpu().numpy()
    assert len(piv) <= k and len(set(piv.tolist())) == len(piv)
    check_greedy(ok.dense_kernel(s.R, SIGMA), piv, k)
