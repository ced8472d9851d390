"""Pivoted-Cholesky selection in blocks at many rows (n >= 32768, whose first 112 pivots
go one at a time) and of several hundred pivots, against the oracle's columns.

Every pivot has to be the largest remaining diagonal of the oracle's own elimination
with the pivots so far, to 1e-9 relative (a near-tie, where rounding decides) and 4 m eps
max diag K of rounding after m steps.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok
from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0


@pytest.mark.parametrize("M,N,k", [(11, 993, 113), (11, 993, 145), (11, 1000, 400), (21, 530, 330), (5, 2300, 300)])
def test_pivots_are_greedy(M, N, k):
    s = synth.make_system(M, N, 0.08, True, 860 + M, 861 + M, 862 + M)
    ctx = ffk.create(0)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    piv = ffk.nystrom_select(ctx, S, "pivchol", k).cpu().numpy()
    print("pivchol", M, N, S.n, len(piv), flush=True)
    assert len(piv) == k and len(set(piv.tolist())) == k
    C = ok.kernel_columns(s.R, piv, SIGMA)
    d = ok.kernel_diag(s.R, SIGMA).reshape(-1).copy()
    assert int(piv[0]) == int(np.argmax(d))
    slack = 4 * k * 2.0 ** -53 * d.max()
    L = np.zeros((S.n, k))
    free = np.ones(S.n, bool)
    for m, p in enumerate(piv):
        best = d[free].max()
        assert free[p] and d[p] >= best - 1e-9 * best - slack, (m, int(p), d[p], best)
        col = (C[:, m] - L[:, :m] @ L[p, :m]) / np.sqrt(d[p])
        col[~free] = 0.0
        L[:, m] = col
        d -= col * col
        free[p] = False
