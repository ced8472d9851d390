"""Descriptors of few geometries where their one kernel ends (8 geometries, 8192
elements): the rows themselves to 4 ulp (a subtraction, three products, a root
and a divide), the product's mean and norms through K v against the oracle at the
FP64 operators' 1e-10, and a coincident pair refused on either side.
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


CASES = [(3, 1), (3, 8), (3, 9), (21, 1), (45, 8), (46, 8), (128, 1), (129, 1)]


@pytest.mark.parametrize("M,N", CASES)
def test_rows_and_product(ffk, ctx, M, N):
    print("few", M, N, flush=True)
    R = synth.make_system(M, N, 0.08, True, 1300 + M, 1, 7).R
    S = ffk.descriptor_build(ctx, torch.as_tensor(R, device="cuda"), 10.0)
    p, q = np.tril_indices(M, -1)
    x = 1.0 / np.sqrt(((R[:, p] - R[:, q]) ** 2).sum(-1))
    X = ffk.descriptor_export(ctx, S).cpu().numpy()
    assert (np.abs(X - x) <= 4 * np.spacing(x)).all()
    v = synth.random_vectors(S.n, 3)
    y = ffk.kernel_mvm(ctx, S, torch.as_tensor(v, device="cuda"), shift=0.5).cpu().numpy()
    ref = ok.kernel_mvm(R, R, v, 10.0) + 0.5 * v
    assert np.linalg.norm(y - ref) <= 1e-10 * np.linalg.norm(ref)


@pytest.mark.parametrize("M,N", [(4, 3), (4, 40)])
def test_coincident_atoms_are_refused_and_leave_no_trace(ffk, ctx, M, N):
    R = synth.make_system(M, N, 0.08, True, 1400 + M, 1, 7).R
    bad = R.copy()
    bad[N - 1, 2] = bad[N - 1, 1]
    with pytest.raises(ffk.FfkError):
        ffk.descriptor_build(ctx, torch.as_tensor(bad, device="cuda"), 10.0)
    ffk.descriptor_build(ctx, torch.as_tensor(R, device="cuda"), 10.0)
