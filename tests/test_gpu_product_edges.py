"""FP64 and FP32 products where the K loops of their GEMMs are shortest and
odd: one chunk of 64 bytes to a few, a last stage of one chunk, segment and
split boundaries inside a stage, and every column tile (D of 3 to 435); and
where FP64 changes between one kernel and the GEMMs (256, 512 and 1024
geometries, D of 128, fewer columns than chunks), against the oracle at the operators' bounds (1e-10 and 1e-6 norm-wise).
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok

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


@pytest.mark.parametrize("M,N", [(3, 1), (3, 8), (4, 9), (5, 17), (6, 25), (8, 63), (9, 65), (11, 100), (13, 129), (15, 200),
                                 (21, 130), (30, 41), (16, 513), (21, 300), (14, 700), (12, 1300), (21, 1300),
                                 (5, 250), (6, 256), (7, 257), (17, 512), (17, 513), (16, 1024), (16, 1025), (17, 1024)])
@pytest.mark.parametrize("prec,tol", [("FP64", 1e-10), ("FP32", 1e-6)])
def test_product_at_k_loop_edges(ffk, ctx, M, N, prec, tol):
    print("product", M, N, prec, flush=True)
    R = synth.make_system(M, N, 0.08, True, 1100 + M, 1, 7).R
    v = synth.random_vectors(3 * M * N, 9)
    S = ffk.descriptor_build(ctx, torch.as_tensor(R, device="cuda"), SIGMA)
    vd = torch.as_tensor(v, device="cuda")
    y = ffk.kernel_mvm(ctx, S, vd, prec=getattr(ffk, prec))
    for _ in range(3):   # and the same bits each time
        assert torch.equal(ffk.kernel_mvm(ctx, S, vd, prec=getattr(ffk, prec)), y)
    ref = ok.kernel_mvm(R, R, v, SIGMA)
    assert np.linalg.norm(y.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)
