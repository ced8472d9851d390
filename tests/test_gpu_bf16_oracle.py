"""BF16 and split-BF16 products on every tile the rules choose, against the oracle on some
of the rows: 64 x 64 and 128 x 64 tiles of GEMM 1, 64 x 128 and 128 x 128 of GEMM 2 below
4096 geometries, 128 x 64 and 256-wide ones above.  Tolerances of the other product
tests: 1e-6 (split BF16) and 3e-3 (BF16) relative, norm-wise.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import kernel as ok
from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

SIGMA = 10.0


@pytest.mark.parametrize("M,N", [(17, 65), (21, 2000), (35, 2501), (45, 1200), (26, 4095), (18, 4654), (33, 4353)])
def test_product_rows(M, N):
    s = synth.make_system(M, N, 0.08, True, 760 + M, 761 + M, 762 + M)
    ctx = ffk.create(0)
    S = ffk.descriptor_build(ctx, torch.as_tensor(s.R, device="cuda"), SIGMA)
    v = np.random.Generator(np.random.PCG64([M, N])).normal(size=S.n)
    rows = np.unique(np.concatenate([np.arange(4), np.random.Generator(np.random.PCG64(N)).integers(0, N, size=48),
                                     np.arange(N - 4, N)]))
    ref = ok.kernel_mvm(s.R[rows], s.R, v, SIGMA).reshape(len(rows), -1)
    vd = torch.from_numpy(v).cuda()
    for prec, tol in ((ffk.BF16X3, 1e-6), (ffk.BF16, 3e-3)):
        y = ffk.kernel_mvm(ctx, S, vd, prec=prec).cpu().numpy().reshape(N, -1)
        err = np.linalg.norm(y[rows] - ref) / np.linalg.norm(ref)
        print("product", M, N, prec, "%.2e" % err, flush=True)
        assert np.isfinite(y).all() and err <= tol
