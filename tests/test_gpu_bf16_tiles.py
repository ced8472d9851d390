"""BF16 and split-BF16 products up to a few thousand geometries where their tiles change:
descriptor widths around multiples of the 128-column tile, one geometry to a
few tiles of 64, and both sides of the rules that choose the wide GEMM 2 tile
and the tall GEMM 1 tile; against the library's FP64 product at the operators'
bounds (1e-6 and 3e-3 norm-wise), the same bits each time.
"""
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N", [(17, 1), (17, 63), (17, 64), (17, 65), (23, 257), (24, 130), (28, 333), (33, 64), (17, 1500),
                                 (25, 1500), (35, 2500), (56, 800), (33, 2000), (17, 2816), (17, 2817), (24, 4095),
                                 (24, 4096), (17, 4200), (32, 4353), (33, 4353)])
def test_product_at_tile_edges(M, N):
    from paper_2212_12737_amd import ffk
    ctx = ffk.create(0)
    R = torch.as_tensor(synth.make_system(M, N, 0.08, True, 1200 + M, 1, 7).R, device="cuda")
    v = torch.as_tensor(synth.random_vectors(3 * M * N, 9), device="cuda")
    S = ffk.descriptor_build(ctx, R, 10.0)
    ref = ffk.kernel_mvm(ctx, S, v)
    for prec, tol in ((ffk.BF16X3, 1e-6), (ffk.BF16, 3e-3)):
        print("product", M, N, prec, flush=True)
        y = ffk.kernel_mvm(ctx, S, v, prec=prec)
        assert float((y - ref).norm()) <= tol * float(ref.norm())
        assert torch.equal(ffk.kernel_mvm(ctx, S, v, prec=prec), y)
