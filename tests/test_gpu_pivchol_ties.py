"""Exact ties in the blocks of the pivoted-Cholesky selection go to the lowest index.

Geometries whose diagonals tie exactly and whose kernel blocks do not touch: three
atoms on a line at 0, 1 and c and, 1e5 away, a pair of spectators whose distance
differs from geometry to geometry.  The spectators' terms vanish in the rounding of
the other atoms' diagonals (1e-20 of them), and with a length scale far below the
descriptors' differences every entry between two geometries is exactly zero
(exp(-z) at z > 745).  So Algorithm 1 takes the middle atoms' x rows of all geometries
first, in the order of their indices, then one end atom's x row of each (the ends'
remaining diagonals are equal but for rounding, the same in every geometry), again in
order.
"""
import numpy as np
import pytest
import torch

from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu

M = 5


def tied_geometries(G, c):
    R = np.zeros((G, M, 3))
    R[:, 1, 0], R[:, 2, 0] = 1.0, c
    R[:, 3:, 1] = 1e5
    R[:, 4, 0] = 10.0 + 0.01 * np.arange(G)
    return R


@pytest.mark.parametrize("c,sigma", [(2.0, 1e-7), (3.0, 1e-7), (3.0, 1.005e-7)])
@pytest.mark.parametrize("G,k", [(104, 200), (104, 208), (70, 140), (64, 128), (90, 170), (128, 250), (300, 590)])
def test_tied_rows_in_order(c, sigma, G, k):
    """G = 104: after 64 pivots one at a time, the pool holds end rows of the last 40
    geometries; then 208 rows tie, more than the pool can list, and those that it
    holds are not the lowest ones.  The other sizes: ties that fit the pool, none left
    of the first kind after the single pivots, more than twice the pool."""
    ctx = ffk.create(0)
    S = ffk.descriptor_build(ctx, torch.from_numpy(tied_geometries(G, c)).cuda(), sigma)
    d = ffk.kernel_diag(ctx, S).cpu().numpy().reshape(G, M, 3)
    assert (d[:, :3, 0] == d[0, :3, 0]).all() and np.argmax(d[0].reshape(-1)) == 3
    K = ffk.kernel_columns(ctx, S, torch.arange(3 * M, 6 * M)).cpu().numpy()
    assert not K[:3 * M].any() and not K[6 * M:].any()
    piv = ffk.nystrom_select(ctx, S, "pivchol", k).cpu().numpy()
    print("tied rows", c, sigma, G, k, piv[G:G + 4], flush=True)
    assert len(piv) == k
    assert (piv[:G] == 3 * M * np.arange(G) + 3).all()
    assert (piv[G:] // (3 * M) == np.arange(k - G)).all()
    assert set((piv[G:] % (3 * M)).tolist()) <= {0, 6}
