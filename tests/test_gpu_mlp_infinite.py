"""An infinite error of the last row of a batch reaches the gradient as infinities, not as
NaN from the steps past the batch's end (batches that do not fill a step of 16)."""
import numpy as np
import pytest
import torch

from paper_2212_12737_amd import ffk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 70, 1030])
def test_infinite_error_of_the_last_row(B):
    D, H = 9, 64
    ctx = ffk.create(0)
    net = ffk.mlp_create(ctx, D, H, 3)
    g = torch.Generator().manual_seed(B)
    X, y = torch.randn(B, D, generator=g), torch.randn(B, generator=g)
    y[-1] = np.inf
    loss, grad = ffk.mlp_grad(ctx, net, X.cuda(), y.cuda())
    theta = ffk.mlp_get_params(ctx, net).cpu().double()
    W1, b1, W2, b2, w3, b3 = torch.split(theta, [H * D, H, H * H, H, H, 1])
    h1 = torch.nn.functional.gelu(X.double() @ W1.reshape(H, D).T + b1)
    z2 = h1 @ W2.reshape(H, H).T + b2
    z = z2.clone().requires_grad_()
    torch.nn.functional.gelu(z).sum().backward()
    # g_W2[i, j] = sum_b dout_b w3_i gelu'(z2_bi) h1_bj, with dout = -inf in the last row only
    sign = -torch.sign(w3 * z.grad[-1])[:, None] * torch.sign(h1[-1])[None, :]
    gW2 = grad.cpu()[H * D + H:H * D + H + H * H].reshape(H, H)
    print("B", B, "NaN", int(torch.isnan(gW2).sum()), flush=True)
    assert torch.isinf(loss).all()
    assert torch.equal(gW2.double(), sign * np.inf)
