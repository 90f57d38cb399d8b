"""GPU parity of the MLP launches that do the work of several: the classifier's with its d-input product (both sides of
each size up to which it takes that product along, remainders in samples, classes and units), and the d-weight products of
all layers in one launch (tile heights mixed, more layers than one launch takes, gradients and fused update)."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
from test_gpu_mlp import check_grads, make

pytestmark = pytest.mark.gpu

# one hidden layer, so that the tight gradient bar (1e-4 median, 2e-3 per worker and block) applies
SHAPES = [
    ([40, 1, 2], 2, 1), ([24, 31, 3], 3, 31), ([24, 33, 16], 3, 33), ([24, 513, 17], 3, 65),
    ([24, 767, 10], 5, 32), ([24, 768, 32], 5, 34), ([24, 769, 10], 5, 32),
    ([24, 255, 33], 4, 40), ([24, 256, 64], 4, 95), ([24, 257, 64], 4, 40),
    ([24, 256, 10], 3, 33), ([24, 257, 10], 3, 33), ([24, 300, 32], 3, 50),
    ([24, 1030, 10], 128, 34), ([24, 4096, 32], 16, 500),        # 256 workgroups: wider layers
    ([200, 300, 40], 16, 50), ([500, 2000, 10], 16, 33), ([64, 20, 65], 3, 50),
]
DEEP = [
    ([13, 50, 40, 70, 33, 60, 20, 45, 9], 3, 37),                # eight layers
    ([784, 300, 100, 10], 8, 50),
    ([128, 256, 128, 64, 10], 4, 128),                           # aligned and other tiles in one pass
]


@pytest.mark.parametrize("dims,W,B", SHAPES + DEEP)
def test_gradients_match_oracle(dims, W, B):
    pr, batch, Xb, y, P, _ = make(dims, W, B, seed=sum(dims) + B)
    pr.g.fill_(float("nan"))
    pr.ora.grad_loss_mlp(dims, Xb, y)
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    g = pr.g.cpu().numpy()
    check_grads(g[:, :P], pr.ora.g[:, :P], dims)
    assert np.all(g[:, P:] == 0)


@pytest.mark.parametrize("dims,W,B", [SHAPES[2], SHAPES[6], SHAPES[8], SHAPES[13]] + DEEP)
def test_fused_update_equals_the_three_call_step(dims, W, B):
    res = []
    for flags in (L.WRITE_BF16_SHADOW, L.WRITE_BF16_SHADOW | L.FUSED_MLP_UPDATE):
        pr, batch, _, _, P, _ = make(dims, W, B, seed=5, momentum=0.9, flags=flags)
        pr.x[:, P:] = 3.0
        pr.pop.step(batch, 0.01, 0.1, 0.05)
        torch.cuda.synchronize()
        assert torch.all(pr.x[:, P:] == 3.0)
        assert torch.equal(pr.xb[:, :P], pr.x[:, :P].to(torch.bfloat16))
        res.append((pr.x[:, :P].clone(), pr.m[:, :P].clone(), pr.Z[:, :P].clone()))
    (x0, m0, z0), (x1, m1, z1) = res
    assert torch.equal(z0, z1)
    # m = g + pulls: a few roundings of terms no larger than max|m|; x moves by eta m
    assert (m1 - m0).abs().max() <= 8 * 2.0 ** -23 * m0.abs().max()
    assert (x1 - x0).abs().max() <= 2.0 ** -23 * x0.abs().max() + 0.01 * 8 * 2.0 ** -23 * m0.abs().max()


def test_infinite_weight_past_the_last_class_stays_out():
    """Three classes on tiles of sixteen: what follows the classifier's weights in memory takes no part."""
    dims, W, B = [16, 48, 3], 2, 20
    pr, batch, Xb, y, P, _ = make(dims, W, B, seed=1)
    pr.pop.sync_shadow()                                         # or the gradient call writes the copy anew
    pr.xb[:, P - 3:] = float("inf")                              # the classifier's biases are read in fp32
    pr.ora.grad_loss_mlp(dims, Xb, y)
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    assert torch.all(torch.isinf(pr.xb[:, P - 3:P]))
    assert torch.all(torch.isfinite(pr.g[:, :P]))
    check_grads(pr.g.cpu().numpy()[:, :P], pr.ora.g[:, :P], dims)
