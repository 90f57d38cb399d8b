"""GPU parity of the forward and d-input products whose operands go straight to LDS: one to nine K steps, last steps of
8 to 64 contraction indices, tiles cut in rows and columns, each tile shape, against the CPU oracle."""
import numpy as np
import pytest
import torch

from test_gpu_mlp import check_grads, make

pytestmark = pytest.mark.gpu

# one hidden layer, so that the tight gradient bar (1e-4 median, 2e-3 per worker and block) applies; more than 64 classes
# give the d-input product a contraction worth the name
SHAPES = [
    ([64, 128, 128], 2, 128),       # whole tiles: one K step forward, two back
    ([192, 320, 192], 3, 256),      # three; 64-column tiles
    ([256, 1024, 256], 20, 128),    # four; 128 x 128 tiles forward
    ([320, 4096, 64], 8, 256),      # five; 256 x 128 tiles
    ([576, 512, 576], 3, 384),      # nine
    ([136, 1096, 136], 16, 65),     # any sizes: last step of 8, one row past half a tile, 64-column tiles
    ([520, 1288, 520], 16, 129),    # 128-column tiles both ways, one row in the second row tile
    ([128, 2050, 10], 8, 127),      # two columns in the last tile, rows of the result on odd 4-byte boundaries
    ([1000, 1333, 10], 13, 300),    # odd width: rows of the result on any 2-byte boundary
    ([248, 1032, 1016], 16, 200),   # last steps of 56
]


@pytest.mark.parametrize("dims,W,B", SHAPES)
def test_direct_products_match_the_oracle(dims, W, B):
    pr, batch, Xb, y, P, _ = make(dims, W, B, seed=sum(dims) + B)
    pr.g.fill_(float("nan"))
    pr.ora.grad_loss_mlp(dims, Xb, y)
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    g = pr.g.cpu().numpy()
    check_grads(g[:, :P], pr.ora.g[:, :P], dims)
    assert np.all(g[:, P:] == 0)
