"""GPU parity of the any-shape matrix products behind the MLP path: sizes on both sides of every tile edge, rows on odd
2-byte boundaries, contractions shorter than one 16-byte piece, each row-tile height, against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
from test_gpu_mlp import check_grads, make

pytestmark = pytest.mark.gpu

# one hidden layer, so that the tight gradient bar (1e-4 median, 2e-3 per worker and block) applies
SHAPES = [
    ([7, 5, 3], 2, 1),            # every contraction shorter than 8, one sample
    ([8, 64, 8], 3, 32),          # exactly one tile and one 16-byte piece
    ([9, 65, 2], 3, 33),          # one past the tile in every direction, two classes
    ([63, 130, 7], 2, 31),        # odd rows: every row of W starts on another 2-byte boundary
    ([136, 128, 16], 2, 64),      # multiples of 8 that are no multiples of a K step
    ([257, 191, 10], 12, 65),     # 32-row tiles (few of them), remainders in m, n and k
    ([129, 1100, 65], 16, 127),   # 128-row tile, classes past one column tile
    ([640, 2050, 10], 9, 130),    # five K steps, 128 x 128 forward tiles, two of rows
    ([383, 515, 100], 5, 300),
    ([96, 70, 33], 3, 32),        # classifier of 33 to 64 classes: 64-column head, one row tile,
    ([200, 150, 50], 4, 33),      # two,
    ([130, 257, 64], 5, 100),     # four, all columns used
    ([1030, 40, 10], 2, 33),      # hidden layer on 32 x 32 tiles of sixteen wavefronts: long contraction, few tiles
    ([2050, 33, 40], 3, 31),
    ([257, 1030, 100], 16, 50),   # 64-row tiles, forward and d-input (double sums every other instruction)
    ([300, 1030], 16, 50),        # logits of more than 64 classes: 64-row tiles
    ([137, 1030], 16, 130),       # ... 128-row tiles, two of them
    ([130, 300, 10], 16, 70),     # 32 rows: 64 columns where tiles fill the compute units once,
    ([257, 1500, 10], 12, 16),    # 32 where they would fill them twice,
    ([70, 1030, 10], 13, 33),     # 64 again beyond
    ([200, 490, 10], 20, 32),     # forward 64 where narrow tiles would be two on some units and one on others, d-input 32
]


@pytest.mark.parametrize("dims,W,B", SHAPES)
def test_ragged_grad_loss_matches_oracle(dims, W, B):
    pr, batch, Xb, y, P, _ = make(dims, W, B, seed=sum(dims) + B)
    pr.g.fill_(float("nan"))
    pr.ora.grad_loss_mlp(dims, Xb, y)
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    g = pr.g.cpu().numpy()
    check_grads(g[:, :P], pr.ora.g[:, :P], dims)
    assert np.all(g[:, P:] == 0)


@pytest.mark.parametrize("dims,W,B", [SHAPES[0], SHAPES[2], SHAPES[3], SHAPES[5], SHAPES[7], SHAPES[10], SHAPES[12], SHAPES[14]])
def test_ragged_fused_update_equals_the_three_call_step(dims, W, B):
    """The update inside the d-weight kernels against gradient + update: the same expression up to the rounding of
    its fused multiply-adds, element by element; nothing outside the parameters is written."""
    res = []
    for flags in (L.WRITE_BF16_SHADOW, L.WRITE_BF16_SHADOW | L.FUSED_MLP_UPDATE):
        pr, batch, _, _, P, _ = make(dims, W, B, seed=5, momentum=0.9, flags=flags)
        pr.x[:, P:] = 3.0
        pr.m[:, P:] = 4.0
        pr.pop.step(batch, 0.01, 0.1, 0.05)
        torch.cuda.synchronize()
        assert torch.all(pr.x[:, P:] == 3.0) and torch.all(pr.m[:, P:] == 4.0)
        assert torch.equal(pr.xb[:, :P], pr.x[:, :P].to(torch.bfloat16))
        res.append((pr.x[:, :P].clone(), pr.m[:, :P].clone(), pr.Z[:, :P].clone()))
    (x0, m0, z0), (x1, m1, z1) = res
    assert torch.equal(z0, z1)
    # m = g + pulls: a few roundings of terms no larger than max|m|; x moves by eta m
    assert (m1 - m0).abs().max() <= 8 * 2.0 ** -23 * m0.abs().max()
    assert (x1 - x0).abs().max() <= 2.0 ** -23 * x0.abs().max() + 0.01 * 8 * 2.0 ** -23 * m0.abs().max()
