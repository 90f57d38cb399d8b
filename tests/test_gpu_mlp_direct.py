"""GPU parity of the forward and d-input products whose operands go straight to LDS: three to nine K steps (whole tiles of one or
two go through registers), last steps of 8 to 64 contraction indices, tiles cut in rows and columns, each tile shape, against
the CPU oracle; and what large weights and gradients change, against populations of one worker."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
import workloads as wl
from test_gpu_mlp import check_grads, make

pytestmark = pytest.mark.gpu

# one hidden layer, so that the tight gradient bar (1e-4 median, 2e-3 per worker and block) applies; more than 64 classes
# give the d-input product a contraction worth the name
SHAPES = [
    ([64, 128, 128], 2, 128),       # whole tiles: one K step forward, two back: through registers
    ([192, 320, 192], 3, 256),      # three: straight to LDS; 64-column tiles
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


def population(x, dims, X, y):
    W, P = x.shape
    ld = wl.padded_ld(P)
    xd = torch.zeros((W, ld), device="cuda")
    xd[:, :P] = x
    g, xb = torch.full_like(xd, float("nan")), torch.zeros((W, ld), dtype=torch.bfloat16, device="cuda")
    batch = L.MLPBatch(dims, X, y)
    return L.Population(xd, g, 1, x_bf16=xb, P=P, largest_batch=batch), batch, g


# more than 120 MB of weights in one layer, one row tile: read past the caches, straight to LDS and (more tiles than compute units)
# through registers; any size, with a d-weight product that is launched alone; gradients of one K step above 240 MB; fp32 inputs
# that a launch converts although the batch is small
@pytest.mark.parametrize("W,B,dims,f32", [(8, 128, [2048, 4096, 10], False), (16, 128, [1024, 4096, 10], False), (8, 100, [3000, 2600, 10], False),
                                          (16, 32, [2048, 2048, 10], False), (16, 32, [2048, 3072, 10], True)])
def test_large_layers_equal_populations_of_one(W, B, dims, f32):
    """Every worker by itself takes the other ways: the sums are the same but for the order of additions inside a tile."""
    P = sum(a * b + b for a, b in zip(dims, dims[1:]))
    gen = torch.Generator(device="cuda").manual_seed(W + B)
    x = torch.empty((W, P), device="cuda").normal_(std=0.02, generator=gen)
    X = torch.randn((W, B, dims[0]), device="cuda", generator=gen)
    X = X if f32 else X.to(torch.bfloat16)
    y = torch.randint(0, dims[-1], (W, B), device="cuda", generator=gen, dtype=torch.int32)
    pop, batch, g = population(x, dims, X, y)
    pop.grad_loss(batch)
    grad_losses, loss = pop.get_losses(), torch.zeros(W, device="cuda")
    pop.loss(batch, loss)
    assert grad_losses == loss.tolist()
    for w in (0, W // 2, W - 1):
        one, b1, g1 = population(x[w:w + 1], dims, X[w:w + 1].contiguous(), y[w:w + 1].contiguous())
        one.grad_loss(b1)
        np.testing.assert_allclose(grad_losses[w], one.get_losses()[0], rtol=1e-5)
        # (an activation on another side of a bf16 boundary: 2^-9 of it, in few places)
        assert (g[w, :P] - g1[0, :P]).norm() <= 2e-3 * g1[0, :P].norm()
    assert torch.all(g[:, P:] == 0)
