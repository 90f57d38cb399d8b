"""Inputs in fp32 that the first product converts as it goes: bit for bit the results of the same values handed over in
bf16, at rows of any length and alignment, and on both sides of the sizes where a launch converts them first."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
from test_gpu_mlp import make

pytestmark = pytest.mark.gpu

SHAPES = [([8, 70, 4], 3, 5), ([9, 64, 10], 2, 1), ([7, 40, 3], 3, 33), ([15, 33, 20, 2], 5, 31), ([130, 65, 10], 4, 33),
          ([784, 300, 100, 10], 8, 50), ([617, 132, 10], 3, 64), ([1030, 40, 10], 2, 33), ([129, 600, 70], 8, 70),
          ([256, 128, 10], 3, 128), ([96, 64], 3, 20), ([200, 1030, 10], 16, 50), ([100, 300, 10], 16, 70),
          ([64, 1500, 10], 12, 16), ([200, 490, 10], 20, 32)]


@pytest.mark.parametrize("dims,W,B", SHAPES)
def test_same_bits_as_from_bf16_inputs(dims, W, B):
    res = []
    for f32 in (False, True):
        pr, batch, Xb, y, P, _ = make(dims, W, B, seed=sum(dims) + B)
        X = torch.from_numpy(Xb.view(np.int16)).view(torch.bfloat16).cuda()
        if f32:
            # values between the bf16 ones that round to them (a quarter of a step off)
            Xf = X.float() * (1.0 + 2.0 ** -11)
            assert torch.equal(Xf.to(torch.bfloat16), X)
            batch = L.MLPBatch(dims, Xf.contiguous(), torch.from_numpy(y).cuda())
            pr.pop = L.Population(pr.x, pr.g, 1, x_bf16=pr.xb, P=P, largest_batch=batch)
        pr.g.fill_(float("nan"))
        pr.pop.sync_shadow()
        loss = torch.zeros(W, device="cuda")
        pr.pop.loss(batch, loss)
        pr.pop.grad_loss(batch)
        torch.cuda.synchronize()
        res.append((loss.cpu(), np.array(pr.pop.get_losses()), pr.g.cpu()))
    (l0, s0, g0), (l1, s1, g1) = res
    assert torch.equal(l0, l1) and np.array_equal(s0, s1)
    assert torch.equal(g0[:, :P], g1[:, :P])
