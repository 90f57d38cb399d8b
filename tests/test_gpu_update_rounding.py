"""The roundings of the update, bit for bit, whichever route a population takes: multiply-adds are fused, and of the two pulls
the local one's product, whose coefficient is the larger in use, is the one that is not rounded by itself."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
import workloads as wl
from gpu_util import Pair

pytestmark = pytest.mark.gpu

F = np.float32


def fma(a, b, c):
    """Rounded once: a product of two floats has 48 bits, the extended format holds 64."""
    return (a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)).astype(F)


def expected(x, g, m, zl, zg, eta, lamL, lamG, mu, wd):
    eta, lamL, lamG, mu, wd = (F(v) for v in (eta, lamL, lamG, mu, wd))
    d = fma(wd, x, g)
    d = d + fma(lamL, x - zl, lamG * (x - zg))
    if m is not None:
        d = m = fma(mu, m, d)
    return fma(-eta, d, x), m


# one launch (groups of several, groups of one), row streams
@pytest.mark.parametrize("mu", [0.0, 0.9])
@pytest.mark.parametrize("W,off", [(4, [0, 4]), (8, [0, 3, 8]), (4, [0, 1, 2, 3, 4]), (9, list(range(10))), (33, [0, 9, 17, 33])])
def test_update_rounds_as_written(W, off, mu):
    P = 20_011
    x0, g0, _ = wl.stress_state(W, P, P, seed=W)
    m0 = wl.stress_grad(W, P, P, 1, 3e-2, seed=W)
    pr = Pair(x0, off, momentum=mu, weight_decay=1e-2)
    if mu:
        pr.m.copy_(torch.from_numpy(m0))
    pr.set_grad(g0, wl.stress_losses(W, 0))
    pr.ora.select()
    pr.pop.step(L.ExternalBatch(pr.losses_dev), 0.05, 0.1, 0.05)
    torch.cuda.synchronize()
    zl = x0[np.repeat(pr.ora.lead, np.diff(off))]
    x, m = expected(x0, g0, m0 if mu else None, zl, x0[pr.ora.glead[0]], 0.05, 0.1, 0.05, mu, 1e-2)
    np.testing.assert_array_equal(pr.x.cpu().numpy(), x)
    if mu:
        np.testing.assert_array_equal(pr.m.cpu().numpy(), m)
