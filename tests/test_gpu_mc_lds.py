"""GPU parity of the matrix-completion gradients that are added up in LDS: either factor or both held there, batches that
do not divide into the workgroups' parts, one workgroup per worker, rows of any alignment, packed records, no index list."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
import workloads as wl
from gpu_util import Pair, dev, rel_l2_rows

pytestmark = pytest.mark.gpu

# small factors (the rule holds either or both; both at wide groups of many workers only), one narrow side
BOTH = [(60, 50, r, 8, 40001) for r in (1, 2, 3, 5, 8, 17, 33, 67)] + [(150, 90, 5, 300, 6001), (7, 9, 4, 1, 30000)] + \
       [(9, 1, 9, 2384, 14), (2, 2, 17, 2018, 15), (6, 3, 38, 1017, 11)]
NARROW = [(90, 9000, 1, 4, 40007), (70, 9001, 4, 5, 60007), (61, 9000, 16, 9, 40000), (41, 9000, 33, 16, 30001),
          (9000, 53, 7, 9, 40000), (9000, 37, 64, 4, 60001), (9000, 500, 67, 8, 40000), (9000, 3, 2, 300, 5000),
          (8, 500, 67, 4, 40001), (500, 8, 64, 4, 20001)]
# of these, what the rule sends by the other routes
BEYOND = [(60, 50, 67, 8, 40001), (150, 90, 5, 300, 6001), (9000, 37, 64, 4, 60001), (9000, 500, 67, 8, 40000)]


@pytest.mark.parametrize("packed,listed,odd", [(False, True, False), (True, True, True), (True, False, False)])
@pytest.mark.parametrize("m,n,r,W,B", BOTH + NARROW)
def test_matches_oracle(m, n, r, W, B, packed, listed, odd):
    g = wl.stream("mc_lds", m, n, r, seed=W)
    n_obs = B if not listed else 60000
    rows = g.integers(0, m, n_obs).astype(np.int32); cols = g.integers(0, n, n_obs).astype(np.int32)
    vals = g.standard_normal(n_obs).astype(np.float32)
    idx = g.integers(0, n_obs, (W, B)).astype(np.int32) if listed else None
    P = (m + n) * r
    x0 = np.zeros((W, P + 1 if odd else wl.padded_ld(P)), np.float32)
    x0[:, :P] = g.standard_normal((W, P)).astype(np.float32) * np.float32(r ** -0.25)
    c = 0.5 / B
    d = [dev(rows), dev(cols), dev(vals)]
    batch = L.MCBatch(m, n, r, *d, dev(idx) if listed else None, c, entries=L.mc_pack_entries(*d) if packed else None)
    pr = Pair(x0, wl.equal_group_offsets(W, 1), P=P, largest_batch=batch)
    pr.ora.grad_loss_mc(m, n, r, rows, cols, vals, idx, c)
    pr.g.fill_(float("nan"))
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    got = pr.g.cpu().numpy()
    # a row of up to 60000/3 addends of either sign: half an ulp of the running sum each, 6e-8 times sqrt(20000) = 8e-6
    assert rel_l2_rows(got[:, :P], pr.ora.g[:, :P]).max() <= 1e-5
    assert np.all(got[:, P:] == 0)
