"""GPU parity of the routes of the matrix-completion gradient (binned, atomics an entry at a time and with entries in flight;
sums in LDS have a file of their own) at every width of a lane's part of a factor row, on shapes that the size rule sends to
each (test_mc_paths.py sees to that), and on workspaces without room for the binned route."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
import workloads as wl
from gpu_util import Pair, dev, rel_l2_rows

pytestmark = pytest.mark.gpu


def problem(m, n, r, n_obs, W, B, seed, ld=None, pop_kw=None, G=1):
    g = wl.stream("mc_routes", m, n, r, seed=seed)
    rows = g.integers(0, m, n_obs).astype(np.int32); cols = g.integers(0, n, n_obs).astype(np.int32)
    vals = g.standard_normal(n_obs).astype(np.float32)
    idx = g.integers(0, n_obs, (W, B)).astype(np.int32)
    P = (m + n) * r
    ld = wl.padded_ld(P) if ld is None else ld(P)
    x0 = np.zeros((W, ld), np.float32)
    x0[:, :P] = g.standard_normal((W, P)).astype(np.float32) * np.float32(r ** -0.25)
    c = 0.5 / B
    batch = L.MCBatch(m, n, r, dev(rows), dev(cols), dev(vals), dev(idx), c)
    pr = Pair(x0, wl.equal_group_offsets(W, G), P=P, largest_batch=batch)
    pr.ora.grad_loss_mc(m, n, r, rows, cols, vals, idx, c)
    return pr, batch, P


# bins of 128 rows: one row past a bin, several bins; ranks with lanes of four, two and one column, exact and not;
# 40000 entries per worker so that the binned route is the faster one by the rule (ranks 1 and 2: sums in LDS), 300 so that it is
# not, but for rank 64
@pytest.mark.parametrize("B", [300, 40000])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 10, 12, 33, 50, 64])
def test_both_routes_match_oracle(r, B):
    W = 9
    pr, batch, P = problem(4001, 3000, r, 60000, W, B, seed=r)
    pr.g.fill_(float("nan"))
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    g = pr.g.cpu().numpy()
    assert rel_l2_rows(g[:, :P], pr.ora.g[:, :P]).max() <= 1e-5
    assert np.all(g[:, P:] == 0)


# W, m, n, r, entries: the atomics an entry at a time, groups of 4, 8, 16, 32 and 64 lanes (1 and 2 above)
ONE_AT_A_TIME = [(4, 210, 580, 3, 12_000), (2, 3300, 520, 5, 50_000), (4, 980, 2300, 9, 44_000), (8, 1220, 1400, 17, 34_400), (9, 4000, 61, 64, 40_000)]
# binned at the lowest ranks
BINNED = [(4, 5600, 4600, 1, 36_000), (7, 5800, 2600, 2, 18_000)]


@pytest.mark.parametrize("W,m,n,r,B", ONE_AT_A_TIME + BINNED)
def test_route_matches_oracle(W, m, n, r, B):
    pr, batch, P = problem(m, n, r, 60000, W, B, seed=r)
    pr.g.fill_(float("nan"))
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    g = pr.g.cpu().numpy()
    assert rel_l2_rows(g[:, :P], pr.ora.g[:, :P]).max() <= 1e-5
    assert np.all(g[:, P:] == 0)


# one side of few rows, many entries: sums in LDS up to rank 33, atomics above
@pytest.mark.parametrize("W,m,n", [(4, 90, 4000), (9, 4000, 61)])     # (628 and 1413 loss sums)
@pytest.mark.parametrize("r", [1, 2, 3, 5, 6, 7, 9, 16, 17, 33, 64, 67])
def test_narrow_side_matches_oracle(r, W, m, n):
    pr, batch, P = problem(m, n, r, 60000, W, 40000, seed=r)
    pr.g.fill_(float("nan"))
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    g = pr.g.cpu().numpy()
    assert rel_l2_rows(g[:, :P], pr.ora.g[:, :P]).max() <= 1e-5
    assert np.all(g[:, P:] == 0)


# worker counts that are no multiples of the eight dies, binned: contiguous runs of bins per die, and a worker per die
# where the fullest bin's records are what the launch waits for
@pytest.mark.parametrize("W,m,n,B", [(2, 5000, 4000, 20000), (3, 5000, 4000, 20000), (9, 5000, 4000, 20000),
                                     (3, 3000, 2500, 20000), (9, 700, 3000, 30000), (12, 1000, 800, 20000)])
def test_bins_on_dies_match_oracle(W, m, n, B):
    pr, batch, P = problem(m, n, 64, 60000, W, B, seed=W)
    pr.g.fill_(float("nan"))
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    assert rel_l2_rows(pr.g.cpu().numpy()[:, :P], pr.ora.g[:, :P]).max() <= 1e-5


@pytest.mark.parametrize("r", [4, 8, 10])
def test_rows_that_are_not_aligned_for_the_widest_lanes(r):
    """Odd row strides: the binned route with two or one column per lane."""
    pr, batch, P = problem(4001, 3000, r, 60000, 9, 40000, seed=r, ld=lambda P: P + 2 if r != 8 else P + 1)
    pr.g.fill_(float("nan"))
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    assert rel_l2_rows(pr.g.cpu().numpy()[:, :P], pr.ora.g[:, :P]).max() <= 1e-5


def test_workspace_without_binned_scratch():
    """A workspace that holds the loss sums but not the binned route's records: other ranks than multiples of four take
    the atomics instead, multiples of four are refused as ever."""
    for r in (5, 8):
        pr, batch, P = problem(4001, 3000, r, 60000, 9, 40000, seed=r)
        small = 9 * ((40000 + 255) // 256) * 4
        need = L.workspace_bytes(9, P, pr.ld, 1) + (small + 255) // 256 * 256
        assert need < L.workspace_bytes(9, P, pr.ld, 1, batch=batch)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
        g = torch.full_like(pr.x, float("nan"))
        pop = L.Population(pr.x, g, 1, P=P, workspace=ws)
        if r == 8:
            with pytest.raises(L.LsgdError, match="workspace"):
                pop.grad_loss(batch)
            continue
        pop.grad_loss(batch)
        torch.cuda.synchronize()
        assert rel_l2_rows(g.cpu().numpy()[:, :P], pr.ora.g[:, :P]).max() <= 1e-5


@pytest.mark.parametrize("W,B", [(1, 700), (2, 40000), (3, 300), (8, 300), (32, 300)])
def test_step_finishes_the_loss_sums_in_the_update(W, B):
    """lsgd_step leaves the partial loss sums to the update's launch (not with one worker, nor with more sums than that
    adds up): losses, leaders and the step as from the calls."""
    pr, batch, P = problem(500, 300, 5, 20000, W, B, seed=W)
    sep, _, _ = problem(500, 300, 5, 20000, W, B, seed=W)
    sep.pop.grad_loss(batch); sep.pop.select_leaders()
    pr.pop.step(batch, 0.01, 0.1, 0.05)
    torch.cuda.synchronize()
    np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-5)
    assert pr.pop.get_losses() == sep.pop.get_losses()       # few sums: one order, whoever adds them up
    assert pr.pop.get_leaders() == sep.pop.get_leaders()
    pr.ora.select(); pr.ora.update(0.01, 0.1, 0.05)
    pr.check_state(1e-6)


def exact_problem(r, m, vals, c, U, V):
    """Entry k couples rows k of both factors, every worker takes all of them; the factors are those given."""
    W, P, k = 2, 2 * m * r, np.arange(len(vals), dtype=np.int32)
    x0 = np.zeros((W, wl.padded_ld(P)), np.float32)
    x0[:, :P] = np.concatenate([U.reshape(-1), V.reshape(-1)])
    batch = L.MCBatch(m, m, r, dev(k), dev(k), dev(vals.astype(np.float32)), None, c)
    return Pair(x0, [0, W], P=P, largest_batch=batch), batch


@pytest.mark.parametrize("call", ["grad_loss", "step"])
@pytest.mark.parametrize("r", [1, 4, 5, 8, 50, 64])
def test_small_batch_sums_squares_in_double(r, call):
    """64 squares of 2^24 and 192 below one: an fp32 chain drops the latter (its unit there is 2), the sum in double,
    2^30 + 168.75, rounds to 2^30 + 128.  Everything else is exact."""
    vals = np.where(np.arange(256) < 64, 4096.0, 0.9375)
    pr, batch = exact_problem(r, 300, vals, 1.0, np.zeros((300, r)), np.zeros((300, r)))
    if call == "step":
        pr.pop.step(batch, 0.0, 0.0, 0.0)
    else:
        pr.pop.grad_loss(batch)
    assert pr.pop.get_losses() == [2.0 ** 30 + 128] * 2


@pytest.mark.parametrize("r", [1, 4, 5, 8, 50, 64])
def test_small_batch_rounds_a_gradient_term_once(r):
    """One entry per factor row, residuals and factors small integers: the gradient is 2c e v rounded once."""
    g = wl.stream("mc_exact", r)
    U, V = g.integers(-7, 8, (300, r)).astype(np.float64), g.integers(-7, 8, (300, r)).astype(np.float64)
    vals = g.integers(-200, 201, 256).astype(np.float64)
    c = np.float32(0.3)
    pr, batch = exact_problem(r, 300, vals, float(c), U, V)
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    e = (U * V).sum(1)[:256] - vals
    want = np.zeros((2, 300, r), np.float32)
    two_c = np.float64(np.float32(2) * c)
    want[0, :256] = (two_c * e[:, None] * V[:256]).astype(np.float32)      # exact in 64 bits up to here
    want[1, :256] = (two_c * e[:, None] * U[:256]).astype(np.float32)
    np.testing.assert_array_equal(pr.g.cpu().numpy()[0, :600 * r], want.reshape(-1))


@pytest.mark.parametrize("r", [1, 4, 5, 50])
def test_small_batch_overflow_stays_infinite(r):
    """A product past the largest float makes that residual, and with it the loss and its gradient rows, infinite, not NaN."""
    U = np.ones((300, r)); V = np.ones((300, r))
    U[7], V[7] = 1e30, 1e30
    pr, batch = exact_problem(r, 300, np.zeros(256), 1.0, U, V)
    pr.pop.grad_loss(batch)
    torch.cuda.synchronize()
    assert pr.pop.get_losses() == [float("inf")] * 2
    g = pr.g.cpu().numpy()[0, :600 * r].reshape(600, r)
    assert np.all(np.isposinf(g[[7, 307]])) and np.all(np.isfinite(np.delete(g, [7, 307], 0)))


# entries in flight, two per lane group: every width of a group, remainders of its workgroups, one slot of sums and several
FEW = [(4, 200, 150, 3, 257), (3, 300, 140, 4, 500), (5, 1000, 800, 5, 256), (2, 400, 300, 9, 1), (4, 700, 600, 17, 1000),
       (2, 300, 200, 50, 400), (16, 2000, 3000, 10, 1500), (1, 3000, 5000, 6, 12_000), (3, 129, 64, 7, 63)]


@pytest.mark.parametrize("W,m,n,r,B", FEW)
def test_few_entries_in_flight_match_oracle(W, m, n, r, B):
    pr, batch, P = problem(m, n, r, min(m * n, 5000), W, B, seed=r + B)
    for _ in range(2):                                   # the slots of the sums are cleared by every call
        pr.g.fill_(float("nan"))
        pr.pop.grad_loss(batch)
        torch.cuda.synchronize()
        np.testing.assert_allclose(pr.pop.get_losses(), pr.ora.losses, rtol=1e-6)
        g = pr.g.cpu().numpy()
        assert rel_l2_rows(g[:, :P], pr.ora.g[:, :P]).max() <= 1e-5
        assert np.all(g[:, P:] == 0)
