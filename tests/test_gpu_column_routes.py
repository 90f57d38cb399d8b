"""The ways through the rows of the one-launch update at their edges: groups of one and iterations of Algorithm 1 whose
rows stream whatever group they are in (batches of 8 rows at one column per thread, of 4 at two or four), iterations with up
to 4 or 8 rows in registers, iterations and pulls walked group by group, elastic averaging with up to 8, 16 or 32 rows in
registers, columns left over for the last workgroup.  Steps bit for bit against row streams; iterations bit for bit against
the calls that they are made of, whose pulls go another way or the same by size, and like pulls against the oracle; elastic
averaging against the oracle."""
import numpy as np
import pytest
import torch

import paper_1905_10395_amd as L
import test_gpu_alg1 as alg1
import test_gpu_column_step as column
import test_gpu_easgd as easgd
import workloads as wl
from gpu_util import Pair, assert_update_elementwise

pytestmark = pytest.mark.gpu


def ones(W):
    return list(range(W + 1))


GROUPS_OF_ONE = [
    (5, ones(5), 1031, 1031),                        # odd stride: one column per thread
    (8, ones(8), 257, 320),                          # one whole batch
    (9, ones(9), 255, 256),                          # a row in the second
    (17, ones(17), 301, 320),                        # ... in the third
    (32, ones(32), 64, 64),
    (5, ones(5), 200_003, 200_064),                  # two columns per thread, one left over
    (3, ones(3), 500_003, 500_032),                  # four (two with momentum), three left over
]
ALG1 = GROUPS_OF_ONE + [
    (2, [0, 2], 1031, 1031),                         # rows in registers: up to four
    (4, [0, 1, 4], 200_001, 200_064),
    (5, [0, 3, 5], 257, 320),                        # ... up to eight
    (8, [0, 3, 8], 500_003, 500_032),
    (9, [0, 4, 9], 100_001, 100_032),                # streamed: two columns per thread, one left over
    (13, [0, 5, 6, 13], 1030, 1088),                 # groups that begin inside a batch
    (16, [0, 16], 500_003, 500_032),
    (32, [0, 9, 17, 32], 301, 320),
]


@pytest.mark.parametrize("mu,flags,wd", column.OPTIONS)
@pytest.mark.parametrize("W,off,P,ld", GROUPS_OF_ONE)
def test_groups_of_one_equal_row_streams(W, off, P, ld, mu, flags, wd):
    column.test_step_equals_row_streams(W, off, P, ld, mu, flags, wd)


@pytest.mark.parametrize("mu,flags,wd", [(0.0, 0, 0.0), (0.9, L.NESTEROV, 1e-2)])
@pytest.mark.parametrize("W,off,P,ld", GROUPS_OF_ONE[:5])
def test_groups_of_one_match_the_oracle(W, off, P, ld, mu, flags, wd):
    column.test_whole_step_matches_oracle(W, off, P, ld, mu, flags, wd)


# few of many re-selected: row streams from 5000 columns and 17 workers (9, as separate calls) on
@pytest.mark.parametrize("W,P,ld", [(8, 5003, 5056), (16, 5003, 5056), (20, 4999, 4999), (20, 5003, 5056)])
def test_few_groups_of_one_re_selected_match_the_oracle(W, P, ld):
    x0, g0, _ = wl.stress_state(W, P, ld, seed=W)
    pr = Pair(x0, ones(W), P=P, momentum=0.9)
    one, none, every = np.eye(W, dtype=np.uint8)[W // 2], np.zeros(W, np.uint8), np.ones(W, np.uint8)
    for t, (rl, rg) in enumerate([(every, 1), (one, 0), (none, 1), (one, 1)]):
        for whole in (True, False):
            pr.set_grad(g0, wl.stress_losses(W, 2 * t + whole, seed=W))
            before = pr.follow_gpu()
            pr.ora.select(rl, rg); pr.ora.update(0.05, 0.1, 0.05, rl, rg)
            if whole:
                pr.pop.step(L.ExternalBatch(pr.losses_dev), 0.05, 0.1, 0.05, rl, rg)
            else:
                pr.pop.select_leaders(pr.losses_dev, rl, rg); pr.pop.pull_update(0.05, 0.1, 0.05)
            assert pr.check_leaders(rl, rg)
            pr.check_step_elementwise(before, f"step {t}")
            np.testing.assert_array_equal(pr.Z.cpu().numpy()[:, :P], pr.ora.Z[:, :P])


@pytest.mark.parametrize("mu", [0.0, 0.9])
@pytest.mark.parametrize("W,off,P,ld", ALG1)
def test_one_call_equals_separate_calls(W, off, P, ld, mu):
    column.test_one_call_equals_separate_calls(W, off, P, ld, mu)


@pytest.mark.parametrize("W,P,ld", [(1, 257, 257), (8, 1031, 1031), (9, 257, 320), (32, 301, 320), (33, 301, 320), (3, 500_003, 500_032),
                                    (10, 500_003, 500_032), (16, 940_003, 940_032)])
def test_easgd_rows_in_registers_or_twice(W, P, ld):
    column.test_easgd_both_routes(W, P, ld)          # 16 x 940 003: two passes (301 MB)


@pytest.mark.parametrize("W,G,P,ld", [(6, 2, 1_000_003, 1_000_064), (13, 1, 500_003, 500_032), (20, 4, 500_003, 500_032), (32, 4, 1031, 1031)])
def test_easgd_without_momentum(W, G, P, ld):
    easgd.test_easgd_update_matches_oracle(W, G, P, ld, 0.0, 0, 1e-4)


# Algorithm 1's iterations whose pull is walked group by group behind the update (a few of large groups communicate; pairs
# above 150 MB, or 70 with half of them; with momentum between 30 and 95 MB; a group of 5 to 8 with momentum), those beside them
# that are not, and many groups of one of which few communicate (row streams: more than 24, or more than 16 above 30 MB)
@pytest.mark.parametrize("mu", [0.0, 0.9])
@pytest.mark.parametrize("W,G,P,ld", [(8, 1, 1031, 1031), (8, 2, 301, 320), (4, 2, 301, 320), (12, 3, 1031, 1031), (16, 4, 100_003, 100_032), (24, 4, 301, 320),
                                      (16, 8, 800_003, 800_032), (28, 28, 5003, 5003), (20, 20, 130_003, 130_048)])
def test_iterations_with_few_groups_match_the_oracle(W, G, P, ld, mu):
    x0, g0, _ = wl.stress_state(W, P, ld, seed=W)
    pr = Pair(x0, wl.equal_group_offsets(W, G), P=P, momentum=mu)
    one, most = np.zeros(G, np.uint8), np.ones(G, np.uint8)
    one[G - 1], most[0] = 1, G == 1
    for t, (rl, rg) in enumerate([(np.ones(G, np.uint8), 1), (one, 0), (most, 0), (np.zeros(G, np.uint8), 1), (one, 1)]):
        pr.set_grad(g0, wl.stress_losses(W, t, seed=G))
        before = pr.follow_gpu()
        alg1.alg1_oracle_iteration(pr.ora, 0.05, 0.02 * (t > 0), 0.01 * (t > 0), 0.1, 0.07, rl, rg)
        comm = (L.COMM_LOCAL if rl.any() else 0) | (L.COMM_GLOBAL if rg else 0)
        pr.pop.step_alg1(L.ExternalBatch(pr.losses_dev), 0.05, 0.02 * (t > 0), 0.01 * (t > 0), 0.1, 0.07, comm, rl)
        assert pr.check_leaders(rl, rg)
        pr.check_step_elementwise(before, f"iteration {t}", k_self=4.0)


# pulls alone, some or all groups communicating: groups of one up to 8 workers and above, pairs, large groups above 16 workers
# and 30 MB, four workers above 100 MB
@pytest.mark.parametrize("W,G,P,ld", [(8, 8, 301, 320), (12, 12, 1031, 1031), (16, 8, 1030, 1088), (24, 4, 120_003, 120_064), (4, 2, 2_100_003, 2_100_032)])
def test_pulls_alone_match_the_oracle(W, G, P, ld):
    alg1.test_leader_pull_matches_oracle(W, G, P, ld)


@pytest.mark.parametrize("call", ["step_alg1", "leader_pull"])
@pytest.mark.parametrize("W,off", [(2, ones(2)), (4, [0, 1, 4]), (8, [0, 3, 8]), (9, [0, 4, 9]), (13, [0, 5, 6, 13]), (32, ones(32)), (40, [0, 9, 40])])
def test_group_that_does_not_communicate_takes_nothing_from_the_one_before(W, off, call):
    """Group 0 has diverged and communicates; the others are only pulled to the global leader, which is in the last group:
    the infinite leader takes no part in their rows, not even times zero."""
    P, G = 257, len(off) - 1
    x0, g0, _ = wl.stress_state(W, P, P, seed=W)
    x0[:off[1]] = np.inf
    pr = Pair(x0, off)
    losses = (np.arange(W, 0, -1) / W).astype(np.float32)
    losses[:off[1]] = np.nan
    pr.set_grad(g0, losses)
    mask = [1] + [0] * (G - 1)
    if call == "step_alg1":
        pr.ora.update(0.05, 0.0, 0.0)
        pr.pop.step_alg1(L.ExternalBatch(pr.losses_dev), 0.05, 0.0, 0.0, 0.1, 0.07, L.COMM_LOCAL | L.COMM_GLOBAL, mask)
    else:
        pr.pop.select_leaders(pr.losses_dev, mask, 1)
        pr.pop.leader_pull(0.1, 0.07)
    rl = np.array(mask, np.uint8)
    pr.ora.select(rl, 1); pr.ora.leader_pull(0.1, 0.07, rl, 1)
    torch.cuda.synchronize()
    rest = slice(off[1], W)
    got, Z = pr.x.cpu().numpy()[rest], pr.Z.cpu().numpy()
    assert np.all(np.isfinite(pr.ora.x[rest])) and np.all(np.isfinite(got))
    assert_update_elementwise(got, pr.ora.x[rest], x0[rest])
    assert not np.any(np.isfinite(Z[0])) and np.all(np.isfinite(Z[G]))
