"""The size rule that chooses between binned and atomics, seen from the host: for ranks that are no multiples of four the
workspace holds the binned route's records exactly where that route is the better of the two (sums in LDS may be better than
either)."""
import pytest
import torch

import paper_1905_10395_amd as L


def binned(m, n, r, W, B):
    t = torch.zeros(1, dtype=torch.int32)
    batch = L.MCBatch(m, n, r, t, t, torch.zeros(1), torch.zeros((W, B), dtype=torch.int32), 1.0)
    P = (m + n) * r
    sums = max((B + 255) // 256, (m + 127) // 128) * W * 4               # loss sums of either route
    return L.workspace_bytes(W, P, P, 1, batch=batch) > L.workspace_bytes(W, P, P, 1) + (sums + 255) // 256 * 256


# measured, us: atomics (the better loop) / binned
@pytest.mark.parametrize("m,n,r,W,B,want", [
    (9468, 466, 2, 16, 62000, True),       # 180 / 134: many entries on a narrow side, of many workers
    (1000, 1000, 3, 16, 62000, True),      # 129 / 100
    (3000, 4001, 5, 16, 62000, True),      # 137 / 79
    (6001, 3517, 10, 8, 16384, True),      # 34 / 26
    (1000, 800, 1, 32, 50000, True),       # 123 / 64
    (100, 20000, 5, 4, 62000, False),      # 84 / 605: one workgroup walks every record of the narrow side (LDS is taken)
    (100, 100, 5, 16, 62000, False),       # 151 / 589
    (466, 9468, 2, 4, 62000, False),       # 66 / 105
    (6001, 3517, 10, 8, 4096, False),      # 16 / 20: launches
])
def test_route_by_size(m, n, r, W, B, want):
    assert binned(m, n, r, W, B) == want
