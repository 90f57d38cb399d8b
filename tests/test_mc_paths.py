"""The GPU tests of the matrix-completion gradient reach the routes that they name: what the library's rule says for their shapes,
on the host."""
import ctypes as C

import pytest

import paper_1905_10395_amd as L
import test_gpu_mc_lds as lds
import test_gpu_mc_routes as routes
from paper_1905_10395_amd import binding

ONE, FLIGHT, BINNED, LDS = range(4)


def path(W, m, n, r, B, vw=None):
    """Route, whether the gradients of U and of V are held in LDS, prepare workgroups and their entries (binned)."""
    return describe(W, m, n, r, B, vw)[:5]


def few(W, m, n, r, B):
    """Workgroups per worker of two entries per lane group, and the slots that their loss sums share; 0, 0: another loop."""
    return tuple(describe(W, m, n, r, B)[5:])


def describe(W, m, n, r, B, vw=None):
    f = getattr(L.lib(), "_ZN4lsgd16mc_describe_pathEiRK13lsgd_mc_batchimPi")
    f.argtypes, f.restype = [C.c_int, C.POINTER(binding._MC), C.c_int, C.c_size_t, C.POINTER(C.c_int)], None
    out = (C.c_int * 7)()
    d = binding._MC(m, n, r, None, None, None, B, 1, B, 1.0, None)      # (the rule reads sizes, no arrays)
    f(W, C.byref(d), vw or (4 if r % 4 == 0 else 2 if r % 2 == 0 else 1), 1 << 40, out)
    return list(out)


@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 10, 12, 33, 50, 64])
def test_few_and_many_entries(r):
    assert path(9, 4001, 3000, r, 300)[0] == (BINNED if r == 64 else ONE if r <= 2 else FLIGHT)
    assert path(9, 4001, 3000, r, 40000)[0] == (LDS if r <= 2 else BINNED)


@pytest.mark.parametrize("r", [1, 2, 3, 5, 6, 7, 9, 16, 17, 33, 64, 67])
@pytest.mark.parametrize("W,m,n", [(4, 90, 4000), (9, 4000, 61)])
def test_narrow_side(W, m, n, r):
    assert (path(W, m, n, r, 40000)[0] == LDS) == (r <= 33)


def test_one_at_a_time_and_binned():
    lanes = [1 << (r - 1).bit_length() for _, _, _, r, _ in routes.ONE_AT_A_TIME]
    assert lanes == [4, 8, 16, 32, 64]
    assert all(path(*s)[0] == ONE for s in routes.ONE_AT_A_TIME)
    assert all(path(*s)[0] == BINNED for s in routes.BINNED)


@pytest.mark.parametrize("W,m,n,B", [(2, 5000, 4000, 20000), (3, 5000, 4000, 20000), (9, 5000, 4000, 20000), (3, 3000, 2500, 20000),
                                     (9, 700, 3000, 30000), (12, 1000, 800, 20000)])
def test_bins_on_dies(W, m, n, B):
    assert path(W, m, n, 64, B)[0] == BINNED


@pytest.mark.parametrize("r", [4, 8, 10])
def test_rows_of_any_alignment(r):
    assert path(9, 4001, 3000, r, 40000, vw=1 if r == 8 else 2)[0] == BINNED


def test_two_entries_per_lane_group():
    """Every shape of the GPU test goes this way: with one slot, with several and with all eight, fewer and more workgroups than
    slots, at every width of a lane group but the narrowest two.  Not where requests queue or meet in the same lines."""
    assert [few(*s) for s in routes.FEW] == [(3, 1), (4, 1), (4, 4), (1, 2), (16, 3), (13, 1), (24, 8), (188, 8), (1, 1)]
    assert {min(64, 1 << (s[3] - 1).bit_length()) for s in routes.FEW} == {4, 8, 16, 32, 64}
    assert few(1, 3000, 5000, 6, 30_000)[0] > 0 and few(1, 3000, 5000, 6, 35_000) == (0, 0)
    assert few(5, 60, 5000, 12, 3_000)[0] > 0 and few(5, 60, 5000, 12, 5_000) == (0, 0)
    assert few(4, 700, 600, 2, 256) == (0, 0)


@pytest.mark.parametrize("m,n,r,W,B,blocks,entries", [(5400, 4400, 4, 2, 263_000, 257, 1024), (3100, 2900, 4, 4, 263_000, 129, 2048),
                                                      (1700, 1500, 4, 8, 263_000, 65, 4096)])
def test_prepare_workgroups(m, n, r, W, B, blocks, entries):
    assert path(W, m, n, r, B) == [BINNED, 0, 0, blocks, entries]


@pytest.mark.parametrize("vw", [None, 1])
@pytest.mark.parametrize("m,n,r,W,B", lds.BOTH + lds.NARROW)
def test_sums_in_lds(m, n, r, W, B, vw):
    assert (path(W, m, n, r, B, vw)[0] == LDS) == ((m, n, r, W, B) not in lds.BEYOND)


def test_every_way_of_sums_in_lds():
    """U, V or both, at every number of lanes per entry (both: where the two factors are small enough for it)."""
    seen = set()
    for m, n, r, W, B in lds.BOTH + lds.NARROW:
        p = path(W, m, n, r, B)
        if p[0] == LDS:
            seen.add((min(64, 1 << (r - 1).bit_length()), p[1], p[2]))
    assert {(s, 1, 1) for s in (1, 2, 4, 8, 16, 32, 64)} <= seen
    assert {s for s, u, v in seen if u != v} >= {4, 8, 16, 32, 64}
    assert {(u, v) for _, u, v in seen} == {(1, 0), (0, 1), (1, 1)}
