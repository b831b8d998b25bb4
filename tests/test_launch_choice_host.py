"""The launch that a bounds call chooses (kbl_bounds_launch; no device): which
kernel the default rules pick on both sides of their thresholds."""

import os

import pytest

from paper_2407_20966_amd import _lib as L

CULL = {2: 14, 3: 9}
INT32_MAX = 2**31 - 1


@pytest.fixture(autouse=True)
def plain_environment(monkeypatch):
    if not os.path.exists(L.LIB_PATH):
        pytest.skip("libkbl.so not built (run __graft_entry__.build())")
    for k in ("KBL_BOUNDS_TILE", "KBL_MIXED_TILE", "KBL_PERSISTENT_BLOCKS"):
        monkeypatch.delenv(k, raising=False)


def launch(n, n_elem, n_s, states, precision=L.PREC_FP64, flags=0):
    """(tile, blocks) for rows of `states` states."""
    p = L.Params()
    L.lib().kbl_default_params(p, 1.4)
    p.precision, p.flags = precision, flags
    g = L.VGrid()
    g.mode, g.k = L.GRID_STENCIL, 4.0
    for i, m in enumerate(n):
        g.n[i] = m
    return L.bounds_launch(p, len(n), n_elem, n_s, states // n_s * n_elem, g)


@pytest.mark.parametrize("n", [(64, 64), (40, 40, 40)])
def test_culling_kernel_only_where_it_takes_the_rows(monkeypatch, n):
    """nnz n_s beyond 2^31 - 1 or 2^16 nodes per element: asked for or not, the
    culling kernel gives way to one that takes them."""
    cull = CULL[len(n)]
    n_s, states = 8, 56
    at_most = INT32_MAX // states
    for forced in (False, True):
        if forced:
            monkeypatch.setenv("KBL_BOUNDS_TILE", str(cull))
        assert launch(n, at_most, n_s, states)[0] == cull
        assert launch(n, at_most + 1, n_s, states)[0] != cull
        assert launch(n, 4000, 65536, 65536)[0] != cull


@pytest.mark.parametrize("n", [(40, 40), (50, 50), (64, 64)])
def test_2d_stencils_beyond_the_staged_states(n):
    for n_elem in (4096, 16384, 100000):
        assert launch(n, n_elem, 16, 128)[0] == 14
        for n_s, states in ((1, 129), (16, 144), (25, 225), (36, 180), (64, 320)):
            assert launch(n, n_elem, n_s, states)[0] != 14


def test_3d_stencils_beyond_the_staged_states():
    # (nodes, kernel): 448 and 729 states, which no kernel can cull
    for n, culls in (((18, 18, 18), True), ((20, 20, 20), True), ((22, 22, 22), False),
                     ((24, 24, 24), False), ((28, 28, 28), True), ((30, 30, 30), False),
                     ((40, 40, 40), True)):
        for n_s, states in ((64, 448), (27, 729)):
            assert (launch(n, 512, n_s, states)[0] == 9) == culls
            assert (launch(n, 20000, n_s, states)[0] == 9) == culls
        assert launch(n, 4096, 32, 256)[0] == 9


@pytest.mark.parametrize("n", [(40, 40), (50, 50), (64, 64)])
def test_2d_few_states(n):
    for states, n_s in ((5, 1), (9, 1), (4, 4)):
        assert launch(n, 4096, n_s, states)[0] != 14
        assert launch(n, 10000, n_s, states)[0] == 14
    assert launch(n, 4096, 4, 20)[0] == 14
    assert launch(n, 2025, 4, 20)[0] != 14


@pytest.mark.parametrize("n,few,many", [(18, 7, 27), (24, 16, 56), (30, 7, 16)])
def test_3d_few_states(n, few, many):
    assert launch((n, n, n), 512, 1, few)[0] != 9
    assert launch((n, n, n), 512, 1, many)[0] == 9
    assert launch((n, n, n), 400, 1, many)[0] != 9
    assert launch((40, 20, 20), 125, 1, few)[0] == 9


MIXED = (L.PREC_MIXED_BF16, L.PREC_MIXED_FP16, L.PREC_MIXED_FP32)


@pytest.mark.parametrize("n,one,two", [((16, 16), (100, 3249, 4624, 8100), (3600, 4096, 8192, 10**6)),
                                       ((32, 32), (2025, 4096, 8100), (8192, 10**6)),
                                       ((48, 48), (1764, 2304, 4096, 8100), (2025, 2048, 8192)),
                                       ((64, 64), (1764, 2304, 3249), (8192, 10**6))])
def test_mixed_elements_per_workgroup(n, one, two):
    for prec in MIXED:
        for states in (16, 80):
            assert all(launch(n, e, 16, states, prec)[1] == 0 for e in one)
            assert all(launch(n, e, 16, states, prec)[1] == -2 for e in two)


def test_mixed_elements_per_workgroup_by_tile(monkeypatch):
    n = (64, 64)
    for n_elem in (2025, 4096):
        assert launch(n, n_elem, 16, 80, L.PREC_MIXED_FP16) == (5, -2)
        assert launch(n, n_elem, 4, 20, L.PREC_MIXED_FP16) == (5, 0)
        assert launch(n, n_elem + 200, 16, 80, L.PREC_MIXED_FP16) == (5, 0)
    assert launch(n, 5000, 16, 80, L.PREC_MIXED_BF16) == (6, -2)
    assert launch(n, 5000, 16, 80, L.PREC_MIXED_FP32) == (6, 0)
    for prec in (L.PREC_MIXED_BF16, L.PREC_MIXED_FP32):
        assert launch(n, 4096, 4, 20, prec) == (6, -2)
        assert launch(n, 2025, 4, 20, prec) == (6, 0)
    monkeypatch.setenv("KBL_MIXED_TILE", "6")
    assert launch((48, 48), 2025, 16, 80, L.PREC_MIXED_FP32) == (6, 0)
    monkeypatch.setenv("KBL_PERSISTENT_BLOCKS", "-4")
    assert launch((48, 48), 2025, 16, 80, L.PREC_MIXED_FP32) == (6, -4)


def test_errors_are_those_of_the_call():
    with pytest.raises(L.KblError) as e:
        launch((65, 64), 10, 1, 5)
    assert e.value.code == L.KBL_ERR_GRID
    with pytest.raises(L.KblError) as e:
        launch((24, 24, 24), 10, 1, 7, precision=L.PREC_MIXED_FP32)
    assert e.value.code == L.KBL_ERR_UNSUPPORTED


def test_overrides_hold_over_the_default(monkeypatch):
    assert launch((64, 64), 20000, 16, 80) == (14, 0)
    monkeypatch.setenv("KBL_PERSISTENT_BLOCKS", "-2")
    assert launch((64, 64), 20000, 16, 80) == (14, -2)
    monkeypatch.setenv("KBL_BOUNDS_TILE", "12")
    assert launch((64, 64), 20000, 16, 80) == (12, -2)
    monkeypatch.setenv("KBL_BOUNDS_TILE", "1")      # does not cover the grid
    assert launch((64, 64), 20000, 16, 80) == (14, -2)
    monkeypatch.delenv("KBL_PERSISTENT_BLOCKS")
    monkeypatch.setenv("KBL_BOUNDS_TILE", "12")
    assert launch((64, 64), 2000, 16, 80) == (12, 0)


# (grid, elements, nodes per element, states, tile): both sides of each threshold of
# the 2D rule for quads of 80 states unless it is about the states or the nodes
@pytest.mark.parametrize("n,n_elem,n_s,states,tile", [
    ((64, 64), 2999, 16, 80, 12), ((64, 64), 3000, 16, 80, 14), ((49, 2), 3000, 16, 80, 14),
    ((40, 40), 2999, 16, 80, 11), ((40, 40), 3000, 16, 80, 14),
    ((48, 48), 8191, 16, 80, 11), ((48, 48), 8192, 16, 80, 14), ((48, 48), 10**6, 1, 48, 11),
    ((48, 48), 10**6, 4, 36, 11), ((48, 48), 10**6, 4, 40, 14),
    ((36, 41), 8191, 16, 80, 11), ((36, 41), 8192, 16, 80, 14),
    ((32, 30), 8191, 16, 80, 1), ((32, 30), 8192, 16, 80, 14), ((32, 24), 10**6, 16, 80, 1),
    ((28, 28), 32767, 16, 80, 1), ((28, 28), 32768, 16, 80, 14), ((28, 28), 10**6, 4, 60, 1),
    ((24, 24), 10**6, 16, 80, 1), ((16, 16), 10**6, 16, 80, 0)])
def test_2d_default_kernel(n, n_elem, n_s, states, tile):
    assert launch(n, n_elem, n_s, states)[0] == tile


def test_2d_default_elements_per_wave_or_workgroup():
    assert [launch((64, 64), e, 16, 80)[1] for e in (2000, 65535, 65536)] == [0, 0, -2]
    assert [launch((16, 16), e, 16, 80)[1] for e in (8191, 8192)] == [0, -2]


@pytest.mark.parametrize("n,n_elem,tile", [
    ((24, 24, 24), 511, 6), ((24, 24, 24), 512, 9), ((16, 16, 64), 10**5, 0), ((17, 2, 2), 512, 9),
    ((30, 30, 30), 511, 2), ((33, 2, 2), 1, 9), ((2, 33, 2), 1, 9), ((40, 40, 40), 1, 9)])
def test_3d_default_kernel(n, n_elem, tile):
    assert launch(n, n_elem, 27, 189) == (tile, 0)
