"""The 2D FP64 kernel that culls stencil states block by block (tile 14):
against the oracle and against the kernel that evaluates every state, at the
edges of its blocks, list rows and staged states."""

import numpy as np
import pytest

import oracle
import synth
from synth.workloads import GRID_GLOBAL, GRID_STENCIL, GridSpec, quad_block_stencils
from tests._parity import bounds_error, stencil_momentum_scale

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-12          # the FP64 paths' bar against the oracle
CULL = 14


@pytest.fixture(scope="module")
def kbl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2407_20966_amd as kbl
    kbl._lib.lib().kbl_autotune_clear()
    return kbl


def run(kbl, monkeypatch, wl, tile, blocks=None):
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    monkeypatch.setenv("KBL_BOUNDS_TILE", str(tile))
    if blocks is None:
        monkeypatch.delenv("KBL_PERSISTENT_BLOCKS", raising=False)
    else:
        monkeypatch.setenv("KBL_PERSISTENT_BLOCKS", str(blocks))
    g = wl.grid
    vg = kbl.make_vgrid(g.mode, g.n[: wl.dim], g.lo, g.hi, g.k)
    prm = kbl.make_params(wl.gamma, r_fac=wl.r_fac)
    b, s = kbl.compute_bounds(t(wl.states), t(wl.rowptr), t(wl.cols), wl.n_s, vg, prm)
    torch.cuda.synchronize()
    return b.cpu().numpy(), s.cpu().numpy().view(np.uint32)


def check(kbl, monkeypatch, wl):
    print(f"[cull] {wl.name} grid {wl.grid.n} n_s {wl.n_s}", flush=True)
    b, s = run(kbl, monkeypatch, wl, CULL)
    rb, rs = oracle.workload_bounds(wl)
    assert np.array_equal(s, rs)
    err, _ = bounds_error(b, rb, 2, stencil_momentum_scale(wl))
    full, _ = run(kbl, monkeypatch, wl, 12)
    ferr, _ = bounds_error(full, rb, 2, stencil_momentum_scale(wl))
    print(f"[cull] err {err:.2e}, full evaluation {ferr:.2e}", flush=True)
    assert err <= TOL
    # bitwise the same under every launch shape
    for blocks in (1, 5, 0, -3):
        c, t = run(kbl, monkeypatch, wl, CULL, blocks)
        assert np.array_equal(b.view(np.uint8), c.view(np.uint8)) and np.array_equal(s, t)


# block sizes 2 to 8 and their remainders, square and not
@pytest.mark.parametrize("n", [(2, 2), (2, 64), (15, 16), (17, 5), (16, 33), (31, 32), (33, 48),
                               (47, 49), (64, 3), (63, 64), (64, 64)])
def test_grid_edges(kbl, monkeypatch, n):
    wl = synth.make_quad_workload(N=5, seed=810 + n[0], grid_nodes=16, name="cull_grid")
    wl.grid = GridSpec(GRID_STENCIL, n, k=4.0)
    check(kbl, monkeypatch, wl)


# wide global box: most blocks far in the tails of every state
@pytest.mark.parametrize("field", ["riemann4", "sine"])
def test_global_box(kbl, monkeypatch, field):
    wl = synth.make_quad_workload(N=6, seed=820, field_kind=field, grid_nodes=52,
                                  grid_mode=GRID_GLOBAL, name="cull_global")
    check(kbl, monkeypatch, wl)


# stencils below, at and above the list rows (32) and the staged states (128):
# (p, elements listed per row)
@pytest.mark.parametrize("p,k", [(1, 1), (3, 2), (4, 1), (7, 1), (2, 9), (1, 25), (3, 8), (3, 9),
                                 (3, 25)])
def test_stencil_sizes(kbl, monkeypatch, p, k):
    N = 6
    wl = synth.make_quad_workload(N=N, p=p, seed=830 + p, grid_nodes=20, name="cull_size")
    _, cols = quad_block_stencils(N, 2)
    wl.cols = np.ascontiguousarray(cols.reshape(N * N, 25)[:, :k]).ravel()
    wl.rowptr = np.arange(0, N * N * k + 1, k).astype(np.int32)
    check(kbl, monkeypatch, wl)


# states all equal (every state ties everywhere), and nearly equal
@pytest.mark.parametrize("spread", [0.0, 1e-15, 1e-9])
def test_ties(kbl, monkeypatch, spread):
    wl = synth.make_quad_workload(N=4, seed=840, grid_nodes=24, name="cull_ties")
    rng = np.random.default_rng(5)
    one = np.array([1.3, 0.4, -0.2, 2.1])[:, None]
    wl.states = one * (1.0 + spread * rng.standard_normal(wl.states.shape))
    check(kbl, monkeypatch, wl)


def test_cold_states_uneven_stencils(kbl, monkeypatch):
    wl = synth.make_tri_workload(N=8, seed=850, grid_nodes=40, name="cull_tri")
    check(kbl, monkeypatch, wl)
    st = wl.states.reshape(4, wl.n_elem, wl.n_s).copy()
    st[1:3, ::5] = 0.0
    st[3, ::5] = st[0, ::5] * 1e-12 / (wl.gamma - 1.0)      # theta = 1e-12 at rest
    wl.states = st.reshape(4, -1)
    check(kbl, monkeypatch, wl)


def test_no_internal_energy_and_strict(kbl, monkeypatch):
    wl = synth.make_quad_workload(N=5, seed=860, gamma=2.0, grid_nodes=34, r_fac=0.0,
                                  name="cull_delta0")
    check(kbl, monkeypatch, wl)


def test_bad_rows_and_states(kbl, monkeypatch):
    wl = synth.make_quad_workload(N=6, seed=870, grid_nodes=20, name="cull_bad")
    wl.cols = wl.cols.copy()
    wl.cols[7] = -1
    wl.cols[21] = wl.n_elem
    wl.states = wl.states.copy()
    wl.states[0, 18 * wl.n_s + 3] = -1.0
    wl.states[3, 25 * wl.n_s] = np.nan
    wl.rowptr = wl.rowptr.copy()
    wl.rowptr[30:] -= 2                      # rows of other lengths, the last one included
    b, s = run(kbl, monkeypatch, wl, CULL)
    c, t = run(kbl, monkeypatch, wl, 12)
    assert np.array_equal(s, t) and (s != 0).any() and (s == 0).any()
    assert np.array_equal(np.isnan(b), np.isnan(c))
    np.testing.assert_allclose(b, c, rtol=1e-11, atol=1e-11)


# d = 3 (tile 9): block sizes 4 and 8 with remainders, several rounds of 256
# blocks, stencils at and above the staged states (256), no internal energy
CULL3 = 9


def hex_wl(n, p=1, N=3, elems=None, **kw):
    wl = synth.make_hex_workload(N=N, p=p, grid_nodes=8, name="cull_hex", **kw)
    wl.grid = GridSpec(GRID_STENCIL, n, k=4.0)
    if elems:
        rng = np.random.default_rng(3)
        wl.cols = np.stack([np.concatenate([[e], rng.choice(np.delete(np.arange(wl.n_elem), e),
                                                            elems - 1, replace=False)])
                            for e in range(wl.n_elem)]).astype(np.int32).ravel()
        wl.rowptr = np.arange(0, wl.n_elem * elems + 1, elems).astype(np.int32)
    return wl


@pytest.mark.parametrize("n,kw", [((2, 2, 2), {}), ((4, 5, 3), {}), ((17, 20, 18), {}),
                                  ((31, 32, 5), {}), ((33, 9, 10), {}), ((24, 6, 40), {}),
                                  ((28, 28, 28), {}), ((9, 64, 12), {}),
                                  ((18, 12, 10), dict(elems=1)),
                                  ((18, 12, 10), dict(p=2, elems=9)),
                                  ((18, 12, 10), dict(p=2, elems=10)),
                                  ((20, 9, 9), dict(gamma=5.0 / 3.0, r_fac=0.0))])
def test_3d_edges(kbl, monkeypatch, n, kw):
    wl = hex_wl(n, seed=880 + n[0], **kw)
    print(f"[cull] hex {n} {kw}", flush=True)
    b, s = run(kbl, monkeypatch, wl, CULL3)
    rb, rs = oracle.workload_bounds(wl)
    assert np.array_equal(s, rs)
    err, _ = bounds_error(b, rb, 3, stencil_momentum_scale(wl))
    print(f"[cull] err {err:.2e}", flush=True)
    assert err <= TOL
    for blocks in (1, 5, -2):
        c, t = run(kbl, monkeypatch, wl, CULL3, blocks)
        assert np.array_equal(b.view(np.uint8), c.view(np.uint8)) and np.array_equal(s, t)


def test_3d_ties(kbl, monkeypatch):
    wl = hex_wl((18, 18, 18), seed=890)
    wl.states = np.array([1.3, 0.4, -0.2, 0.1, 2.1])[:, None] * np.ones_like(wl.states)
    b, s = run(kbl, monkeypatch, wl, CULL3)
    rb, rs = oracle.workload_bounds(wl)
    assert np.array_equal(s, rs)
    assert bounds_error(b, rb, 3, stencil_momentum_scale(wl))[0] <= TOL
