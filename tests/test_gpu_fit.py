"""Kernels whose threads are split to fit the velocity grid, at the edges of the
split: tile 1 and the table tiles (11 and 12) against the oracle and the tiles
that are not split, with stencils beyond one chunk of tables and of states; the per-state
energy bounds and the backward against the oracle."""

import numpy as np
import pytest

import oracle
import synth
from synth.workloads import GRID_STENCIL, GridSpec, quad_block_stencils
from tests._parity import bounds_error, stencil_momentum_scale
from tests.test_gpu_backward import compare_with_oracle, dev_inputs
from tests.test_gpu_cull import kbl, run  # noqa: F401
from tests.test_gpu_variants import check_energy

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-12          # the FP64 paths' bar against the oracle


# one thread, one row or column of threads, all 256 threads (32 x 16, 16 x 32, 32 x
# 48, 48 x 30 nodes), remainders in both directions; (29, 28), (48, 33), (64, 47) and
# (49, 64) do not fit
@pytest.mark.parametrize("n", [(2, 2), (2, 48), (48, 2), (3, 4), (32, 48), (31, 46), (48, 30),
                               (47, 29), (33, 41), (41, 35), (48, 33), (50, 50), (49, 60), (60, 49), (64, 44),
                               (3, 64), (49, 2), (64, 47), (49, 64), (32, 16), (16, 32),
                               (22, 23), (27, 26), (32, 24), (29, 28), (17, 2), (2, 31)])
@pytest.mark.parametrize("p,k", [(1, 1), (3, 5), (3, 25)])
def test_fit_edges(kbl, monkeypatch, n, p, k):  # noqa: F811
    N = 5
    wl = synth.make_quad_workload(N=N, p=p, seed=900 + n[0] + p, grid_nodes=20, name="fit")
    _, cols = quad_block_stencils(N, 2)
    wl.cols = np.ascontiguousarray(cols.reshape(N * N, 25)[:, :k]).ravel()
    wl.rowptr = np.arange(0, N * N * k + 1, k).astype(np.int32)
    wl.grid = GridSpec(GRID_STENCIL, n, k=4.0)
    print(f"[fit] grid {n} states {k * wl.n_s}", flush=True)
    tile, plain = (1, 10) if max(n) <= 32 else (11, 2) if max(n) <= 48 else (12, 5)
    b, s = run(kbl, monkeypatch, wl, tile)
    rb, rs = oracle.workload_bounds(wl)
    full, fs = run(kbl, monkeypatch, wl, plain)
    assert np.array_equal(s, rs) and np.array_equal(fs, rs)
    err, _ = bounds_error(b, rb, 2, stencil_momentum_scale(wl))
    ferr, _ = bounds_error(full, rb, 2, stencil_momentum_scale(wl))
    print(f"[fit] err {err:.2e}, plain tile {ferr:.2e}", flush=True)
    assert err <= TOL
    for blocks in (1, 3, 0, -3):     # bitwise the same under every launch shape
        c, _ = run(kbl, monkeypatch, wl, tile, blocks)
        assert np.array_equal(b.view(np.uint8), c.view(np.uint8))


GRIDS = [(2, 48), (32, 48), (33, 41), (48, 29), (48, 33), (49, 60), (64, 44), (64, 47)]


@pytest.mark.parametrize("n", GRIDS)
def test_fit_energy(kbl, n):  # noqa: F811
    wl = synth.make_quad_workload(N=6, seed=930 + n[0], grid_nodes=20, name="fit_energy")
    wl.grid = GridSpec(GRID_STENCIL, n, k=4.0)
    check_energy(kbl, wl)


@pytest.mark.parametrize("n", GRIDS[1:])
def test_fit_backward(kbl, n):  # noqa: F811
    wl = synth.make_quad_workload(N=4, seed=940 + n[0], grid_nodes=20, name=f"fit_bwd{n}")
    wl.grid = GridSpec(GRID_STENCIL, n, k=4.0)
    wl.target = wl.states + 10.0 * (wl.target - wl.states)
    compare_with_oracle(kbl, wl)


@pytest.mark.parametrize("n", [(33, 41), (49, 60)])
def test_fit_backward_mixed(kbl, n):  # noqa: F811
    """The FP32 forward's gradient against the FP64 one, to the bars of the mixed
    backward's own test (the limiter amplifies 1e-7 differences of the bounds)."""
    wl = synth.make_quad_workload(N=32, seed=52, grid_nodes=48, name="fit_mixed")
    wl.grid = GridSpec(GRID_STENCIL, n, k=4.0)
    st, tg, rp, cl, vg, prm = dev_inputs(kbl, wl)
    prm_m = kbl.make_params(wl.gamma, r_fac=wl.r_fac, precision=3)
    G = torch.zeros_like(st)
    G[0] = torch.from_numpy(np.random.default_rng(5).standard_normal(wl.n_nodes)).to(st.device)
    g = [sum(kbl.bounds_limit_backward(st, rp, cl, wl.n_s, vg, q, tg, wl.node_weights, G)[:2])
         for q in (prm, prm_m)]
    err, scale = (g[1] - g[0]).abs(), g[0].abs().max()
    assert err.max() <= 5e-2 * scale
    assert (err <= 1e-6 * scale).double().mean() >= 0.9
