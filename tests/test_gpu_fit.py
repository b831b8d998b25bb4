"""The 48 x 48 table tile (11) on grids that its threads are split to fit:
against the oracle and against the 3 x 3 tile without tables (2), at the edges
of the split and with stencils beyond one chunk of tables and of states."""

import numpy as np
import pytest

import oracle
import synth
from synth.workloads import GRID_STENCIL, GridSpec, quad_block_stencils
from tests._parity import bounds_error, stencil_momentum_scale
from tests.test_gpu_cull import kbl, run  # noqa: F401

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-12          # the FP64 paths' bar against the oracle


# one thread, one row or column of threads, all 256 threads (32 x 48, 48 x 30
# nodes), remainders in both directions; (48, 33) no longer fits
@pytest.mark.parametrize("n", [(2, 2), (2, 48), (48, 2), (3, 4), (32, 48), (31, 46), (48, 30),
                               (47, 29), (33, 41), (41, 35), (48, 33)])
@pytest.mark.parametrize("p,k", [(1, 1), (3, 5), (3, 25)])
def test_fit_edges(kbl, monkeypatch, n, p, k):  # noqa: F811
    N = 5
    wl = synth.make_quad_workload(N=N, p=p, seed=900 + n[0] + p, grid_nodes=20, name="fit")
    _, cols = quad_block_stencils(N, 2)
    wl.cols = np.ascontiguousarray(cols.reshape(N * N, 25)[:, :k]).ravel()
    wl.rowptr = np.arange(0, N * N * k + 1, k).astype(np.int32)
    wl.grid = GridSpec(GRID_STENCIL, n, k=4.0)
    print(f"[fit] grid {n} states {k * wl.n_s}", flush=True)
    b, s = run(kbl, monkeypatch, wl, 11)
    rb, rs = oracle.workload_bounds(wl)
    full, fs = run(kbl, monkeypatch, wl, 2)
    assert np.array_equal(s, rs) and np.array_equal(fs, rs)
    err, _ = bounds_error(b, rb, 2, stencil_momentum_scale(wl))
    ferr, _ = bounds_error(full, rb, 2, stencil_momentum_scale(wl))
    print(f"[fit] err {err:.2e}, 3 x 3 tile {ferr:.2e}", flush=True)
    assert err <= TOL
    for blocks in (1, 3, 0, -3):     # bitwise the same under every launch shape
        c, _ = run(kbl, monkeypatch, wl, 11, blocks)
        assert np.array_equal(b.view(np.uint8), c.view(np.uint8))
