"""Culling kernels on a state of denormal temperature: its q has no finite bound,
and it is the smallest wherever no node meets its velocity.  Bounds against the
kernels that evaluate every state."""

import numpy as np
import pytest

import synth
from synth.workloads import GRID_GLOBAL, GridSpec
from tests.test_gpu_cull import kbl, run  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# nodes at odd integers: 3 blocks per direction in 2D, whose middle one is centred at
# the cold state's velocity 0; 500 nodes of a 1D grid are not culled
@pytest.mark.parametrize("dim,n,box,tile,plain", [(1, 700, 699.0, 0, 500), (2, 6, 5.0, 14, 0),
                                                  (3, 6, 5.0, 9, 0)])
def test_denormal_temperature(kbl, monkeypatch, dim, n, box, tile, plain):  # noqa: F811
    make = {1: lambda: synth.make_line_workload(n_elem=8, seed=71, name="cold1"),
            2: lambda: synth.make_quad_workload(N=4, p=2, seed=72, grid_nodes=16, name="cold2"),
            3: lambda: synth.make_hex_workload(N=3, p=1, seed=73, grid_nodes=8, name="cold3")}
    wl = make[dim]()
    wl.states = wl.states.copy()
    col = 2 * wl.n_s + 1
    wl.states[:, col] = 0.0
    wl.states[0, col], wl.states[-1, col] = 1.0, 2.5e-310
    wl.grid = GridSpec(GRID_GLOBAL, (n,) * dim, (-box,) * dim, (box,) * dim, 0.0)
    print(f"[cold] {dim}D {n} nodes", flush=True)
    b, s = run(kbl, monkeypatch, wl, tile)
    if dim == 1:
        wl.grid = GridSpec(GRID_GLOBAL, (plain,), (-box,), (box,), 0.0)
        c, t = run(kbl, monkeypatch, wl, 0)
    else:
        c, t = run(kbl, monkeypatch, wl, plain)
    near = [e for e in range(wl.n_elem) if 2 in wl.cols[wl.rowptr[e]:wl.rowptr[e + 1]]]
    assert 2 in near and np.array_equal(s, t)
    # its neighbours' lower envelope is 0 everywhere: rho_min at its floor, E_min 0
    assert np.all(s[near] == kbl._lib.ST_RHO_FLOOR) and np.all(b[dim + 1, near] == 0.0)
    if dim > 1:
        np.testing.assert_allclose(b, c, rtol=1e-12, atol=1e-12)
