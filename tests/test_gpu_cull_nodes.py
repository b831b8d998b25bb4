"""The culling kernels on node stencils (one node per unit, which they index on a
path of their own), against the oracle and the kernels that evaluate every state."""

import numpy as np
import pytest

import oracle
import synth
from synth.workloads import GRID_STENCIL, GridSpec
from tests._parity import bounds_error, node_stencil_momentum_scale
from tests.test_gpu_cull import TOL, kbl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rows_of_nodes(dim, sizes, seed):
    """States of a mesh, and rows of the given sizes over its nodes."""
    rng = np.random.default_rng(seed)
    wl = (synth.make_quad_workload(N=5, seed=seed, grid_nodes=16, name="nodes2") if dim == 2
          else synth.make_hex_workload(N=3, p=2, seed=seed, grid_nodes=8, name="nodes3"))
    cols = [rng.choice(wl.n_nodes, k, replace=False) for k in sizes]
    rowptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    return wl, rowptr, np.concatenate(cols).astype(np.int32)


# one state, uneven rows, rows at and beyond the staged states (128 and 256)
@pytest.mark.parametrize("dim,n,tile,plain", [(2, (33, 40), 14, 11), (2, (64, 50), 14, 12),
                                              (3, (18, 20, 9), 9, 6), (3, (33, 12, 10), 9, 3)])
@pytest.mark.parametrize("sizes", [(1, 2, 3, 48, 48, 48, 5, 17), (127, 128, 129, 200), (255, 256, 257, 300)])
def test_node_stencils(kbl, monkeypatch, dim, n, tile, plain, sizes):  # noqa: F811
    wl, rowptr, cols = rows_of_nodes(dim, sizes, 980 + dim)
    g = GridSpec(GRID_STENCIL, n, k=4.0)
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    vg = kbl.make_vgrid(g.mode, g.n[:dim], g.lo, g.hi, g.k)
    prm = kbl.make_params(wl.gamma, r_fac=wl.r_fac)
    got = {}
    for tl in (tile, plain):
        monkeypatch.setenv("KBL_BOUNDS_TILE", str(tl))
        print(f"[nodes] {dim}D {n} rows {sizes} tile {tl}", flush=True)
        b, s = kbl.compute_bounds_nodes(t(wl.states), t(rowptr), t(cols), vg, prm)
        got[tl] = b.cpu().numpy(), s.cpu().numpy().view(np.uint32)
    rb, rs = oracle.bounds(dim, wl.gamma, wl.states, rowptr, cols, 1, g.mode, n, g.lo, g.hi, g.k,
                           wl.r_fac, n_src=wl.n_nodes)
    scale = node_stencil_momentum_scale(wl.states, rowptr, cols, dim, range(len(sizes)))
    for b, s in got.values():
        assert np.array_equal(s, rs)
        assert bounds_error(b, rb, dim, scale)[0] <= TOL
