"""Culling kernels on flows that vary little within a stencil: the bounds are those of
the oracle, and a variation of 1e-6 is culled as a variation of 1e-2 is (the
time of the call says so)."""

import numpy as np
import pytest

import oracle
import synth
from synth.workloads import GRID_GLOBAL, GRID_STENCIL, GridSpec
from tests._parity import bounds_error, stencil_momentum_scale
from tests.test_gpu_cull import TOL, kbl, run  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GRIDS = {1: (1100,), 2: (40, 40), 3: (24, 18, 20)}
TILE = {1: 0, 2: 14, 3: 9}


def workload(dim, n, eps):
    """Smooth periodic fields of relative amplitude eps around one state."""
    make = {1: lambda: synth.make_line_workload(n_elem=n, seed=75, name="amp1"),
            2: lambda: synth.make_quad_workload(N=n, p=2, seed=76, grid_nodes=16, name="amp2"),
            3: lambda: synth.make_hex_workload(N=n, p=2, seed=77, grid_nodes=8, name="amp3")}
    wl = make[dim]()
    x = np.arange(wl.n_nodes) / wl.n_nodes
    wave = [1.0 + eps * np.sin(2.0 * np.pi * (k + 3) * n * x + k) for k in range(dim + 2)]
    rho, P = 1.3 * wave[0], 0.9 * wave[1]
    U = [(0.4 - 0.3 * d) * wave[2 + d] for d in range(dim)]
    wl.states = np.stack([rho] + [rho * u for u in U]
                         + [P / (wl.gamma - 1.0) + 0.5 * rho * sum(u * u for u in U)])
    wl.grid = GridSpec(GRID_STENCIL, GRIDS[dim], k=8.0 if dim == 1 else 4.0)
    return wl


@pytest.mark.parametrize("eps", [1e-16, 1e-14, 1e-12, 1e-9, 1e-6, 1e-4])
@pytest.mark.parametrize("dim", [1, 2, 3])
def test_small_amplitudes(kbl, monkeypatch, dim, eps):  # noqa: F811
    wl = workload(dim, {1: 12, 2: 5, 3: 3}[dim], eps)
    print(f"[amplitude] {dim}D {eps:g}", flush=True)
    b, s = run(kbl, monkeypatch, wl, TILE[dim])
    rb, rs = oracle.workload_bounds(wl)
    assert np.array_equal(s, rs)
    assert bounds_error(b, rb, dim, stencil_momentum_scale(wl))[0] <= TOL


def timed(kbl, monkeypatch, dim, n, amplitudes):  # noqa: F811
    """Time of a call per amplitude, in us."""
    monkeypatch.setenv("KBL_BOUNDS_TILE", str(TILE[dim]))
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    us = {}
    for eps in amplitudes:
        wl = workload(dim, n, eps)
        vg = kbl.make_vgrid(wl.grid.mode, wl.grid.n[:dim], wl.grid.lo, wl.grid.hi, wl.grid.k)
        prm = kbl.make_params(wl.gamma, r_fac=wl.r_fac)
        args = (t(wl.states), t(wl.rowptr), t(wl.cols), wl.n_s, vg, prm)
        times = []
        for _ in range(8):
            e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
            e0.record()
            for _ in range(5):
                kbl.compute_bounds(*args)
            e1.record()
            e1.synchronize()
            times.append(e0.elapsed_time(e1) * 200.0)
        us[eps] = min(times)
    print(f"[amplitude] {dim}D {us}", flush=True)
    return us


@pytest.mark.parametrize("dim,n", [(2, 100), (3, 14)])
def test_small_amplitudes_are_culled(kbl, monkeypatch, dim, n):  # noqa: F811
    us = timed(kbl, monkeypatch, dim, n, (1e-2, 1e-6))
    assert us[1e-6] <= 1.35 * us[1e-2]


def test_constant_stencils(kbl, monkeypatch):  # noqa: F811
    """Constant fields, with one element of another state: bounds against the oracle,
    and the time of a constant field is no more than that of a varying one."""
    for dim in (1, 2, 3):
        for odd in (False, True):
            wl = workload(dim, {1: 12, 2: 5, 3: 3}[dim], 0.0)
            wl.states = wl.states[:, :1] * np.ones_like(wl.states)
            if odd:
                wl.states[-1, 3 * wl.n_s + 1] *= 1.5
            print(f"[amplitude] {dim}D constant, odd {odd}", flush=True)
            b, s = run(kbl, monkeypatch, wl, TILE[dim])
            rb, rs = oracle.workload_bounds(wl)
            assert np.array_equal(s, rs)
            assert bounds_error(b, rb, dim, stencil_momentum_scale(wl))[0] <= TOL


@pytest.mark.parametrize("dim,n", [(1, 3000), (2, 100), (3, 14)])
def test_constant_stencils_are_culled(kbl, monkeypatch, dim, n):  # noqa: F811
    us = timed(kbl, monkeypatch, dim, n, (1e-2, 0.0))
    assert us[0.0] <= us[1e-2]


def test_constant_stencil_where_q_overflows(kbl, monkeypatch):  # noqa: F811
    """A constant cold state at the corner of a box so long that q is finite in the
    first of its four blocks only, the blocks of one wave in 3D: every wave deals the
    passes alike all the same."""
    for dim, plain in ((2, 1), (3, 6)):
        wl = workload(dim, 3, 0.0)
        wl.states = np.zeros_like(wl.states)
        wl.states[0], wl.states[-1] = 1.0, 1e-150 / (wl.gamma - 1.0)
        hi = (1e80,) + (1e-74,) * (dim - 1)
        wl.grid = GridSpec(GRID_GLOBAL, (16,) + (18,) * (dim - 1), (0.0,) * dim, hi, 0.0)
        print(f"[amplitude] {dim}D constant, q overflows", flush=True)
        b, s = run(kbl, monkeypatch, wl, TILE[dim])
        c, t = run(kbl, monkeypatch, wl, plain)
        assert np.array_equal(s, t) and np.all(np.isfinite(c)) and np.all(c[0] > 1e50)
        np.testing.assert_allclose(b, c, rtol=1e-12, atol=0.0)
