"""1D bounds where the default rule changes the kernel: node counts around the
splits, few and many elements, stencils beyond the staged states.  Bounds against
the oracle (1e-12, the FP64 paths' bar), times against the same call's at half the
states."""

import numpy as np
import pytest

import oracle
import synth
from synth.workloads import GRID_STENCIL, GridSpec
from tests._parity import bounds_error, stencil_momentum_scale
from tests.test_gpu_1d import kbl  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-12


def line(n_elem, p, k, nu, seed):
    """k consecutive elements of p + 1 nodes per stencil, nu velocity nodes."""
    wl = synth.make_line_workload(n_elem=n_elem, p=p, seed=seed, name="line_sizes")
    e = np.arange(n_elem)[:, None]
    wl.cols = ((e + np.arange(k)[None, :]) % n_elem).astype(np.int32).ravel()
    wl.rowptr = np.arange(0, n_elem * k + 1, k).astype(np.int32)
    wl.grid = GridSpec(GRID_STENCIL, (nu,), k=8.0)
    return wl


def device_call(kbl, wl):  # noqa: F811
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    args = (t(wl.states), t(wl.rowptr), t(wl.cols), wl.n_s,
            kbl.make_vgrid(wl.grid.mode, wl.grid.n, wl.grid.lo, wl.grid.hi, wl.grid.k),
            kbl.make_params(wl.gamma, r_fac=wl.r_fac))
    return lambda: kbl.compute_bounds(*args)


def check(kbl, wl):  # noqa: F811
    print(f"[1d] {wl.n_elem} elements, {wl.stencil_sizes()[0] * wl.n_s} states, {wl.grid.n[0]} nodes",
          flush=True)
    b, s = device_call(kbl, wl)()
    elems = synth.sample_elements(wl, 24) if wl.n_elem > 64 else np.arange(wl.n_elem)
    rb, rs = oracle.workload_bounds(wl, elems=elems)
    b, s = b.cpu().numpy()[:, elems], s.cpu().numpy().view(np.uint32)[elems]
    assert np.array_equal(s, rs)
    assert bounds_error(b, rb, 1, stencil_momentum_scale(wl, elems))[0] <= TOL


def best_us(call):
    call()
    times = []
    for _ in range(8):
        e0, e1 = torch.cuda.Event(True), torch.cuda.Event(True)
        e0.record()
        for _ in range(10):
            call()
        e1.record()
        e1.synchronize()
        times.append(e0.elapsed_time(e1) * 100.0)
    return min(times)


@pytest.mark.parametrize("nu", [2, 64, 65, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096])
def test_stencils_beyond_the_staged_states(kbl, nu):  # noqa: F811
    check(kbl, line(6, 6, 37, nu, 300 + nu))          # 259 states: a chunk of three
    check(kbl, line(5, 7, 64, nu, 301 + nu))          # 512: two full chunks


def test_stencils_beyond_the_staged_states_are_staged_once(kbl):  # noqa: F811
    us = {k: best_us(device_call(kbl, line(1000, 4, k, 2048, 310))) for k in (30, 60)}
    print(f"[1d] us by elements per stencil: {us}", flush=True)
    assert us[60] <= 2.0 * us[30]          # 300 and 150 states


@pytest.mark.parametrize("nu", [257, 384, 385, 511, 512, 513, 768, 769, 1023, 1024])
@pytest.mark.parametrize("n_elem", [40, 767, 768, 1023, 1024])
def test_splits_by_mesh_size(kbl, n_elem, nu):  # noqa: F811
    for p, k in ((2, 1), (2, 3), (3, 3), (5, 3)):      # 3, 9, 12 and 18 states
        check(kbl, line(n_elem, p, k, nu, 320 + nu))
