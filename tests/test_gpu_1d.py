"""The 1D kernels at their edges: a limited step of the FR solver (one kernel
per stage) against the same step composed of the library's residual, bounds
and limiter entry points, and 1D bounds around the node and state counts where
the kernel changes its split, against the oracle.

Tolerances: the composed step runs the same formulas on the same inputs, so
three stages differ by rounding alone: 1e-12 of the element value scale (200
times the 5e-15 of a few dozen roundings).  Bounds: 1e-12, the FP64 paths'
bar against the oracle."""

import numpy as np
import pytest

import oracle
from oracle import fr1d as ofr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kbl():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2407_20966_amd as kbl
    return kbl


def states_1d(rng, shape, gamma, amp):
    ex = shape[:-1] + (1,)
    f = lambda lo, hi: rng.uniform(lo, hi, ex) + amp * rng.uniform(-1, 1, shape)
    return ofr.conserved(np.exp(f(-1, 1)), f(-1, 1), np.exp(f(-1, 1)), gamma)


def composed_step(kbl, g, o, dt):
    """(U [3, n_tot, n_v], status) of one step from g's residual and the bounds and
    limiter entry points."""
    n_v, n_tot, rowptr, cols = o.stencil_layout()
    dev = g.U.device
    rowptr, cols = torch.from_numpy(rowptr).to(dev), torch.from_numpy(cols).to(dev)
    at = torch.tensor(np.stack([o.at_m1, o.at_p1], 1), device=dev)
    cw = np.concatenate([o.w, [0.0, 0.0]])

    def layout(points):
        V = torch.cat([points, points @ at], 2)
        if o.bc == "dirichlet":
            ghosts = torch.tensor(np.stack([o.left, o.right], 1), device=dev)
            V = torch.cat([V, ghosts[:, :, None].expand(3, 2, n_v)], 1)
        return V.reshape(3, n_tot * n_v).contiguous()

    points = g.solution()
    u0, V, st = points, layout(points), None
    for a, b in ((0.0, 1.0), (0.75, 0.25), (1.0 / 3.0, 2.0 / 3.0)):
        bnd, _ = kbl.compute_bounds_nodes(V, rowptr, cols, g.vgrid, g.params)
        g.solution_view().copy_(points)
        new = a * u0 + b * (points + dt * g.rhs())
        V, _, st = kbl.limit(layout(new), bnd, cw, n_v, g.params)
        points = V.view(3, n_tot, n_v)[:, :o.n_elem, :o.p + 1].contiguous()
    return V.view(3, n_tot, n_v), st


CASES = [  # p, n_elem, velocity nodes, bc, options
    (1, 2, 2, "periodic", {}),
    (2, 9, 63, "dirichlet", {}),
    (3, 8, 64, "periodic", {"independent": True}),
    (4, 7, 65, "dirichlet", {"box": True}),
    (5, 17, 256, "periodic", {"bad": True}),
    (6, 5, 257, "dirichlet", {"bad": True, "independent": True}),
    (7, 33, 513, "dirichlet", {"gamma": 3.0}),
    (7, 11, 2048, "periodic", {"box": True, "r_fac": 0.0}),
    (3, 16, 4096, "dirichlet", {"p_floor": 0.8}),
]


@pytest.mark.parametrize("p,n,nu,bc,opt", CASES)
def test_limited_step_matches_composition(kbl, p, n, nu, bc, opt):
    rng = np.random.default_rng(100 * p + n)
    gamma = opt.get("gamma", 1.4)
    left, right = (ofr.conserved(*[np.array(x) for x in s], gamma)
                   for s in ((1.1, 0.2, 0.9), (0.4, -0.1, 0.5)))
    U = states_1d(rng, (n, p + 1), gamma, 0.02)
    if opt.get("bad"):
        U[2, n // 2, 0] = 0.1 * U[1, n // 2, 0] ** 2 / U[0, n // 2, 0] - 0.5   # P < 0
    g, ref = (kbl.FR1D(p, n, 0.0, 1.0, gamma, bc=bc, left=left, right=right, n_u=nu)
              for _ in range(2))
    o = ofr.FR1D(p, n, 0.0, 1.0, gamma, bc=bc, left=left, right=right)
    for s in (g, ref):
        s.params = kbl.make_params(gamma, r_fac=opt.get("r_fac", 1e-3),
                                   p_floor=opt.get("p_floor", 1e-12),
                                   independent_alpha=opt.get("independent", False))
        if opt.get("box"):
            s.vgrid = kbl.make_vgrid(kbl.GRID_GLOBAL, (nu,), (-14.0,), (15.0,))
        s.solution_view().copy_(torch.from_numpy(U))
    dt = 0.3 / n / (2 * p + 1) / 5.0
    print(f"[1d] step p {p} n {n} nodes {nu} {bc} {opt}", flush=True)
    g.step(dt)
    V, st = composed_step(kbl, ref, o, dt)
    torch.cuda.synchronize()
    got, want = g.U.cpu().numpy().reshape(3, -1, p + 3), V.cpu().numpy()
    nan = np.isnan(want)
    assert np.array_equal(np.isnan(got), nan)
    a = np.nan_to_num(np.abs(want)).max(2)
    a[1] = np.maximum(a[1], np.sqrt(np.abs(a[0] * a[2])))
    err = np.where(nan, 0.0, np.abs(got - want) / np.maximum(a[:, :, None], 1e-300)).max()
    sg, sw = (x.cpu().numpy().view(np.uint32) for x in (g.status, st))
    print(f"[1d] err {err:.2e}, limited {(sw[:n] != 0).sum()}, nan {nan.sum()}", flush=True)
    assert err <= 1e-12
    assert np.array_equal(sg[:n], sw[:n])


@pytest.mark.parametrize("n_s,width,nu", [(4, 3, 2), (5, 3, 64), (6, 3, 65), (16, 16, 256),
                                          (64, 4, 257), (43, 6, 300), (64, 9, 513),
                                          (2, 3, 4095)])
def test_bounds_1d(kbl, n_s, width, nu):
    rng = np.random.default_rng(n_s + nu)
    n = 40
    U = states_1d(rng, (n, n_s), 1.4, 0.1).reshape(3, -1)
    cols = ((np.arange(n)[:, None] + np.arange(width)[None] - width // 2) % n).astype(np.int32)
    rowptr = np.arange(0, n * width + 1, width, dtype=np.int32)
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    vg = kbl.make_vgrid(kbl.GRID_STENCIL, (nu,), k=8.0)
    print(f"[1d] bounds states {n_s * width} nodes {nu}", flush=True)
    b, s = kbl.compute_bounds(t(U), t(rowptr), t(cols.reshape(-1)), n_s, vg, kbl.make_params(1.4))
    rb, rs = oracle.bounds(1, 1.4, U, rowptr, cols.reshape(-1), n_s, kbl.GRID_STENCIL, (nu,),
                           k=8.0, r_fac=1e-3)
    b = b.cpu().numpy()
    assert np.array_equal(s.cpu().numpy().view(np.uint32), rs)
    a = np.abs(rb)
    a[[1, 4]] = np.maximum(a[[1, 4]], np.sqrt(a[3] * a[5]))   # momentum scale sqrt(rho E)
    err = (np.abs(b - rb) / np.maximum(a, 1e-300)).max()   # a bound may underflow to 0
    print(f"[1d] err {err:.2e}", flush=True)
    assert err <= 1e-12


# state counts around the cull's lane groups (16, 32, 64) and its lower bound (10),
# grids of two to nine rounds with a remainder; wide boxes, no internal degrees of
# freedom, and states that tie (all equal, nearly equal)
@pytest.mark.parametrize("n_s,width,nu", [(5, 2, 4096), (3, 4, 513), (4, 4, 2048), (17, 1, 700),
                                          (16, 2, 1025), (11, 3, 1500), (16, 4, 2048),
                                          (13, 5, 1100), (3, 3, 2048)])
@pytest.mark.parametrize("kind", ["wide", "monatomic", "equal", "near"])
def test_bounds_1d_cull(kbl, n_s, width, nu, kind):
    rng = np.random.default_rng(7 * n_s + nu)
    n, gamma = 24, 3.0 if kind == "monatomic" else 1.4
    U = states_1d(rng, (n, n_s), gamma, 0.2)
    if kind in ("equal", "near"):
        U = np.broadcast_to(U[:, :1, :1], U.shape) * (
            1.0 + (1e-9 if kind == "near" else 0.0) * rng.uniform(-1, 1, U.shape))
    U = np.ascontiguousarray(U.reshape(3, -1))
    cols = ((np.arange(n)[:, None] + np.arange(width)[None]) % n).astype(np.int32).reshape(-1)
    rowptr = np.arange(0, n * width + 1, width, dtype=np.int32)
    box = dict(lo=(-40.0,), hi=(35.0,)) if kind == "wide" else dict(k=8.0)
    mode = kbl.GRID_GLOBAL if kind == "wide" else kbl.GRID_STENCIL
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(a).to(dev)
    print(f"[1d] cull {kind} states {n_s * width} nodes {nu}", flush=True)
    b, s = kbl.compute_bounds(t(U), t(rowptr), t(cols), n_s, kbl.make_vgrid(mode, (nu,), **box),
                              kbl.make_params(gamma))
    rb, rs = oracle.bounds(1, gamma, U, rowptr, cols, n_s, mode, (nu,), r_fac=1e-3,
                           **{**box, "lo": (*box.get("lo", (0.0,)), 0.0),
                              "hi": (*box.get("hi", (0.0,)), 0.0)})
    b = b.cpu().numpy()
    assert np.array_equal(s.cpu().numpy().view(np.uint32), rs)
    a = np.abs(rb)
    a[[1, 4]] = np.maximum(a[[1, 4]], np.sqrt(a[3] * a[5]))
    err = (np.abs(b - rb) / np.maximum(a, 1e-300)).max()
    print(f"[1d] err {err:.2e}", flush=True)
    assert err <= 1e-12
