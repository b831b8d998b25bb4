"""The calls whose time matters, over the range in which they are used.

A solver calls the bounds and the limiter once per Runge-Kutta stage on every
element of its mesh, so a case is one such call (or a whole limited step) on
a mesh, a velocity grid and a flow: smallest meshes, where launches count, to
millions of elements; 1D, 2D and 3D; element and node stencils; per-stencil
and global velocity boxes; FP64 and the mixed precisions; forward and
backward.  Flows are smooth fields with jumps (four-quadrant and octant
Riemann states, a sine field with a Sod jump, a radial shock), optionally
with node-to-node noise as under-resolved solutions have it.

`listed()` are fixed cases, `draw(rng)` gives others of the same ranges,
`prepare` makes a case's inputs on the GPU from a seed, `run` is one pass,
`exact` the same outputs by direct evaluation in 64 bits, and `work` the
bytes and operations that a pass cannot do without.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2407_20966_amd as kbl

DEV = "cuda:0"
F64 = torch.float64
PRECISIONS = {"fp64": kbl.PREC_FP64, "fp32": kbl.PREC_MIXED_FP32,
              "fp16": kbl.PREC_MIXED_FP16, "bf16": kbl.PREC_MIXED_BF16}
DIM = {"line": 1, "fr1d": 1, "quad": 2, "fr2d": 2, "tri": 2, "hex": 3}

# op: "stage"  compute_bounds + limit (element stencils)
#     "nodes"  compute_bounds_nodes + limit (solution and flux points)
#     "grad"   bounds_and_limit forward and its backward
#     "limit"  the limiter alone, on given bounds
#     "step"   one limited SSP-RK3 step of the 1D flux reconstruction solver
DEFAULTS = dict(op="stage", mesh="quad", n=64, p=3, nu=48, nv=48, box="stencil", precision="fp64",
                field="riemann", rough=0.0, r_fac=1e-3, independent=False, perstate=False,
                target=0.05)


def _case(**kw):
    bad = set(kw) - set(DEFAULTS) - {"name"}
    assert not bad, bad
    return {**DEFAULTS, **kw}


def listed():
    return [
        # a 1D validation run: two launches on 64 elements, all latency
        _case(name="line_64", mesh="line", n=64, nu=64, box="global", field="sine"),
        # a whole limited step of the 1D solver on its usual 2048-node grid
        _case(name="fr1d_step_3200", op="step", mesh="fr1d", n=3200, nu=2048, field="sine"),
        # a small mesh with odd sizes everywhere, independent limiting, noisy flow
        _case(name="quad_45_odd", n=45, p=2, nu=33, nv=41, rough=0.05, independent=True),
        # the stage of a 2D flux reconstruction scheme: node stencils
        _case(name="fr2d_256", op="nodes", mesh="fr2d", n=256),
        # a training or adjoint step: forward and backward, 1% of elements limited
        _case(name="quad_grad_256", op="grad", n=256),
        # the same where the limiter is active in every element
        _case(name="quad_grad_150_dense", op="grad", n=150, target=1.0),
        # a large global grid around a flow with a strong jump
        _case(name="quad_512_global", n=512, nu=64, nv=64, box="global", field="sine"),
        # energy bounds from the per-state integrand
        _case(name="quad_300_energy", n=300, perstate=True, rough=0.01),
        # FP32 envelopes, FP32 contraction
        _case(name="quad_512_fp32", n=512, precision="fp32"),
        # FP32 envelopes, FP16 matrix contraction, uneven stencils
        _case(name="tri_500_fp16", mesh="tri", n=500, p=2, nu=64, nv=64, precision="fp16",
              field="radial"),
        # 3D hexahedra
        _case(name="hex_32", mesh="hex", n=32, p=2, nu=24, nv=24),
        # the largest: two million triangles with uneven stencils
        _case(name="tri_1000", mesh="tri", n=1000, p=2, nu=64, nv=64, field="radial"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["line", "fr1d", "fr2d", "quad", "quad", "quad", "tri", "tri", "hex",
                       "mixed", "mixed", "grad", "grad", "limit", "energy"])
    rough = rng.choice([0.0, 0.0, 0.0, 0.01, 0.05])
    box = rng.choice(["stencil", "stencil", "global"])
    r_fac = rng.choice([1e-3, 1e-3, 0.0])
    if kind == "line":
        return _case(mesh="line", n=_log(rng, 16, 40000), p=rng.randint(1, 5),
                     nu=_log(rng, 40, 2048), box=box, field=rng.choice(["sine", "riemann"]),
                     rough=rough, r_fac=r_fac)
    if kind == "fr1d":
        return _case(op="step", mesh="fr1d", n=_log(rng, 25, 12000), p=rng.randint(1, 6),
                     nu=rng.choice([512, 1000, 2048]), field="sine", r_fac=r_fac)
    if kind == "fr2d":
        return _case(op="nodes", mesh="fr2d", n=_log(rng, 12, 400), p=rng.randint(1, 4),
                     nu=rng.randint(24, 64), nv=rng.randint(24, 64), rough=rough, r_fac=r_fac)
    if kind == "tri":
        return _case(mesh="tri", n=_log(rng, 10, 600), p=2, nu=rng.randint(24, 64),
                     nv=rng.randint(24, 64), field=rng.choice(["radial", "riemann"]),
                     rough=rough, r_fac=r_fac)
    if kind == "hex":
        return _case(mesh="hex", n=_log(rng, 5, 30), p=rng.randint(1, 2), nu=rng.randint(10, 26),
                     nv=rng.randint(10, 26), rough=rough, r_fac=r_fac)
    if kind == "limit":
        return _case(op="limit", n=_log(rng, 16, 900), p=rng.randint(1, 4),
                     target=rng.choice([0.05, 1.0]), independent=rng.random() < 0.3)
    p = rng.randint(1, 4)
    base = dict(n=_log(rng, 12, 700 if p < 4 else 450), p=p, nu=rng.randint(20, 64),
                nv=rng.randint(20, 64), box=box, field=rng.choice(["riemann", "sine"]),
                rough=rough, r_fac=r_fac)
    if kind == "mixed":
        return _case(**base, precision=rng.choice(["fp32", "fp16", "bf16"]))
    if kind == "grad":
        base["n"] = _log(rng, 12, 256)
        base["p"] = min(p, 3)
        return _case(**base, op="grad", target=rng.choice([0.05, 0.05, 1.0]),
                     precision=rng.choice(["fp64", "fp64", "fp32"]))
    if kind == "energy":
        base["n"] = min(base["n"], 400)
        return _case(**base, perstate=True)
    return _case(**base, independent=rng.random() < 0.3)


# ------------------------------------------------------------------- meshes

def _gl(p):
    x, w = np.polynomial.legendre.leggauss(p + 1)
    return x, w


def _rows(cols):
    """Equal-length rows [n_elem, k] as CSR."""
    n, k = cols.shape
    rowptr = torch.arange(0, n * k + 1, k, dtype=torch.int32, device=DEV)
    return rowptr, cols.reshape(-1).to(torch.int32).contiguous()


def _tensor_mesh(dim, n, p):
    """Node coordinates [dim][n_elem, n_s], weights, rowptr, cols of a periodic
    line, quad or hexahedral mesh with face stencils (self first)."""
    x, w = _gl(p)
    n1 = p + 1
    e = torch.arange(n ** dim, device=DEV)
    ids = [(e // n ** k) % n for k in range(dim)]
    j = np.arange(n1 ** dim)
    loc = [(j // n1 ** k) % n1 for k in range(dim)]
    X = [(ids[k][:, None] + torch.tensor(0.5 * (x[loc[k]] + 1.0), device=DEV)[None]) / n
         for k in range(dim)]
    cols = [e]
    for k in range(dim):
        for s in (-1, 1):
            cols.append(e + ((ids[k] + s) % n - ids[k]) * n ** k)
    rowptr, cols = _rows(torch.stack(cols, 1))
    return X, np.prod([w[q] for q in loc], axis=0), rowptr, cols


_TRI = [(0.445948490915965, 0.223381589678011), (0.091576213509771, 0.109951743655322)]


def _tri_mesh(n, gen):
    """2 n^2 jittered P2 triangles, vertex-neighbour stencils."""
    h = 1.0 / n
    nv = n * n
    jit = (torch.rand(2, nv, generator=gen, device=DEV, dtype=F64) - 0.5) * 0.4 * h
    c = torch.arange(nv, device=DEV)
    cx, cy = c % n, c // n

    def corner(a, b):
        v = ((cy + b) % n) * n + (cx + a) % n
        return torch.stack([v.to(F64), (cx + a) * h + jit[0][v], (cy + b) * h + jit[1][v]])

    c00, c10, c01, c11 = corner(0, 0), corner(1, 0), corner(0, 1), corner(1, 1)
    d = (torch.rand(nv, generator=gen, device=DEV) < 0.5)[None, None]
    t1 = torch.where(d, torch.stack([c00, c10, c11], 1), torch.stack([c00, c10, c01], 1))
    t2 = torch.where(d, torch.stack([c00, c11, c01], 1), torch.stack([c10, c11, c01], 1))
    t = torch.stack([t1, t2], 3).reshape(3, 3, 2 * nv)          # [id|x|y, corner, triangle]
    tris = t[0].long().t().contiguous()
    bary, wts = [], []
    for a, w in _TRI:
        b = 1.0 - 2.0 * a
        bary += [(a, a, b), (a, b, a), (b, a, a)]
        wts += [w] * 3
    B = torch.tensor(bary, dtype=F64, device=DEV)
    X = [(B @ t[1]).t().contiguous(), (B @ t[2]).t().contiguous()]
    # triangles around each vertex, then around each triangle's vertices
    nt = tris.shape[0]
    v, order = torch.sort(tris.reshape(-1), stable=True)
    tr = order // 3
    first = torch.searchsorted(v, torch.arange(nv, device=DEV))
    slot = torch.arange(3 * nt, device=DEV) - first[v]
    deg = int(slot.max()) + 1
    table = torch.full((nv, deg), nt, device=DEV)
    table[v, slot] = tr
    cand = table[tris].reshape(nt, 3 * deg)
    own = torch.arange(nt, device=DEV)[:, None]
    cand = torch.sort(torch.where(cand == own, nt, cand), dim=1)[0]
    keep = cand < nt
    keep[:, 1:] &= cand[:, 1:] != cand[:, :-1]
    rowptr = torch.zeros(nt + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(keep.sum(1) + 1, 0)
    cols = torch.empty(int(rowptr[-1]), dtype=torch.int32, device=DEV)
    cols[rowptr[:-1]] = own[:, 0].int()
    at = rowptr[:-1, None] + torch.cumsum(keep, 1)
    cols[at[keep]] = cand[keep].int()
    return X, np.array(wts), rowptr.int(), cols


# -------------------------------------------------------------------- flows

def _smooth(gen, X, modes=8, kmax=4):
    """A periodic smooth field in [-1, 1]."""
    r = lambda *s: torch.rand(*s, generator=gen, device=DEV, dtype=F64)
    amp = 0.5 + 0.5 * r(modes)
    k = torch.randint(-kmax, kmax + 1, (modes, len(X)), generator=gen, device=DEV).to(F64)
    ph = 2 * math.pi * r(modes)
    out = torch.zeros_like(X[0])
    for m in range(modes):
        arg = ph[m]
        for d, x in enumerate(X):
            arg = arg + (2 * math.pi) * k[m, d] * x
        out = out + amp[m] * torch.sin(arg)
    return out / amp.sum()


def _conserved(gamma, rho, U, P):
    ke = 0.5 * rho * sum(u * u for u in U)
    rows = [rho] + [rho * u for u in U] + [P / (gamma - 1.0) + ke]
    return torch.stack([r.reshape(-1) for r in rows]).contiguous()


def _flow(kind, X, rough, gen, gamma, n):
    """Conserved states of a flow at the coordinates X."""
    dim = len(X)
    r = lambda *s: torch.rand(*s, generator=gen, device=DEV, dtype=F64)
    if kind == "riemann":
        cut = (n // 2 + 0.2 + 0.6 * r(dim)) / n
        q = sum((X[d] >= cut[d]).long() << d for d in range(dim))
        m = 1 << dim
        rho0 = torch.exp(math.log(0.1) + math.log(100.0) * r(m))
        p0 = torch.exp(math.log(0.1) + math.log(1000.0) * r(m))
        dirs = torch.randn(m, dim, generator=gen, device=DEV, dtype=F64)
        u0 = 3.0 * r(m)[:, None] * dirs / dirs.norm(dim=1, keepdim=True)
        rho = rho0[q] * (1.0 + 0.01 * _smooth(gen, X))
        P = p0[q] * (1.0 + 0.01 * _smooth(gen, X))
        U = [u0[:, d][q] + 0.03 * _smooth(gen, X) for d in range(dim)]
    elif kind == "sine":
        ph = 2 * math.pi * r(dim + 1)
        left = X[0] < (n // 2 + 0.2 + 0.6 * r(1)) / n
        one = torch.ones_like(X[0])
        rho = (1.25 + 0.75 * torch.sin(2 * math.pi * sum(X) + ph[0])) * torch.where(left, one, 0.125 * one)
        P = torch.where(left, one, 0.1 * one)
        U = [torch.sin(2 * math.pi * X[d] + ph[d + 1]) for d in range(dim)]
    else:
        rad = torch.hypot(X[0] - 0.5, X[1] - 0.5).clamp_min(1e-12)
        inside = rad < 0.3
        one = torch.ones_like(rad)
        rho = torch.where(inside, one, 1e-3 * one) * (1.0 + 0.01 * _smooth(gen, X))
        P = torch.where(inside, one, 1e-5 * one) * (1.0 + 0.01 * _smooth(gen, X))
        speed = 0.5 * torch.where(inside, rad / 0.3, 0.3 / rad)
        U = [speed * (X[d] - 0.5) / rad + 0.005 * _smooth(gen, X) for d in range(2)]
    if rough:
        nz = lambda: 1.0 + rough * (2.0 * r(*rho.shape) - 1.0)
        rho, P = rho * nz(), P * nz()
        c = torch.sqrt(P / rho)
        U = [u + c * (nz() - 1.0) for u in U]
    return _conserved(gamma, rho, U, P), float((P / rho).max())


def _row_of(rowptr):
    n = torch.diff(rowptr.long())
    return torch.repeat_interleave(torch.arange(n.numel(), device=DEV), n)


def _target(states, rowptr, cols, n_s, w, amp, gen):
    """States plus a zero-mean deviation: amp times the stencil's range where
    the density jumps, a small share of it elsewhere (amp 1: everywhere)."""
    nv, nn = states.shape
    ne = nn // n_s
    per = states.reshape(nv, ne, n_s)
    row = _row_of(rowptr)
    big, low = per.amax(2)[:, cols.long()], per.amin(2)[:, cols.long()]
    idx = row[None].expand(nv, -1)
    big = torch.full((nv, ne), -math.inf, dtype=F64, device=DEV).scatter_reduce_(1, idx, big, "amax")
    low = torch.full((nv, ne), math.inf, dtype=F64, device=DEV).scatter_reduce_(1, idx, low, "amin")
    a = torch.where(big[0] / low[0] > 1.5, min(amp, 0.05), 1.0 if amp >= 1.0 else 2e-3)
    s = torch.randint(0, 2, (nv, ne, n_s), generator=gen, device=DEV).to(F64) * 2.0 - 1.0
    c = torch.tensor(w / w.sum(), device=DEV)
    s = s - (s * c).sum(2, keepdim=True)
    return (per + a[None, :, None] * (big - low)[:, :, None] * s).reshape(nv, nn).contiguous()


def _fr_ops(p):
    """Lagrange values at the ends, differentiation matrix and the slopes of
    the DG correction functions on the Gauss-Legendre points."""
    P = np.polynomial.polynomial
    L = np.polynomial.legendre
    x, w = _gl(p)
    at = np.zeros((2, p + 1))
    D = np.zeros((p + 1, p + 1))
    for k in range(p + 1):
        o = np.delete(x, k)
        b = P.polyfromroots(o) / np.prod(x[k] - o)
        at[0, k], at[1, k] = P.polyval(-1.0, b), P.polyval(1.0, b)
        D[:, k] = P.polyval(x, P.polyder(b))
    hi = np.zeros(p + 2)
    lo = np.zeros(p + 2)
    hi[p + 1], lo[p] = 1.0, 1.0
    gl = (-1.0) ** p * 0.5 * (lo - hi)
    gr = 0.5 * (lo + hi)
    return x, w, at, D, L.legval(x, L.legder(gl)), L.legval(x, L.legder(gr))


# ------------------------------------------------------------------ prepare

def _inputs(case, seed):
    """Mesh, states, target and grid of a case, as tensors and numbers."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    mesh, n, p = case["mesh"], case["n"], case["p"]
    dim = DIM[mesh]
    gamma = 1.4
    s = {"dim": dim, "gamma": gamma}
    if mesh == "fr1d":
        x, w = _gl(p)
        X = (torch.arange(n, device=DEV)[:, None] + torch.tensor(0.5 * (x + 1.0), device=DEV)) / n
        U, _ = _flow(case["field"], [X], case["rough"], gen, gamma, n)
        s["U0"] = U.reshape(3, n, p + 1)
        s["left"] = [float(v) for v in U[:, 0]]
        s["right"] = [float(v) for v in U[:, -1]]
        return s
    if mesh == "tri":
        X, w, rowptr, cols = _tri_mesh(n, gen)
    else:
        X, w, rowptr, cols = _tensor_mesh(dim, n, p)
    ne, n_s = X[0].shape
    states, theta = _flow(case["field"], X, case["rough"], gen, gamma, n)
    target = _target(states, rowptr, cols, n_s, w, case["target"], gen)
    if mesh == "fr2d":
        # flux points: the element polynomial on the four faces; elements whose
        # face values are not admissible take their nearest solution points'
        n1 = p + 1
        at = torch.tensor(_fr_ops(p)[2], device=DEV)

        def faces(V):
            V = V.reshape(4, ne, n1, n1)                        # [v, e, jy, jx]
            return torch.cat([V @ at[0], V @ at[1], torch.tensordot(V, at[0], ([2], [0])),
                              torch.tensordot(V, at[1], ([2], [0]))], 2)

        V = states.reshape(4, ne, n1, n1)
        F = faces(states)
        Pf = F[3] - 0.5 * (F[1] ** 2 + F[2] ** 2) / F[0]
        ok = ((F[0] > 0) & (Pf > 0)).all(1)
        near = torch.cat([V[..., 0], V[..., -1], V[:, :, 0], V[:, :, -1]], 2)
        F = torch.where(ok[None, :, None], F, near)
        s["el"] = cols.reshape(ne, 5).long()
        el = s["el"]
        base, e = ne * n_s, torch.arange(ne, device=DEV)
        fl = lambda q, f: base + q[:, None] * (4 * n1) + f * n1 + torch.arange(n1, device=DEV)
        ids = [e[:, None] * n_s + torch.arange(n_s, device=DEV)] + [fl(e, f) for f in range(4)]
        ids += [fl(el[:, 1], 1), fl(el[:, 2], 0), fl(el[:, 3], 3), fl(el[:, 4], 2)]
        rowptr, cols = _rows(torch.cat(ids, 1))
        target = torch.cat([target.reshape(4, ne, n_s), faces(target)], 2).reshape(4, -1).contiguous()
        states = torch.cat([states, F.reshape(4, -1)], 1).contiguous()
        w = np.concatenate([w, np.zeros(4 * n1)])
        n_s = n_s + 4 * n1
    half = 12.0 * math.sqrt(theta)
    s |= dict(states=states, target=target, rowptr=rowptr, cols=cols, w=w, n_s=n_s, ne=ne,
              half=half)
    return s


def _grid(case, s):
    n = {1: (case["nu"],), 2: (case["nu"], case["nv"]),
         3: (case["nu"], case["nv"], case["nu"])}[s["dim"]]
    k = 8.0 if s["dim"] == 1 else 4.0
    if case["box"] == "global":
        return kbl.make_vgrid(kbl.GRID_GLOBAL, n, (-s["half"],) * s["dim"], (s["half"],) * s["dim"])
    return kbl.make_vgrid(kbl.GRID_STENCIL, n, k=k)


def prepare(case, seed):
    s = _inputs(case, seed)
    s["op"] = case["op"]
    if case["op"] == "step":
        f = kbl.FR1D(case["p"], case["n"], 0.0, 1.0, s["gamma"], bc="dirichlet", left=s["left"],
                     right=s["right"], r_fac=case["r_fac"], n_u=case["nu"], device=DEV)
        f.set_solution(s["U0"])
        s["solver"], s["start"] = f, f.U.clone()
        s["dt"] = 0.1 / case["n"] / ((2 * case["p"] + 1) * f.max_speed())
        return s
    s["vgrid"] = _grid(case, s)
    s["params"] = kbl.make_params(s["gamma"], r_fac=case["r_fac"],
                                  precision=PRECISIONS[case["precision"]],
                                  independent_alpha=case["independent"],
                                  energy_perstate=case["perstate"])
    if case["op"] == "limit":
        s["bounds"] = _simple_bounds(s)
    if case["op"] == "grad":
        gen = torch.Generator(device=DEV).manual_seed(seed + 1)
        s["G"] = torch.randn(s["target"].shape, generator=gen, device=DEV, dtype=F64)
        s["states"].requires_grad_(True)
        s["target"].requires_grad_(True)
    return s


def _simple_bounds(s):
    """Bounds as a solver keeps them from an earlier call: the stencil's own
    range of every variable, a little widened."""
    nv = s["states"].shape[0]
    per = s["states"].reshape(nv, s["ne"], s["n_s"])
    c = s["cols"].reshape(s["ne"], -1).long()
    hi, lo = per.amax(2)[:, c].amax(2), per.amin(2)[:, c].amin(2)
    return torch.cat([lo - 1e-3 * lo.abs(), hi + 1e-3 * hi.abs()]).contiguous()


def run(s):
    op = s["op"]
    if op == "step":
        f = s["solver"]
        f.U.copy_(s["start"])            # the step is taken from the same state each time
        f.step(s["dt"])
        return {"U": f.solution()}
    if op == "grad":
        lim = kbl.bounds_and_limit(s["states"], s["target"], s["rowptr"], s["cols"], s["n_s"],
                                   s["vgrid"], s["params"], s["w"])
        gs, gt = torch.autograd.grad(lim, (s["states"], s["target"]), s["G"])
        return {"limited": lim.detach(), "grad_states": gs, "grad_solution": gt}
    if op == "limit":
        lim, alpha, st = kbl.limit(s["target"], s["bounds"], s["w"], s["n_s"], s["params"])
        return {"limited": lim, "alpha": alpha, "lstatus": st}
    if op == "nodes":
        b, bst = kbl.compute_bounds_nodes(s["states"], s["rowptr"], s["cols"], s["vgrid"], s["params"])
    else:
        b, bst = kbl.compute_bounds(s["states"], s["rowptr"], s["cols"], s["n_s"], s["vgrid"],
                                    s["params"])
    lim, alpha, st = kbl.limit(s["target"], b, s["w"], s["n_s"], s["params"])
    return {"bounds": b, "bstatus": bst, "limited": lim, "alpha": alpha, "lstatus": st}


# -------------------------------------------------------------------- exact

def _pressure(gm1, w):
    return gm1 * (w[-1] - 0.5 * (w[1:-1] ** 2).sum(0) / w[0])


def _bounds64(st, half, gamma, n, k, r_fac, perstate, smask=None):
    """Bounds [2(d+2), c] of stencil states st [d+2, c, S] by direct evaluation."""
    d = st.shape[0] - 2
    gm1 = gamma - 1.0
    hd = 0.5 * max(0.0, (2.0 - d * gm1) / gm1)
    rho, U = st[0], st[1:-1] / st[0]
    th = _pressure(gm1, st) / rho
    neg = None if smask is None else ~smask
    ax, wt, fac = [], [], []
    for j in range(d):
        m = n[j]
        if half is None:
            sd = k * torch.sqrt(th)
            lo, hi = U[j] - sd, U[j] + sd
            if neg is not None:
                lo, hi = lo.masked_fill(neg, math.inf), hi.masked_fill(neg, -math.inf)
            lo, hi = lo.amin(1, keepdim=True), hi.amax(1, keepdim=True)
        else:
            lo, hi = st.new_full((st.shape[1], 1), -half), st.new_full((st.shape[1], 1), half)
        h = (hi - lo) / (m - 1)
        v = lo + torch.arange(m, device=st.device, dtype=F64) * h
        q = torch.ones(m, device=st.device, dtype=F64)
        q[0] = q[-1] = 0.5
        ax.append(v)
        wt.append(h * q)
        fac.append(torch.exp(-(v[:, None, :] - U[j][:, :, None]) ** 2 / (2.0 * th[:, :, None])))
    g = (rho * (2 * math.pi * th) ** (-0.5 * d))[:, :, None] * fac[0]        # [c, S, n0]
    for f in fac[1:]:
        g = (g[..., None] * f.reshape(f.shape[:2] + (1,) * (g.dim() - 2) + (-1,)))
    c = g.shape[0]
    one = (c,) + (1,) * d
    pos = lambda x, j: x.reshape((c,) + tuple(-1 if i == j else 1 for i in range(d)))
    M = sum(torch.log(pos(wt[j], j)) for j in range(d)).exp()
    V = [pos(ax[j], j).expand((c,) + tuple(n[:d])) for j in range(d)]
    V2 = 0.5 * sum(v * v for v in V)
    gI = (hd * th).reshape(th.shape + (1,) * d)

    def ext(x):
        if neg is None:
            return x.amin(1), x.amax(1)
        mask = neg.reshape(neg.shape + (1,) * d)
        return x.masked_fill(mask, math.inf).amin(1), x.masked_fill(mask, -math.inf).amax(1)

    fmin, fmax = ext(g)
    emin, emax = ext(g * (V2[:, None] + gI)) if perstate else ext(g * gI)
    lo_f, hi_f = (1.0 - r_fac), (1.0 + r_fac)
    fmin, fmax, emin, emax = lo_f * fmin, hi_f * fmax, lo_f * emin, hi_f * emax
    total = lambda x: (M * x).flatten(1).sum(1)
    lower, upper = [total(fmin)], [total(fmax)]
    for v in V:
        lower.append(total(torch.where(v < 0, v * fmax, v * fmin)))
        upper.append(total(torch.where(v < 0, v * fmin, v * fmax)))
    lower.append(total(emin if perstate else V2 * fmin + emin))
    upper.append(total(emax if perstate else V2 * fmax + emax))
    lower[0] = lower[0].clamp_min(1e-12)
    return torch.stack(lower + upper)


def _limit64(w, b, weights, gamma, independent):
    """Limited nodes [d+2, c, n_s] and alpha [2, c]."""
    nv = w.shape[0]
    c = torch.tensor(weights / weights.sum(), device=w.device)
    mean = (w * c).sum(2)
    big, low = w.amax(2), w.amin(2)
    du, dl = (big - mean).abs(), (low - mean).abs()
    flat = (du < 1e-13) | (dl < 1e-13)
    one = torch.ones_like(du)
    up = (b[nv:] - mean).abs() / torch.where(flat, one, du)
    lo = (b[:nv] - mean).abs() / torch.where(flat, one, dl)
    a = torch.where(flat, torch.zeros_like(one), torch.minimum(torch.minimum(up, lo), one))
    amin = a.amin(0)
    a = a if independent else amin[None].expand_as(a)
    x = mean[:, :, None] + a[:, :, None] * (w - mean[:, :, None])
    pm = _pressure(gamma - 1.0, x).amin(1)
    pb = _pressure(gamma - 1.0, mean)
    fire = pm < 1e-12
    safe = torch.where(fire, pm - pb, -torch.ones_like(pm))
    ap = torch.where(fire, torch.where(pb > 1e-12, ((1e-12 - pb) / safe).abs(), torch.zeros_like(pm)),
                     torch.ones_like(pm))
    y = torch.where(fire[None, :, None], mean[:, :, None] + ap[None, :, None] * (x - mean[:, :, None]), x)
    return y, torch.stack([amin, ap])


def _chunks(case, s, copies):
    """Element ranges whose pair tensors take a few GiB each."""
    S = int(torch.diff(s["rowptr"].long()).max()) * (1 if case["op"] == "nodes" else s["n_s"])
    n = {1: case["nu"], 2: case["nu"] * case["nv"], 3: case["nu"] ** 2 * case["nv"]}[s["dim"]]
    step = max(1, int(6e9 / copies / (8 * S * n)))
    return [(a, min(a + step, s["ne"])) for a in range(0, s["ne"], step)]


def _stencil(case, s, states, a, b):
    """States [d+2, c, S] of the rows a..b and their mask (None: all rows full)."""
    rp = s["rowptr"].long()
    n = torch.diff(rp)[a:b]
    k = int(n.max())
    at = rp[a:b, None] + torch.arange(k, device=DEV)
    mask = torch.arange(k, device=DEV)[None] < n[:, None]
    col = s["cols"].long()[torch.where(mask, at, rp[a:b, None])]
    n_s = 1 if case["op"] == "nodes" else s["n_s"]
    nodes = (col[:, :, None] * n_s + torch.arange(n_s, device=DEV)).reshape(b - a, -1)
    full = bool(mask.all())
    return states[:, nodes], None if full else mask[:, :, None].expand(-1, -1, n_s).reshape(b - a, -1)


def exact(case, seed):
    s = _inputs(case, seed)
    if case["op"] == "step":
        return _step64(case, s)
    if _pairs(case) > (2e10 if case["op"] == "grad" else 4e11):
        return None
    d, nv = s["dim"], s["dim"] + 2
    n = (case["nu"], case["nv"], case["nu"]) if d > 1 else (case["nu"],)
    half = s["half"] if case["box"] == "global" else None
    k = 8.0 if d == 1 else 4.0
    per = s["target"].reshape(nv, s["ne"], s["n_s"])
    if case["op"] == "limit":
        lim, alpha = _limit64(per, _simple_bounds(s), s["w"], s["gamma"], case["independent"])
        return {"limited": lim.reshape(nv, -1), "alpha": alpha, "lstatus": None}
    if case["op"] == "grad":
        G = torch.randn(s["target"].shape, device=DEV, dtype=F64,
                        generator=torch.Generator(device=DEV).manual_seed(seed + 1))
        Gp = G.reshape(per.shape)
        states = s["states"].requires_grad_(True)
        gs, gt, lim = torch.zeros_like(states), torch.zeros_like(per), torch.empty_like(per)
        for a, b in _chunks(case, s, 10):
            w = per[:, a:b].clone().requires_grad_(True)
            st, mask = _stencil(case, s, states, a, b)
            y, _ = _limit64(w, _bounds64(st, half, s["gamma"], n, k, case["r_fac"],
                                         case["perstate"], mask), s["w"], s["gamma"], False)
            ga, gb = torch.autograd.grad(y, (states, w), Gp[:, a:b])
            gs += ga
            gt[:, a:b] = gb
            lim[:, a:b] = y.detach()
        f = lambda x: x.reshape(nv, -1)
        if case["precision"] != "fp64":
            gs = None                # which bound binds differs with the bounds' precision
        return {"limited": f(lim), "grad_states": gs, "grad_solution": None if gs is None else f(gt)}
    bs = torch.empty(2 * nv, s["ne"], dtype=F64, device=DEV)
    for a, b in _chunks(case, s, 3):
        st, mask = _stencil(case, s, s["states"], a, b)
        bs[:, a:b] = _bounds64(st, half, s["gamma"], n, k, case["r_fac"], case["perstate"], mask)
    lim, alpha = _limit64(per, bs, s["w"], s["gamma"], case["independent"])
    return {"bounds": bs, "bstatus": None, "limited": lim.reshape(nv, -1), "alpha": alpha,
            "lstatus": None}


def _step64(case, s):
    """One limited SSP-RK3 step of the flux reconstruction scheme."""
    n, p, g = case["n"], case["p"], s["gamma"]
    T = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=F64, device=DEV)
    x, w, at, D, dl, dr = _fr_ops(p)
    at, D, dl, dr = T(at), T(D), T(dl), T(dr)
    left, right = T(s["left"])[:, None], T(s["right"])[:, None]
    wv = np.concatenate([w, [0.0, 0.0]])

    def flux(u):
        v, P = u[1] / u[0], _pressure(g - 1.0, u)
        return torch.stack([u[1], u[1] * v + P, (u[2] + P) * v])

    def hllc(L, R):
        ul, ur, pl, pr = L[1] / L[0], R[1] / R[0], _pressure(g - 1, L), _pressure(g - 1, R)
        cl, cr = torch.sqrt(g * pl / L[0]), torch.sqrt(g * pr / R[0])
        a, b = torch.minimum(ul - cl, ur - cr), torch.maximum(ul + cl, ur + cr)
        ql, qr = L[0] * (a - ul), R[0] * (b - ur)
        m = (pr - pl + ul * ql - ur * qr) / (ql - qr)

        def side(W, u, P, q, S):
            f = q / (S - m)
            star = torch.stack([f, f * m, f * (W[2] / W[0] + (m - u) * (m + P / q))])
            return flux(W) + S * (star - W)

        out = torch.where(b >= 0, side(R, ur, pr, qr, b), flux(R))
        out = torch.where(m >= 0, side(L, ul, pl, ql, a), out)
        return torch.where(a >= 0, flux(L), out)

    ends = lambda u: (u @ at[0], u @ at[1])

    def rhs(u):
        F = flux(u)
        a, b = ends(u)
        Fr = hllc(torch.cat([left, b], 1), torch.cat([a, right], 1))
        fa, fb = ends(F)
        d = F @ D.t() + (Fr[:, :-1] - fa)[..., None] * dl + (Fr[:, 1:] - fb)[..., None] * dr
        return -2.0 * n * d

    def nodes(u):
        a, b = ends(u)
        return torch.cat([u, a[..., None], b[..., None]], 2)

    def bounds(st):
        out = []
        for a in range(0, n, 4096):
            out.append(_bounds64(st[:, a:a + 4096], None, g, (case["nu"],), 8.0, case["r_fac"], False))
        return torch.cat(out, 1)

    def stage(u, mix):
        a, b = ends(u)
        st = torch.cat([nodes(u), torch.cat([left, b[:, :-1]], 1)[..., None],
                        torch.cat([a[:, 1:], right], 1)[..., None]], 2)
        y, _ = _limit64(nodes(mix(u + dt * rhs(u))), bounds(st), wv, g, False)
        return y[..., :p + 1]

    # initial data: elements with a node that is not admissible are limited first
    u = s["U0"]
    v = nodes(u)
    P = _pressure(g - 1.0, v)
    bad = ~((v[0] > 0) & (P > 0)).all(1)
    if bool(bad.any()):
        gl, gr = left[:, :, None].expand(3, 1, p + 1), right[:, :, None].expand(3, 1, p + 1)
        st = torch.cat([u, torch.cat([gl, u[:, :-1]], 1), torch.cat([u[:, 1:], gr], 1)], 2)
        y, _ = _limit64(v, bounds(st), wv, g, False)
        u = torch.where(bad[None, :, None], y[..., :p + 1], u)
    speed = ((u[1] / u[0]).abs() + torch.sqrt(g * _pressure(g - 1.0, u) / u[0])).max()
    dt = 0.1 / n / ((2 * p + 1) * speed)
    u1 = stage(u, lambda z: z)
    u2 = stage(u1, lambda z: 0.75 * u + 0.25 * z)
    return {"U": stage(u2, lambda z: u / 3.0 + 2.0 / 3.0 * z)}


# --------------------------------------------------------------------- work

def _shape(case):
    """(dim, elements, nodes per element, stencil states per element, listed ids
    per element, velocity nodes)."""
    d, n, p = DIM[case["mesh"]], case["n"], case["p"]
    m = {1: case["nu"], 2: case["nu"] * case["nv"], 3: case["nu"] ** 2 * case["nv"]}[d]
    if case["mesh"] == "tri":
        return d, 2 * n * n, 6, 6 * 13, 13, m
    if case["mesh"] == "fr1d":
        return d, n, p + 1, p + 5, p + 5, m
    n_s = (p + 1) ** d
    if case["mesh"] == "fr2d":
        S = n_s + 8 * (p + 1)
        return d, n * n, n_s, S, S, m
    return d, n ** d, n_s, (2 * d + 1) * n_s, 2 * d + 1, m


def _pairs(case):
    d, ne, _, S, _, m = _shape(case)
    return ne * S * m


def work(case):
    d, ne, n_s, S, ids, m = _shape(case)
    nv = d + 2
    node = 8 * nv * ne * n_s
    # the limiter: nodes and bounds in, limited nodes, alpha and status out
    lim_bytes, lim_flops = 2 * node + 8 * 2 * nv * ne + 20 * ne, ne * n_s * nv * 8
    if case["mesh"] == "fr2d":
        lim_bytes += 2 * 8 * nv * ne * 4 * (case["p"] + 1)
    # the bounds: every state once, the stencil ids, bounds and status out; the
    # coefficients of every state of a stencil, and at every velocity node the
    # four envelope values formed, compared and summed into the moments
    b_bytes = node + 4 * ne * (ids + 1) + 8 * 2 * nv * ne + 4 * ne
    b_flops = ne * (30.0 * S + 20.0 * m)
    if case["op"] == "limit":
        return {"bytes": lim_bytes, "flops": lim_flops}
    if case["op"] == "step":
        return {"bytes": 2 * node, "flops": 3 * (b_flops + lim_flops + ne * n_s * (6 * n_s + 60))}
    if case["op"] == "grad":
        # the backward: inputs, bounds and the incoming gradient in, two gradients
        # out; envelopes again only in elements where a bound binds
        share = 1.0 if case["target"] >= 1.0 else 0.01
        return {"bytes": b_bytes + lim_bytes + 5 * node,
                "flops": b_flops * (1.0 + share) + 3 * lim_flops}
    return {"bytes": b_bytes + lim_bytes, "flops": b_flops + lim_flops}
