"""1D bounds around the node and state counts where the kernel changes its
split, against the oracle at 1e-12, the FP64 paths' bar."""

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
