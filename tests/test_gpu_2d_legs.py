"""The 2D legs (up to two sweeps and the transfer beside them on 32 x 32 tiles)
and the coarse-level kernel (levels n <= 64) against the 2D oracle at the sizes
where their indexing can go wrong: a grid one node short of, at and past a tile
or the coarse-level kernel's limit, odd grids, a coarsest grid above that limit,
and sweep counts that change how the legs alternate between the arrays.

Tolerance 1e-12 of max |u| as in the other oracle comparisons: the GPU and the
oracle evaluate the same formulas in a different order, and each update divides
differences of order eps |u| by nothing smaller than 1 (u_p += sigma h^2 / 2)."""
import sys

import numpy as np
import pytest

from oracle import ma2
from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
TOL = 1e-12
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def note(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def start(p, seed, amp=0.01):
    rng = np.random.default_rng(seed)
    return P.initial_guess2(p, p.u_exact * (1 + amp * rng.standard_normal(p.u_exact.shape)))


def solver(n, order, rm, **kw):
    from paper_1411_7018_amd.solver2d import Solver2D
    return Solver2D(n, order=order, restriction="half" if rm == 0 else "full", **kw)


@pytest.mark.parametrize("n,count", [(30, 1), (31, 3), (32, 2), (63, 5), (64, 4), (95, 1),
                                     (97, 3), (131, 6)])
@pytest.mark.parametrize("order", ["rb", "4c"])
def test_sweeps(n, count, order):
    """Odd and even numbers of legs; some F <= 0, whose count has to be the
    oracle's although halo nodes are updated by several tiles."""
    note("legs sweep", n, count, order)
    p = P.example2d(1, n)
    f = p.f.copy()
    f[1:-1:7, 2:-1:5] = -0.5
    u0 = start(p, n)
    want = u0.copy()
    bad = sum(ma2.sweep(want, f, order) for _ in range(count))
    u = dev(u0)
    assert solver(n, order, 0).sweep(u, dev(f), count) == bad > 0
    assert np.abs(host(u) - want).max() <= TOL * np.abs(want).max()


@pytest.mark.parametrize("n", [62, 64, 66, 68, 96, 124, 128, 130, 192, 260])
@pytest.mark.parametrize("order,rm", [("rb", 0), ("rb", 1), ("4c", 0), ("4c", 1)])
def test_vcycle_then_fmg(n, order, rm):
    """130 ends on 65 and 62 on 31: coarsest grids above and below the
    coarse-level kernel's limit."""
    note("legs vcycle", n, order, rm)
    p = P.example2d(1, n)
    pr = ma2.params(order=order, rmode=rm)
    s = solver(n, order, rm)
    want = start(p, n, 1e-4)
    u = dev(want)
    ma2.vcycle(want, p.f, pr)
    s.vcycle(u, dev(p.f))
    assert np.abs(host(u) - want).max() <= TOL * np.abs(want).max()
    ma2.fmg(want, p.f, pr)
    s.fmg(u, dev(p.f))
    assert np.abs(host(u) - want).max() <= TOL * np.abs(want).max()


@pytest.mark.parametrize("nu1,nu2,nu0", [(0, 1, 1), (1, 0, 1), (1, 1, 2), (3, 1, 1), (2, 3, 1),
                                         (1, 4, 3), (4, 2, 1), (3, 5, 2), (0, 0, 1)])
@pytest.mark.parametrize("n,order", [(136, "rb"), (136, "4c"), (32, "rb")])
def test_sweep_counts(nu1, nu2, nu0, n, order):
    note("legs counts", nu1, nu2, nu0, n, order)
    p = P.example2d(1, n)
    pr = ma2.params(order=order, rmode=1, nu1=nu1, nu2=nu2, nu0=nu0)
    s = solver(n, order, 1, nu1=nu1, nu2=nu2, nu0=nu0)
    want = start(p, n, 1e-4)
    u, f = dev(want), dev(p.f)
    for _ in range(2):
        ma2.vcycle(want, p.f, pr)
        s.vcycle(u, f)
    assert np.abs(host(u) - want).max() <= TOL * np.abs(want).max()


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 130])
def test_residual_and_start_norm(n):
    """r is 0 on the boundary whatever it held; the norm of the zero-interior
    start does not read u's interior."""
    note("legs residual", n)
    p = P.example2d(1, n)
    u0 = start(p, n)
    r_o, ss = ma2.residual(u0, p.f)
    out = dev(np.full_like(u0, 7.0))
    s = solver(n, "rb", 0, max_cycles=1)
    l2 = s.residual(dev(u0), dev(p.f), out)
    scale = max(np.abs(r_o).max(), np.abs(p.f).max())
    assert np.abs(host(out) - r_o).max() <= TOL * scale
    assert l2 == pytest.approx(np.sqrt(ss) / n, rel=1e-12)
    zero = P.initial_guess2(p)
    _, ss0 = ma2.residual(zero, p.f)
    rep = s.solve(dev(P.initial_guess2(p, float("nan"))), dev(p.f), tol=1.0)
    assert rep["res0"] == pytest.approx(np.sqrt(ss0) / n, rel=1e-12)


def test_nonfinite_start_leaves_the_zero_interior():
    from paper_1411_7018_amd import _lib as L
    n = 70
    p = P.example2d(1, n)
    f = p.f.copy()
    f[20, 30] = np.inf
    u = dev(P.initial_guess2(p, 3.0))
    with pytest.raises(L.MAError) as ei:
        solver(n, "rb", 0).solve(u, dev(f))
    assert ei.value.status == L.MA_ERR_NONFINITE
    assert np.array_equal(host(u), P.initial_guess2(p))
