"""8-colour block sweeps, the one-launch-per-sweep Gauss-Seidel iteration and
the single-grid component kernels at the edges of their tiles.  Sweeps are
bitwise those of the colour launches (the same point update on the same
values); residuals, restrictions and corrections are compared with the oracle
at 1e-12 of the array's largest value (sums of at most 27 terms in another
order and FMA contraction: ~ 1e-14)."""
import sys

import numpy as np
import pytest

import oracle
from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
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


def note(*args):
    print("[case]", *args, file=sys.stderr, flush=True)


def solver(n, **kw):
    from paper_1411_7018_amd import Solver
    return Solver(n, **kw)


def start(p, seed, eps=1e-3):
    rng = np.random.default_rng(seed)
    return P.initial_guess(p, p.u_exact * (1.0 + eps * rng.standard_normal(p.u_exact.shape)))


def close(got, want):
    assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()


@pytest.mark.parametrize("count", [1, 2])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 8, 9, 17, 32, 33, 34, 64, 65, 66, 127, 128, 135, 136,
                               137, 160, 161, 201])
def test_8_colour_block_sweep_bitwise(n, count):
    note("8c block sweep", n, count)
    p = P.exp_cos(n, seed=n)
    u0, f = start(p, 3, 0.05), dev(p.f)
    ua, ub, uf = dev(u0), dev(u0), dev(u0)
    want = solver(n, order="8c", smoother="color").sweep(ua, f, count)
    assert solver(n, order="8c").sweep(ub, f, count) == want
    assert solver(n, order="8c", smoother="fused").sweep(uf, f, count) == want
    assert np.array_equal(host(ub), host(ua)) and np.array_equal(host(uf), host(ua))


@pytest.mark.parametrize("order", ["4c", "8c"])
@pytest.mark.parametrize("n,coarse", [(40, 4), (72, 8), (144, 17), (288, 17)])
def test_8_colour_levels_bitwise(n, coarse, order):
    """Whole V-cycles, Poisson guess included, block levels against colour
    launches on every multi-block level."""
    note("levels", n, coarse, order)
    p = P.example4(n)
    out = []
    for sm in ("color", "auto", "fused"):
        u = dev(start(p, 1))
        rep = solver(n, order=order, smoother=sm, coarse_n=coarse).solve(u, dev(p.f), tol=1e-8)
        out.append((host(u), rep["cycles"], rep["nonconvex"]))
    for o in out[1:]:
        assert np.array_equal(o[0], out[0][0]) and o[1:] == out[0][1:]


@pytest.mark.parametrize("order", ["4c", "8c"])
@pytest.mark.parametrize("n", [2, 4, 8, 9, 16, 33, 40, 41])
def test_gs_steps_same_iterates(n, order):
    """Launches that test the iterate before last stop where a test after
    every sweep stops, with its iterate, counts and residuals."""
    note("gs", n, order)
    p = P.exp_cos(n, seed=5)
    u0, f = start(p, 2, 0.05), dev(p.f)
    ua, ub = dev(u0), dev(u0)
    a = solver(n, order=order, smoother="color").gs_solve(ua, f, tol=1e-2)
    b = solver(n, order=order).gs_solve(ub, f, tol=1e-2)
    assert b["cycles"] == a["cycles"] and b["nonconvex"] == a["nonconvex"]
    assert b["converged"] == a["converged"] == 1
    assert np.array_equal(host(ub), host(ua))
    k = min(a["cycles"], 64)
    ha, hb = np.array(a["history"][:k]), np.array(b["history"][:k])
    assert np.abs(ha - hb).max() <= 1e-12 * ha.max()


@pytest.mark.parametrize("order", ["4c", "8c"])
@pytest.mark.parametrize("sweeps", [1, 2, 3, 31, 32, 33, 64, 65, 66, 97])
def test_gs_steps_at_the_limit(sweeps, order):
    """The sweep limit at every place of a batch and of the ring of sums; and
    a first residual that already meets the tolerance still takes a sweep."""
    from paper_1411_7018_amd import _lib as L
    note("gs limit", sweeps, order)
    n = 20
    p = P.exp_cos(n, seed=5)
    u0, f = start(p, 2, 0.05), dev(p.f)
    ua, ub = dev(u0), dev(u0)
    for sm, u in (("color", ua), ("auto", ub)):
        with pytest.raises(L.MAError) as ei:
            solver(n, order=order, smoother=sm).gs_solve(u, f, tol=1e-14, max_sweeps=sweeps)
        assert ei.value.status == L.MA_ERR_NOT_CONVERGED
    assert np.array_equal(host(ub), host(ua))
    uc = dev(u0)
    rep = solver(n, order=order).gs_solve(uc, f, tol=10.0, max_sweeps=sweeps)
    assert rep["cycles"] == 1


def test_gs_steps_not_finite():
    from paper_1411_7018_amd import _lib as L
    p = P.example4(12)
    f = p.f.copy()
    f[5, 5, 5] = np.inf
    with pytest.raises(L.MAError) as ei:
        solver(12).gs_solve(dev(start(p, 1)), dev(f), tol=1e-6, max_sweeps=40)
    assert ei.value.status == L.MA_ERR_NONFINITE


@pytest.mark.parametrize("n", [2, 3, 6, 7, 8, 9, 16, 62, 64, 66, 126, 130])
def test_components_vs_oracle(n):
    note("components", n)
    p = P.exp_cos(n, seed=n)
    u0 = start(p, 4)
    u, f = dev(u0), dev(p.f)
    s = solver(n)
    r = torch.full_like(u, 7.0)
    l2 = s.residual(u, f, out=r)
    want, ss = oracle.residual(u0, p.f)
    assert np.abs(host(r) - want).max() <= 1e-12 * max(np.abs(p.f).max(), np.abs(want).max())
    assert abs(l2 - np.sqrt(ss / n**3)) <= 1e-12 * np.sqrt(ss / n**3)
    assert s.residual(u, f) == l2
    if n % 2 or n < 4:
        return
    for mode, rm in (("half", oracle.RESTRICT_HALF), ("full", oracle.RESTRICT_FULL)):
        wc, bc = solver(n, restriction=mode).restrict(u, f)
        w, b = oracle.restrict(u0, want, rmode=rm)
        assert np.array_equal(host(wc), w)
        assert np.abs(host(bc) - b).max() <= 1e-12 * max(np.abs(b).max(), np.abs(p.f).max())
    uc = w * (1.0 + 1e-3 * np.random.default_rng(1).standard_normal(w.shape))
    s.prolong_correct(u, dev(uc), dev(w))
    v = u0.copy()
    oracle.prolong_correct(v, uc, w)
    close(host(u), v)
