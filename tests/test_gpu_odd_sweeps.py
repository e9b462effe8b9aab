"""An odd number of sweeps, whose last one runs in one launch with a copy back
or per colour by the size (in two dimensions too), and the Gauss-Seidel solver's
first sweeps, looked at one by one: the bits of the colour launches on both sides
of each size."""
import sys

import numpy as np
import pytest

from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def start(n):
    from paper_1411_7018_amd import Solver  # noqa: F401  (the library must load)
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = P.exp_cos(n, seed=n)
    rng = np.random.default_rng(n)
    u = P.initial_guess(p, p.u_exact * (1.0 + 0.01 * rng.standard_normal(p.u_exact.shape)))
    return torch.from_numpy(u).cuda(), torch.from_numpy(p.f.copy()).cuda()


@pytest.mark.parametrize("count", [1, 3])
@pytest.mark.parametrize("order,n", [("4c", 49), ("4c", 50), ("4c", 64), ("4c", 192), ("4c", 224),
                                     ("4c", 240), ("8c", 80), ("8c", 81), ("8c", 88)])
def test_odd_sweeps_bitwise(order, n, count):
    print("[case] odd sweeps", order, n, count, file=sys.stderr, flush=True)
    from paper_1411_7018_amd import Solver
    u, f = start(n)
    out = []
    for smoother in ("color", "auto", "fused"):
        t = u.clone()
        nc = Solver(n, order=order, smoother=smoother).sweep(t, f, count)
        out.append((nc, t.cpu().numpy().view(np.int64)))
    for o in out[1:]:
        assert o[0] == out[0][0] and np.array_equal(o[1], out[0][1])


@pytest.mark.parametrize("sweeps", [1, 2, 5, 9, 10, 18])
@pytest.mark.parametrize("order,n", [("4c", 48), ("4c", 90), ("8c", 76)])
def test_gs_first_sweeps_bitwise(order, n, sweeps):
    print("[case] gs first sweeps", order, n, sweeps, file=sys.stderr, flush=True)
    from paper_1411_7018_amd import Solver, _lib as L
    u, f = start(n)
    out = []
    for smoother in ("color", "auto"):
        t = u.clone()
        with pytest.raises(L.MAError) as ei:
            Solver(n, order=order, smoother=smoother).gs_solve(t, f, tol=1e-14, max_sweeps=sweeps)
        out.append((ei.value.report["cycles"], ei.value.report["nonconvex"],
                    t.cpu().numpy().view(np.int64), np.array(ei.value.report["history"])))
    assert out[0][:2] == out[1][:2] and np.array_equal(out[0][2], out[1][2])
    assert np.abs(out[0][3] - out[1][3]).max() <= 1e-12 * out[0][3].max()


@pytest.mark.parametrize("order,n", [("4c", 12), ("4c", 40), ("4c", 41), ("4c", 57), ("4c", 76),
                                     ("4c", 77), ("8c", 12), ("8c", 41), ("8c", 64), ("8c", 73)])
def test_gs_stops_bitwise(order, n):
    """A tolerance met at every place of the batches: the iterate, the counts and
    the history of the sweeps looked at one by one."""
    print("[case] gs stops", order, n, file=sys.stderr, flush=True)
    from paper_1411_7018_amd import Solver, _lib as L
    p = P.exp_cos(n, seed=n)
    t = np.sin(3.0 * np.arange(n + 1) / n)
    bump = 1.0 + 0.02 * t[:, None, None] * t[None, :, None] * t[None, None, :]
    u = torch.from_numpy(P.initial_guess(p, p.u_exact * bump)).cuda()
    f = torch.from_numpy(p.f.copy()).cuda()
    one, auto = Solver(n, order=order, smoother="color"), Solver(n, order=order)
    with pytest.raises(L.MAError) as ei:
        one.gs_solve(u.clone(), f, tol=1e-14, max_sweeps=64)
    h = np.array(ei.value.report["history"][:64])
    # sweeps whose residual is below all before it by more than the sums' round-off
    ks = [k for k in (*range(1, 21), 31, 32, 33, 34, 35, 63, 64)
          if h[k - 1] < (1.0 - 1e-6) * min([ei.value.report["res0"], *h[:k - 1]])]
    assert len(ks) >= 10
    for k in ks:
        out = []
        for s in (one, auto):
            v = u.clone()
            rep = s.gs_solve(v, f, tol=(1.0 + 1e-7) * h[k - 1] / ei.value.report["res0"])
            out.append((rep["cycles"], rep["nonconvex"], v.cpu().numpy().view(np.int64)))
        assert out[0][0] == out[1][0] == k and out[0][1] == out[1][1]
        assert np.array_equal(out[0][2], out[1][2])


@pytest.mark.parametrize("order,n", [("4c", 702), ("4c", 704), ("4c", 1025), ("rb", 990),
                                     ("rb", 992), ("rb", 1025)])
def test_lone_2d_sweep_bitwise(order, n):
    """A lone sweep as a launch per phase, against the first of three sweeps (no
    phase launches): the second and third, run apart, end in the same bits."""
    from paper_1411_7018_amd.solver2d import Solver2D
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] lone 2D sweep", order, n, file=sys.stderr, flush=True)
    x = torch.arange(n + 1, dtype=torch.float64, device="cuda") / n
    r = x[None, :] ** 2 + x[:, None] ** 2
    g = torch.Generator(device="cuda").manual_seed(n)
    u = torch.exp(r / 2)
    u[1:-1, 1:-1] *= 1.0 + 1e-6 * torch.randn((n - 1, n - 1), generator=g, dtype=torch.float64,
                                              device="cuda")
    f = ((1.0 + r) * torch.exp(r)).contiguous()
    a, b = u.clone(), u.clone()
    s = Solver2D(n, order=order)
    na = s.sweep(a, f, 3)
    nb = s.sweep(b, f, 1) + s.sweep(b, f, 2)
    torch.cuda.synchronize()
    assert na == nb and not torch.equal(a, u)
    assert torch.equal(a.view(torch.int64), b.view(torch.int64))
