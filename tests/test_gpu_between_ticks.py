"""Calls on a resident solve's solver between ticks: the batch's results are
bitwise those of an undisturbed batch, whatever other grids the component
entry points, whole solves on the same solver and changes of the launch shape
leave in its scratch arrays."""
import sys

import numpy as np
import pytest

from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def sweep(s, u, f):
    s.sweep(u, f)


def gs(s, u, f):
    from paper_1411_7018_amd import _lib as L
    with pytest.raises(L.MAError):   # stops at the limit
        s.gs_solve(u, f, tol=1e-14, max_sweeps=2)


def restrict_over_f(s, u, f):
    from paper_1411_7018_amd.solver import L
    m = (s.n // 2 + 1) ** 3
    w, b = f.view(-1)[:m], f.view(-1)[m:2 * m]
    L.ma_restrict(s.handle, u.data_ptr(), f.data_ptr(), w.data_ptr(), b.data_ptr())


def poisson(s, u, f):
    s.poisson_init(u, f)


def fmg(s, u, f):
    s.fmg(u, f)


def solve(s, u, f):
    s.solve(u, f, tol=1e-6)


CALLS = {c.__name__: c for c in (sweep, gs, restrict_over_f, poisson, fmg, solve)}


def run(n, between=None, init="none", **kw):
    """A resident solve, between(batch, solver, tick) called after each tick;
    its result, cycles and residuals."""
    from paper_1411_7018_amd import Solver
    from paper_1411_7018_amd.batch import ResidentBatch
    p = P.exp_cos(n, seed=n)
    b, s = ResidentBatch(4), Solver(n, **kw)
    u = dev(P.initial_guess(p, p.u_exact * 1.01))
    slot = b.add(s, u, dev(p.f), tol=1e-7, init=init)
    for tick in range(100):
        done = b.tick()
        if slot in done:
            assert done[slot] == 1
            rep = b.report(slot)
            return u.cpu().numpy(), rep["cycles"], rep["history"]
        if between:
            between(b, s, tick)
    raise AssertionError("no convergence")


def other_grid(n):
    q = P.example4(n)
    rng = np.random.default_rng(n)
    u = q.u_exact * (1.0 + 0.01 * rng.standard_normal(q.u_exact.shape))
    return dev(P.initial_guess(q, u)), dev(2.0 * q.f)


def same(got, want):
    assert got[1] == want[1] and got[2] == want[2]
    assert np.array_equal(got[0], want[0])


@pytest.mark.parametrize("call", list(CALLS))
@pytest.mark.parametrize("n", [24, 40, 72])
def test_component_calls_between_mixed_ticks(n, call):
    print("[case] mixed between ticks", n, call, file=sys.stderr, flush=True)

    def between(b, s, tick):
        u, f = other_grid(n)
        CALLS[call](s, u, f)

    same(run(n, between, precision="mixed"), run(n, precision="mixed"))


@pytest.mark.parametrize("first,then", [(16, 32), (32, 16), (0, 32), (32, 8)])
@pytest.mark.parametrize("n", [24, 32])
def test_coarse_n_between_mixed_ticks(n, first, then):
    """The levels move between the row kernels and the coarse-level kernel
    while a solve is resident: the engine takes the new coarse_n over when
    another solve joins or leaves."""
    from paper_1411_7018_amd import Solver
    print("[case] coarse_n between ticks", n, first, then, file=sys.stderr, flush=True)
    q = P.example4(16)
    other = []

    def between(b, s, tick):
        if tick == 1:
            s.retune(coarse_n=then)
            t = Solver(16, precision="mixed", inner_cycles=1, coarse_n=then)
            slot = b.add(t, dev(P.initial_guess(q, q.u_exact * 1.01)), dev(q.f), tol=1e-12,
                         init="none")
            other.append((t, slot))
        if tick == 3:
            s.retune(coarse_n=first)
            b.remove(other[0][1])

    kw = dict(precision="mixed", inner_cycles=1, coarse_n=first)
    got, want = run(n, between, **kw), run(n, **kw)
    assert other and want[1] > 5
    same(got, want)


@pytest.mark.parametrize("call", ["vcycle", "poisson", "fmg", "solve"])
@pytest.mark.parametrize("n,init", [(40, "none"), (40, "poisson"), (96, "poisson")])
def test_whole_cycles_between_fp64_ticks(n, init, call):
    """The right-hand side of the Poisson guess (n = 40) and the copy of the
    right-hand side in colour order (n = 96: colour launches)."""
    print("[case] fp64 between ticks", n, init, call, file=sys.stderr, flush=True)

    def between(b, s, tick):
        u, f = other_grid(n)
        s.vcycle(u, f) if call == "vcycle" else CALLS[call](s, u, f)

    same(run(n, between, init=init), run(n, init=init))
