"""The 52 x 44 tiles of 4-colour legs (n >= 768) against the 2D oracle: grids on
both sides of the rule, ending one node short of, at and past a tile.  Tolerance
1e-12 of max |u| as in the other comparisons with it: the same formulas, summed
in another order."""
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


def close(t, want):
    torch.cuda.synchronize()
    assert np.abs(t.cpu().numpy() - want).max() <= TOL * np.abs(want).max()


def start(p, seed, amp):
    rng = np.random.default_rng(seed)
    return P.initial_guess2(p, p.u_exact * (1 + amp * rng.standard_normal(p.u_exact.shape)))


def solver(n, rm, **kw):
    from paper_1411_7018_amd.solver2d import Solver2D
    return Solver2D(n, order="4c", restriction="half" if rm == 0 else "full", **kw)


# 779 = 15 * 52 - 1: the last column is the only one of its tile; 791 = 18 * 44
# - 1: so is the last row; 780, 792 one node on
@pytest.mark.parametrize("n,count", [(767, 2), (768, 1), (779, 2), (780, 3), (791, 5), (792, 4)])
def test_sweeps(n, count):
    print("[case] big tiles", n, count, file=sys.stderr, flush=True)
    p = P.example2d(1, n)
    f = p.f.copy()
    f[1:-1:7, 2:-1:5] = -0.5
    want = start(p, n, 0.01)
    u = dev(want)
    bad = sum(ma2.sweep(want, f, "4c") for _ in range(count))
    assert solver(n, 0).sweep(u, dev(f), count) == bad > 0
    close(u, want)


@pytest.mark.parametrize("n", [768, 780, 832])
@pytest.mark.parametrize("rm", [0, 1])
def test_vcycle_fmg_and_norm(n, rm):
    print("[case] big tiles vcycle", n, rm, file=sys.stderr, flush=True)
    p = P.example2d(1, n)
    pr = ma2.params(order="4c", rmode=rm)
    s = solver(n, rm)
    want = start(p, n, 1e-4)
    u = dev(want)
    ma2.vcycle(want, p.f, pr)
    s.vcycle(u, dev(p.f))
    close(u, want)
    ma2.fmg(want, p.f, pr)
    s.fmg(u, dev(p.f))
    close(u, want)
    # the residual that the last leg of a solve's cycle leaves
    v = dev(P.initial_guess2(p))
    rep = solver(n, rm, max_cycles=1).solve(v, dev(p.f), tol=1.0)
    assert rep["res"] == pytest.approx(s.residual(v, dev(p.f)), rel=1e-10)
