"""The coarse-level kernel in LDS at every level size it has a case for (n = 2
.. 16 as its top level, and so every chain of sizes below) and just above
(17 .. 20: the other forms), against the row kernels (coarse_n = 0), which
run every level as separate launches: the same bits and the same count of
uncertified updates, for V-cycles, the linear cycles of the Poisson start, both
restrictions and several sweep counts."""
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


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def cycles(n, coarse_n, bad, **kw):
    from paper_1411_7018_amd import Solver, _lib as L
    p = P.make("exp_cos", n, n)
    f = p.f.copy()
    if bad and n > 3:
        f[1:-1:3, 2:-1:4, 1:-1:5] = -0.3   # the general root on some nodes
    rng = np.random.default_rng(n)
    noise = 1 + 1e-3 * rng.standard_normal(p.u_exact.shape)
    s = Solver(n, coarse_n=coarse_n, init_max_cycles=3, max_cycles=2, **kw)
    u, v = dev(P.initial_guess(p, p.u_exact * noise)), dev(P.initial_guess(p))
    s.vcycle(u, dev(f))
    s.vcycle(u, dev(f))
    s.poisson_init(v, dev(p.f))
    w = dev(P.initial_guess(p, p.u_exact * noise))
    try:
        rep = s.solve(w, dev(f), tol=1e-30, init="none")
    except L.MAError as e:
        rep = e.report
    s.close()
    return host(u), host(v), rep["nonconvex"], rep["history"]


@pytest.mark.parametrize("n", range(2, 21))
@pytest.mark.parametrize("kw", [{}, {"restriction": "half"}, {"nu1": 0, "nu2": 1, "nu0": 3},
                                {"nu1": 3, "nu2": 0}], ids=str)
def test_every_level_size(n, kw):
    print("[case] tail size", n, kw, file=sys.stderr, flush=True)
    for bad in (False, True):
        u0, v0, c0, h0 = cycles(n, 0, bad, **kw)
        u, v, c, h = cycles(n, 32, bad, **kw)
        assert np.array_equal(u0, u, equal_nan=True) and np.array_equal(v0, v)
        assert c0 == c and np.array_equal(h0, h, equal_nan=True)
