"""An odd number of sweeps, whose last one runs in one launch with a copy back
or per colour by the size: the bits of the colour launches on both sides of each size."""
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
