"""The mixed inner problem in launches large enough for restriction tiles of
eight planes, on grids small enough for the independent form: batches of 20
solves at n = 32 (20 x 125 tiles; eight planes from 2048 on) and 40 at n = 24 (64
each, ragged last tiles) through the row kernels, against lone solves in the
global-memory coarse-level kernel (coarse_n = 32), which forms H for every
update; and convergence as fast as the FP64 form's on grids that no other form
takes whole."""
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


@pytest.mark.parametrize("coarse_n", [0, 8, 16])
@pytest.mark.parametrize("n,count", [(32, 20), (24, 40)])
def test_wide_tiles_bitwise(n, count, coarse_n):
    from paper_1411_7018_amd import Solver
    from paper_1411_7018_amd.batch import solve_batch
    print("[case] mixed wide tiles", n, coarse_n, file=sys.stderr, flush=True)
    probs = [P.exp_cos(n, seed=i) for i in range(count)]
    kw = dict(precision="mixed")
    starts = [P.initial_guess(p, p.u_exact * 1.01) for p in probs]
    us, fs = [dev(u) for u in starts], [dev(p.f) for p in probs]
    st, reps = solve_batch([Solver(n, coarse_n=coarse_n, **kw) for _ in probs], us, fs, tol=1e-8)
    assert st == 0
    for i in range(0, count, 3):
        u = dev(starts[i])
        rep = Solver(n, coarse_n=32, **kw).solve(u, fs[i], tol=1e-8)
        assert rep["converged"] == 1 and np.isfinite(rep["res"])
        for key in ("cycles", "outer", "nonconvex", "fp64_fallbacks", "res"):
            assert reps[i][key] == rep[key], (i, key)
        assert np.array_equal(us[i].cpu().numpy(), u.cpu().numpy()), i


@pytest.mark.parametrize("n", [48, 96, 192, 256])
def test_mixed_converges_like_fp64(n):
    """A wrong coarse right-hand side or H slows the inner cycles down and
    nothing else: no more outer corrections, of two cycles each, than FP64
    cycles."""
    from paper_1411_7018_amd import Solver
    print("[case] mixed rate", n, file=sys.stderr, flush=True)
    p = P.exp_cos(n, seed=n)
    f = dev(p.f)
    reps = []
    for precision in ("fp64", "mixed"):
        u = dev(P.initial_guess(p))
        reps.append(Solver(n, precision=precision).solve(u, f, tol=1e-8))
        assert reps[-1]["converged"] == 1 and bool(torch.isfinite(u).all())
    print("[rate]", n, reps[0]["cycles"], reps[1]["outer"], file=sys.stderr, flush=True)
    assert 2 * reps[1]["outer"] <= reps[0]["cycles"] + 2
