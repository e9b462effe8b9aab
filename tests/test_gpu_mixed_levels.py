"""The mixed inner problem's kernels at the edges of their tiles: row kernels
with the stored H, the fused residual and restriction, and the coarse levels in
LDS, against the coarse-level kernel in global memory (coarse_n = 32), which
forms H for every update.  The arithmetic is the same, so solves are bitwise
the same wherever the levels are split between the kernels.  Levels of more than
32 intervals run in the row kernels on both sides of a comparison; restriction
tiles of eight planes are in test_gpu_mixed_wide_tiles.py."""
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


def solve(p, n, tol=1e-9, **kw):
    from paper_1411_7018_amd import Solver, _lib as L
    f = torch.from_numpy(np.ascontiguousarray(p.f)).cuda()
    u = torch.from_numpy(np.ascontiguousarray(P.initial_guess(p, p.u_exact * 1.01))).cuda()
    try:
        rep = Solver(n, precision="mixed", **kw).solve(u, f, tol=tol)
    except L.MAError as e:   # 8 colours and half weighting need not converge
        rep = e.report
    torch.cuda.synchronize()
    return u.cpu().numpy(), rep["cycles"], rep["nonconvex"], rep["fp64_fallbacks"]


# 32 and 24 / 12: every level in the coarse kernel, global or LDS; 40, 56: a
# ragged last tile of the restriction, odd coarsest levels; 144: its levels 36, 18
# and 9 split, below two levels that are the same on both sides
@pytest.mark.parametrize("order", ["4c", "8c"])
@pytest.mark.parametrize("restriction", ["half", "full"])
@pytest.mark.parametrize("n", [4, 12, 16, 24, 32, 40, 56, 144])
def test_mixed_splits_bitwise(n, restriction, order):
    print("[case] mixed", n, restriction, order, file=sys.stderr, flush=True)
    p = P.exp_cos(n, seed=n)
    kw = dict(order=order, restriction=restriction)
    want = solve(p, n, coarse_n=32, **kw)
    if restriction == "full" and order == "4c":
        assert np.isfinite(want[0]).all()
    for cn in (0, 2, 8, 16):
        got = solve(p, n, coarse_n=cn, **kw)
        # (8 colours and half weighting may end in NaN on every split)
        assert np.array_equal(got[0], want[0], equal_nan=True), cn
        assert got[1:] == want[1:], cn


def test_mixed_zero_start_after_a_failed_solve():
    """A solver whose last solve failed starts the next one from a zero
    correction."""
    from paper_1411_7018_amd import Solver, _lib as L
    n = 40
    p = P.exp_cos(n, seed=1)
    f = torch.from_numpy(np.ascontiguousarray(p.f)).cuda()
    u0 = torch.from_numpy(np.ascontiguousarray(P.initial_guess(p, p.u_exact * 1.01))).cuda()
    want = solve(p, n)
    s = Solver(n, precision="mixed")
    bad = u0.clone()
    bad[3, 3, 3] = float("nan")
    with pytest.raises(L.MAError):
        s.solve(bad, f, tol=1e-9, init="none")
    u = u0.clone()
    s.solve(u, f, tol=1e-9)
    torch.cuda.synchronize()
    assert np.array_equal(u.cpu().numpy(), want[0])
