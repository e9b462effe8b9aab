"""Colour phases with a row's nodes packed into wavefronts (rows after each
other): the bits and the count of uncertified updates of the block sweep, which
enumerates nodes another way, at rows shorter than, equal to and longer than a
wavefront, odd and even, in both orderings; through the component call and
through whole solves.  (The oracle pins the same phases to round-off at n <= 67
in test_gpu_fp64.py.)"""
import sys

import numpy as np
import pytest

from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [2, 3, 5, 66, 97, 127, 128, 129, 130, 149])
@pytest.mark.parametrize("order", ["4c", "8c"])
def test_sweep_packed_rows(n, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1411_7018_amd import Solver
    print("[case] packed rows", n, order, file=sys.stderr, flush=True)
    p = P.exp_cos(n, seed=n)
    rng = np.random.default_rng(n)
    u = P.initial_guess(p, p.u_exact * (1.0 + 0.01 * rng.standard_normal(p.u_exact.shape)))
    f = torch.from_numpy(p.f.copy()).cuda()
    out = []
    for smoother in ("color", "fused"):
        t = torch.from_numpy(u.copy()).cuda()
        nc = Solver(n, order=order, smoother=smoother).sweep(t, f, 2)
        out.append((nc, t.cpu().numpy().view(np.int64)))
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("n", [6, 34, 66, 96, 130, 160])
@pytest.mark.parametrize("order,precision", [("4c", "fp64"), ("8c", "fp64"), ("4c", "mixed")])
def test_cycles_packed_rows(n, order, precision):
    """Levels of several row lengths in the engine, colour launches only
    (block_n = -1, no coarse-level kernel) against the automatic choice.  (In
    the mixed form the levels from n = 34 on are the same launches on both sides
    but for their strips: what is compared is their work order and the smaller
    levels; test_gpu_mixed_wide_tiles.py has the rest.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1411_7018_amd import Solver, _lib as L
    print("[case] packed rows cycles", n, order, precision, file=sys.stderr, flush=True)
    p = P.exp_cos(n, seed=n)
    f = torch.from_numpy(p.f.copy()).cuda()
    out = []
    for kw in ({"block_n": -1, "coarse_n": 0, "strip_rows": 5}, {}):
        t = torch.from_numpy(P.initial_guess(p)).cuda()
        try:
            rep = Solver(n, order=order, precision=precision, max_cycles=3, **kw).solve(t, f)
        except L.MAError as e:   # stops at the cycle limit
            rep = e.report
        out.append((rep["cycles"], rep["res"], t.cpu().numpy().view(np.int64)))
    assert out[0][:2] == out[1][:2]
    assert np.array_equal(out[0][2], out[1][2])
