"""Outputs laid over f: the restriction's coarse arrays and the residual in
place give the bits of separate arrays."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [4, 34, 64])
def test_outputs_over_f_same_bits(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1411_7018_amd import Solver
    from paper_1411_7018_amd.solver import L
    print("[case] outputs over f", n, file=sys.stderr, flush=True)
    rng = np.random.default_rng(n)
    s = Solver(n)
    u, f0 = (torch.from_numpy(rng.standard_normal((n + 1,) * 3)).cuda() for _ in range(2))
    w, b = s.restrict(u, f0)
    for over in ("w", "b"):
        f = f0.clone()
        other = torch.empty_like(w)
        mine = f.view(-1)[5:5 + w.numel()]   # inside f, off its start
        pw, pb = (mine, other) if over == "w" else (other, mine)
        L.ma_restrict(s.handle, u.data_ptr(), f.data_ptr(), pw.data_ptr(), pb.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(pw.view(w.shape), w) and torch.equal(pb.view(b.shape), b)
    r = torch.empty_like(u)
    l2 = L.ma_residual(s.handle, u.data_ptr(), f0.data_ptr(), r.data_ptr())
    f = f0.clone()
    l2_in = L.ma_residual(s.handle, u.data_ptr(), f.data_ptr(), f.data_ptr())
    torch.cuda.synchronize()
    assert l2 == l2_in and torch.equal(f[1:-1, 1:-1, 1:-1], r[1:-1, 1:-1, 1:-1])
