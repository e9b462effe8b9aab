"""The residual on grids whose rows end at, just before and just after a wavefront
of 64 columns: values, zeros on the whole boundary and the norm against the oracle."""
import sys

import numpy as np
import pytest

import oracle
from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# Both sides take the same differences in the same order; they part in the
# determinant's contracted products, a few eps of its largest term.
TOL = 1e-12


@pytest.mark.parametrize("n", [2, 62, 63, 64, 65, 66, 127, 128, 129, 130])
def test_residual_at_row_ends(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1411_7018_amd import Solver
    print("[case] residual columns", n, file=sys.stderr, flush=True)
    p = P.exp_cos(n, seed=n)
    rng = np.random.default_rng(n)
    u0 = P.initial_guess(p, p.u_exact * (1.0 + 0.01 * rng.standard_normal(p.u_exact.shape)))
    want, ss = oracle.residual(u0, p.f)
    scale = max(np.abs(want).max(), np.abs(p.f).max())
    u, f = torch.from_numpy(u0).cuda(), torch.from_numpy(p.f.copy()).cuda()
    s = Solver(n)
    r = torch.full_like(u, float("nan"))
    norms = [s.residual(u, f, out=r), s.residual(u, f)]
    got = r.cpu().numpy()
    inner = np.zeros_like(got, bool)
    inner[1:-1, 1:-1, 1:-1] = True
    assert not got[~inner].any()
    assert np.abs(got - want)[inner].max() <= TOL * scale
    for l2 in norms:
        assert l2 == pytest.approx(oracle.l2(ss, n), rel=1e-12)
