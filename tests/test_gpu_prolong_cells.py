"""The prolongation by coarse cells (eight fine nodes a lane) against the oracle,
whose terms and order it has: bitwise, at sizes around the 64 cells of a
wavefront, through the component call and, batched, through solves; and the
Dirichlet layer keeps its bits."""
import sys

import numpy as np
import pytest

import oracle
from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [4, 6, 32, 62, 64, 66, 126, 128, 130, 254, 258])
def test_prolong_correct_bitwise(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1411_7018_amd import Solver
    print("[case] prolong cells", n, file=sys.stderr, flush=True)
    rng = np.random.default_rng(n)
    shape, cshape = (n + 1,) * 3, (n // 2 + 1,) * 3
    u = rng.standard_normal(shape)
    u[0], u[:, -1], u[:, :, 0] = -0.0, np.nan, -0.0   # boundary: never read or written
    uc, wc = rng.standard_normal(cshape), rng.standard_normal(cshape)
    want = u.copy()
    oracle.prolong_correct(want, uc, wc)
    t, c, w = (torch.from_numpy(a.copy()).cuda() for a in (u, uc, wc))
    Solver(n).prolong_correct(t, c, w)
    torch.cuda.synchronize()
    got = t.cpu().numpy()
    assert np.array_equal(got.view(np.int64), want.view(np.int64))
