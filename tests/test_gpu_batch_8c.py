"""8-colour batches on both sides of the tile count from which a depth's grids
take colour launches instead of block sweeps: the bits of lone solves."""
import sys

import numpy as np
import pytest

from paper_1411_7018_amd import problems as P

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# 8^3 tiles of the finest level: 1024, 1536 (limit 1200), 20 x 64, 40 x 27
@pytest.mark.parametrize("n,count", [(64, 2), (64, 3), (32, 20), (24, 40)])
def test_8_colour_batch_bitwise(n, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1411_7018_amd import Solver, _lib as L
    from paper_1411_7018_amd.batch import solve_batch
    print("[case] 8c batch", n, count, file=sys.stderr, flush=True)
    probs = [P.exp_cos(n, seed=i) for i in range(count)]
    kw = dict(order="8c", max_cycles=3)
    us, fs = [dev(P.initial_guess(p)) for p in probs], [dev(p.f) for p in probs]
    _, reps = solve_batch([Solver(n, **kw) for _ in probs], us, fs, tol=1e-14)
    for i in (0, count - 1):
        u = dev(P.initial_guess(probs[i]))
        with pytest.raises(L.MAError) as ei:   # stops at the cycle limit
            Solver(n, **kw).solve(u, fs[i], tol=1e-14)
        assert reps[i]["cycles"] == 3 and reps[i]["res"] == ei.value.report["res"]
        assert reps[i]["nonconvex"] == ei.value.report["nonconvex"]
        assert np.array_equal(us[i].cpu().numpy(), u.cpu().numpy())
