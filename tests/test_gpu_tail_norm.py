"""The norm that the coarse-level kernel takes when it is the whole cycle: the
same bits, and so the same history and stopping, as the norm launches that run
when a larger grid shares the batch, for every size that takes this path."""
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


@pytest.mark.parametrize("init", ["poisson", "none"])
@pytest.mark.parametrize("restriction", ["half", "full"])
@pytest.mark.parametrize("n", list(range(2, 17)))
def test_norm_in_the_coarse_kernel_same_bits(n, restriction, init):
    from paper_1411_7018_amd import Solver
    from paper_1411_7018_amd.batch import solve_batch
    print("[case] tail norm", n, restriction, init, file=sys.stderr, flush=True)
    kw = dict(restriction=restriction, nu0=16, max_cycles=200)
    probs = [P.exp_cos(n, seed=n), P.example4(n), P.example4(40)]
    fs = [dev(p.f) for p in probs]

    def run(k):
        us = [dev(P.initial_guess(p, 1.02 * p.u_exact)) for p in probs[:k]]
        _, reps = solve_batch([Solver(p.n, **kw) for p in probs[:k]], us, fs[:k], tol=1e-6,
                               init=init)
        torch.cuda.synchronize()
        return [u.cpu().numpy() for u in us], reps

    alone, ra = run(2)      # every cycle is one launch
    mixed, rm = run(3)      # 40 has levels above the coarse-level kernel
    for u, v, a, m in zip(alone, mixed, ra, rm):
        assert np.array_equal(u, v)
        assert a["cycles"] == m["cycles"] and a["history"] == m["history"]
        assert a["res0"] == m["res0"] and a["res"] == m["res"]
        assert a["converged"] == m["converged"]
