"""The results that an iteration leaves in pinned host memory: statistics of one
call of several iterations against calls of one, with and without a convergence
test, more contexts at once than there are pinned slots (the others copy), and
contexts made and destroyed by two threads meanwhile."""
import math
import threading

import pytest

torch = pytest.importorskip("torch")

from workloads import ModelParams

pytestmark = pytest.mark.gpu

P = ModelParams(Lx=2, Ly=1, Nv=4, U=1.1, beta=2.0, tp=-0.1, mu_mode=1, alpha=0.6)
KEYS = ("iteration", "dsigma", "mu", "flagged_blocks", "resolved_blocks", "unresolved_blocks", "max_err_est")


def stats(st):
    return [getattr(st, k) for k in KEYS]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("tol", [0.0, 1e-14])
def test_statistics(prec, tol):
    print("CASE host results", prec, tol, flush=True)
    from paper_1510_03330_amd.ops import Solver
    a, b = Solver(P, prec), Solver(P, prec)
    _, _, sa = a.iterate(5, tol)
    for _ in range(5):
        _, _, sb = b.iterate(1, tol)
    assert stats(sa) == stats(sb)
    assert sa.mu == a.get("mu").item() and sa.iteration == 5
    assert sa.ms_total > 0.0 and all(math.isfinite(ms) for ms in sa.ms_stage)
    assert sum(sa.n_bse_launch) == sum(sb.n_bse_launch) > 0


def test_more_contexts_than_slots():
    print("CASE host results, many contexts", flush=True)
    from paper_1510_03330_amd.ops import Solver
    ref = Solver(P, "fp64")
    ref.iterate(3)
    out, stop = [], threading.Event()

    def churn():
        while not stop.is_set():
            s = Solver(P, "fp64")
            s.iterate(3)
            out.append(stats(s.last_stats) == stats(ref.last_stats))
            s.close()

    th = [threading.Thread(target=churn) for _ in range(2)]
    for t in th:
        t.start()
    many = [Solver(P, "fp64") for _ in range(70)]
    for _ in range(3):
        for s in many:
            s.iterate(1)
    stop.set()
    for t in th:
        t.join()
    assert out and all(out)
    for s in many:
        assert stats(s.last_stats) == stats(ref.last_stats)
