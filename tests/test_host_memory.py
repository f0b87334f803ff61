"""Workspace sizes and what the callers make of them, on the CPU (the queries are
host code; allocations and contexts are stand-ins)."""
import ctypes
import random
import types

import pytest

torch = pytest.importorskip("torch")

from paper_1510_03330_amd import native as N
from paper_1510_03330_amd import ops
from workloads import ModelParams


def box(lx=2, ly=2, nv=16, **kw):
    return ModelParams(Lx=lx, Ly=ly, Nv=nv, U=1.3, beta=2.5, mu_mode=0, alpha=0.6, **kw)


def full(p, prec):
    return ops._workspace("parquet_query_workspace", N.make_params(p, prec))


def least(p, prec):
    return ops._workspace("parquet_query_workspace_min", N.make_params(p, prec))


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
def test_least_workspace(prec):
    """Below the preferred one for a small box, the same where the channels go one by one."""
    assert least(box(), prec) < 0.7 * full(box(), prec)
    assert least(box(8, 8, 16), prec) == full(box(8, 8, 16), prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("budget,width", [(4.5, 4), (2.2, 2), (1e6, 4)])
def test_runner_admits_what_least_workspaces_allow(monkeypatch, prec, budget, width):
    """budget: in least workspaces of the largest instance; at most four run at a time."""
    ps = [box(nv=16 if i % 2 else 14) for i in range(8)]
    budget = budget * least(ps[1], prec)
    live, most, compacts = [], [], set()

    class Context:
        def __init__(self, p, precision, device, stream=None, compact=False):
            self.bytes = least(p, precision) if compact else full(p, precision)
            compacts.add(compact)
            live.append(self.bytes)
            assert sum(live) <= budget

        def get(self, name):
            return torch.zeros(1, dtype=torch.complex128)

        def close(self):
            live.remove(self.bytes)

    def iterate(solvers, n, tol=0.0):
        most.append(len(solvers))
        return [n] * len(solvers), [True] * len(solvers)

    monkeypatch.setattr(ops, "Solver", Context)
    monkeypatch.setattr(ops, "iterate_batch", iterate)
    monkeypatch.setattr(ops, "new_stream", lambda d: types.SimpleNamespace())
    monkeypatch.setattr(ops, "release_stream", lambda s: None)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda d=None: None)
    r = ops.BatchRunner(ps, prec, mem_budget=budget, widths=(1, 2, 4))
    r.autotune()
    assert sorted(r.tuning) == [w for w in (1, 2, 4) if w <= width]
    r.width, most[:] = 4, []
    out, _ = r.run()
    assert max(most) >= width and all(o["converged"] for o in out)
    assert (True in compacts) == (4 * full(ps[1], prec) > budget)


class Device:
    """torch.empty over `room` bytes."""

    def __init__(self, room):
        self.room, self.sizes = room, []

    def empty(self, size, dtype, device):
        if size > self.room:
            raise torch.OutOfMemoryError("no room")
        self.sizes.append(size)
        return types.SimpleNamespace(numel=lambda: size, record_stream=lambda s: None)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("p", [box(), box(3, 2, 4), box(8, 8, 16)])
def test_context_on_a_device_short_of_memory(monkeypatch, prec, p):
    """Accepted down to the least workspace, to the byte; the full one where it fits."""
    hi, lo = full(p, prec), least(p, prec)
    monkeypatch.setattr(ops.Solver, "reinit", lambda self, p=None: None)
    for room, size in ((hi, hi), (hi - 1, lo), (lo, lo), (lo - 1, None)):
        dev = Device(room)
        monkeypatch.setattr(torch, "empty", dev.empty)
        if size is None or size > room:
            with pytest.raises(torch.OutOfMemoryError):
                ops.Solver(p, prec)
        else:
            ops.Solver(p, prec)
            assert dev.sizes == [size]
    dev = Device(2 * hi)
    monkeypatch.setattr(torch, "empty", dev.empty)
    ops.Solver(p, prec, ws_bytes=2 * hi)
    ops.Solver(p, prec, compact=True)
    assert dev.sizes == [2 * hi, lo]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("p,count", [(box(), 3), (box(3, 2, 4), 2), (box(), 1)])
def test_batch_on_a_device_short_of_memory(monkeypatch, prec, p, count):
    """As a context; a bound below the full size takes the least one at once, and
    holds nothing besides."""
    pp = (N.PqParams * count)(*[N.make_params(p, prec)] * count)
    hi, lo = ctypes.c_size_t(), ctypes.c_size_t()
    N.check(N.load().parquet_batch_query_workspace(pp, count, ctypes.byref(hi)))
    N.check(N.load().parquet_batch_query_workspace_min(pp, count, ctypes.byref(lo)))
    hi, lo = hi.value, lo.value
    assert (lo < hi) == (count > 1)
    made = []
    monkeypatch.setattr(ops.Batch, "_bind", lambda self, n, tune: made.append(torch.empty(n, torch.uint8, None)))
    for room, bound, size in ((hi, 0, hi), (hi - 1, 0, lo), (lo, 0, lo), (lo - 1, 0, None), (2 * hi, hi, hi),
                              (2 * hi, hi - 1, lo), (2 * hi, lo - 1, lo), (lo, 1, lo)):
        dev = Device(room)
        monkeypatch.setattr(torch, "empty", dev.empty)
        if size is None or size > room:
            with pytest.raises(torch.OutOfMemoryError):
                ops.Batch([p] * count, prec, max_bytes=bound)
        else:
            ops.Batch([p] * count, prec, max_bytes=bound)
            assert dev.sizes == [size]


def test_sums_scratch_holds_one_array_of_nodes():
    """A context's workspace grows with the quadrature nodes by the one array over
    them that is used; their number is even, as the launches by pairs need."""
    def up(x):
        return (x + 255) // 256 * 256

    rng = random.Random(7)
    for _ in range(200):
        lx, ly = rng.choice([(1, 1), (2, 1), (3, 3), (1, 5), (4, 4), (7, 1)])
        p = box(lx, ly, 2 * rng.randint(1, 6), f_ext=rng.randint(1, 5), D=rng.uniform(0.1, 3.0), tp=rng.uniform(-1.0, 1.0))
        nodes, bytes_ = [], []
        for beta in (rng.uniform(0.1, 5.0), rng.uniform(5.0, 80.0)):
            q = p.replace(beta=beta)
            nodes.append(N.dims(N.make_params(q, "fp64")).ntau)
            bytes_.append(least(q, "fp64"))
        assert nodes[0] % 2 == nodes[1] % 2 == 0
        assert bytes_[1] - bytes_[0] == up(16 * nodes[1] * lx * ly) - up(16 * nodes[0] * lx * ly)
