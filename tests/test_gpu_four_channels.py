"""The Bethe-Salpeter equations of a small box's four channels in shared launches
against the same context channel by channel (a workspace one byte short of the
queried size), with blocks re-solved in FP64, and a context started again on
parameters of another box.

The two differ in the launch shapes only: bounds as for a stage against another
order of its sums, a few eps kappa n^(1/2) over three iterations (1e-11
complex128, 2e-4 FP32 products, 2e-3 BF16x3)."""
import pytest

torch = pytest.importorskip("torch")

from workloads import ModelParams

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-11, "fp32": 2e-4, "bf16x3": 2e-3}


def rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("lx,ly,nv,tol", [(1, 1, 2, 0.0), (1, 1, 20, 0.0), (2, 1, 34, 0.0), (3, 2, 4, 0.0), (2, 2, 18, 0.0),
                                          (3, 2, 4, 1e-12), (2, 1, 34, 1e-12)])
def test_four_channels(prec, lx, ly, nv, tol):
    print("CASE four channels", prec, lx, ly, nv, tol, flush=True)
    from paper_1510_03330_amd.ops import Solver
    p = ModelParams(Lx=lx, Ly=ly, Nv=nv, U=1.3, beta=2.5, tp=-0.1, mu_mode=0, alpha=0.6)
    a = Solver(p, prec, bse_tol=tol)
    b = Solver(p, prec, bse_tol=tol)
    b.ws = b.ws[:-1]
    b.reinit()
    for s in (a, b):
        s.iterate(3)
    for f in ("sigma", "phi", "k1", "k2"):
        assert rel(a.get(f), b.get(f)) < TOL[prec], f
    for f in ("flagged_blocks", "resolved_blocks", "unresolved_blocks", "iteration"):
        assert getattr(a.last_stats, f) == getattr(b.last_stats, f), f
    if tol > 0.0 and prec != "fp64":
        assert a.last_stats.resolved_blocks > 0


def test_reinit_other_box():
    print("CASE reinit other box", flush=True)
    from paper_1510_03330_amd.ops import Solver
    p = ModelParams(Lx=2, Ly=2, Nv=8, U=1.3, beta=2.5, mu_mode=0, alpha=0.6)
    small = ModelParams(Lx=2, Ly=1, Nv=8, U=1.1, beta=2.0, mu_mode=0, alpha=0.6)
    large = ModelParams(Lx=3, Ly=3, Nv=16, U=1.3, beta=2.5, mu_mode=0, alpha=0.6)
    s = Solver(p, "fp64")
    s.iterate(2)
    kept = s.get("phi")
    with pytest.raises(ValueError):
        s.reinit(large)
    assert torch.equal(s.get("phi"), kept)           # the solver is as it was
    s.reinit(small)
    s.iterate(2)
    ref = Solver(small, "fp64")
    ref.iterate(2)
    assert torch.equal(s.get("phi"), ref.get("phi"))


@pytest.mark.parametrize("share,ok", [(0.8, True), (0.2, False)])
def test_device_short_of_memory(monkeypatch, share, ok):
    print("CASE short of memory", share, flush=True)
    from paper_1510_03330_amd.ops import Solver, workspace_bytes
    p = ModelParams(Lx=2, Ly=2, Nv=16, U=1.3, beta=2.5, mu_mode=0, alpha=0.6)
    ref = Solver(p, "fp64")
    ref.iterate(2)
    real, room = torch.empty, int(share * workspace_bytes(p, "fp64"))

    def empty(size, *args, **kw):
        if kw.get("dtype") is torch.uint8 and size > room:
            raise torch.OutOfMemoryError("no room")
        return real(size, *args, **kw)

    monkeypatch.setattr(torch, "empty", empty)
    if not ok:
        with pytest.raises(torch.OutOfMemoryError):
            Solver(p, "fp64")
        return
    s = Solver(p, "fp64")
    assert s.ws.numel() <= room
    s.iterate(2)
    assert rel(s.get("phi"), ref.get("phi")) < TOL["fp64"]
