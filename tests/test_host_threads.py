"""Host state that threads share, on the CPU."""
import contextlib
import threading
import types
import weakref

import pytest

torch = pytest.importorskip("torch")

from paper_1510_03330_amd import ops


def test_stream_pool_last_stream_taken_by_another_thread(monkeypatch):
    """Two threads find one pooled stream: one takes it, the other gets a new one."""
    both = threading.Barrier(2)

    class Pool(list):
        def __len__(self):                   # a thread that asks waits for the other to ask too
            n = super().__len__()
            with contextlib.suppress(threading.BrokenBarrierError):
                both.wait(0.2)
            return n

    made = []
    hip = types.SimpleNamespace(hipStreamCreate=lambda h: 0)
    monkeypatch.setattr(ops, "_hip", hip)
    monkeypatch.setattr(ops, "_stream_pool", {"cuda:0": Pool(["pooled"])})
    monkeypatch.setattr(torch.cuda, "device", lambda d: contextlib.nullcontext())
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda h, device: made.append(device) or "new")
    got, errors = [], []

    def take():
        try:
            got.append(ops.new_stream("cuda:0"))
        except Exception as err:             # reported below, in the main thread
            errors.append(err)

    th = [threading.Thread(target=take) for _ in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errors and sorted(got) == ["new", "pooled"] and len(made) == 1


class Lib:
    """The batch's entry points without a device."""

    def __init__(self, status=ops.N.PQ_OK):
        self.status = status

    def parquet_batch_query_workspace(self, pp, count, out):
        out._obj.value = 1000
        return ops.N.PQ_OK

    parquet_batch_query_workspace_min = parquet_batch_query_workspace

    def parquet_batch_init(self, pp, count, ws, size, stream, autotune, out):
        out._obj.value = 1
        return self.status

    def parquet_batch_destroy(self, h):
        return ops.N.PQ_OK

    def parquet_last_error(self):
        return b"refused"


class Device:
    """torch's allocations, those still held."""

    def __init__(self):
        self.live = []

    def empty(self, size, dtype, device):
        t = Buffer(size)
        self.live.append(weakref.ref(t))
        return t

    def held(self):
        return sum(r() is not None for r in self.live)


class Buffer:
    def __init__(self, size):
        self.size = size

    def numel(self):
        return self.size

    def data_ptr(self):
        return 0x1000

    def record_stream(self, stream):
        pass


@pytest.mark.parametrize("status", [ops.N.PQ_OK, ops.N.PQ_ERR_HIP])
def test_batch_frees_its_workspace_before_its_stream(monkeypatch, status):
    """A stream that goes back to the pool may be captured by its next user at once;
    freeing a tensor recorded on it puts an event there. Closed and refused batches."""
    from workloads import ModelParams
    ps = [ModelParams(Lx=2, Ly=1, Nv=4, U=1.0, beta=2.0, mu_mode=0, alpha=0.6)] * 3
    dev, lib, held = Device(), Lib(status), []
    monkeypatch.setattr(ops.N, "load", lambda: lib)
    monkeypatch.setattr(ops, "Stage", lambda *a: None)
    monkeypatch.setattr(torch, "empty", dev.empty)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda d=None: None)
    monkeypatch.setattr(ops, "new_stream", lambda d: types.SimpleNamespace(cuda_stream=0x20))
    monkeypatch.setattr(ops, "release_stream", lambda s: held.append(dev.held()))
    if status == ops.N.PQ_OK:
        b = ops.Batch(ps, "fp64")
        assert dev.held() == 1
        b.close()
    else:
        with pytest.raises(ops.N.ParquetError):
            ops.Batch(ps, "fp64")
    assert held == [0]
