"""The library's host code without a device, over the calls of fake_hip.c: what
it launches and when, from a process of its own."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

HEAD = """
import ctypes, sys, threading
sys.path.insert(0, sys.argv[2])
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from ctypes import byref, c_int32, c_size_t, c_void_p
from paper_1510_03330_amd import native as N
from workloads import ModelParams
lib = N.load()

def setting(name):
    return ctypes.c_int.in_dll(fake, name)

def room(nbytes):                           # host memory in place of a workspace
    return ctypes.create_string_buffer(int(nbytes) + 256)
"""


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-pthread", os.path.join(HERE, "fake_hip.c"), "-o", so], check=True)
    return so


def run(so, body):
    res = subprocess.run([sys.executable, "-c", HEAD + textwrap.dedent(body), so, ROOT], capture_output=True, text=True,
                         timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr


def test_one_thread_at_a_time_in_graph_calls(fake_hip):
    """Two batches and two sets of contexts, each with a thread of its own: no graph
    call of one meets one of another, and every round is launched."""
    run(fake_hip, """
        setting("fake_graph_us").value = 3000
        p = ModelParams(Lx=2, Ly=1, Nv=4, U=1.0, beta=2.0, mu_mode=0, alpha=0.6)
        start = threading.Barrier(4)
        bad = []

        def batch(t):
            pp = (N.PqParams * 2)(*[N.make_params(p, "fp64")] * 2)
            need, h, left = c_size_t(), c_void_p(), c_int32()
            N.check(lib.parquet_batch_query_workspace(pp, 2, byref(need)))
            ws = room(need.value)
            N.check(lib.parquet_batch_init(pp, 2, ws, need, c_void_p(16 + t), 0, byref(h)))
            start.wait()
            for _ in range(5):
                bad.append(lib.parquet_batch_iterate(h, 2, 0.0, 0.0, byref(left)) or left.value != 2)
            N.check(lib.parquet_batch_destroy(h))

        def contexts(t):
            pp = N.make_params(p, "fp64")
            need, done = c_size_t(), (c_int32 * 2)()
            N.check(lib.parquet_query_workspace(byref(pp), byref(need)))
            ws, cs = [room(need.value) for _ in range(2)], (c_void_p * 2)()
            for i in range(2):
                c = c_void_p()
                N.check(lib.parquet_init(byref(pp), ws[i], need, c_void_p(32 + 2 * t + i), byref(c)))
                cs[i] = c.value
            start.wait()
            for _ in range(5):
                bad.append(lib.parquet_iterate_batch(cs, 2, 2, 0.0, done, None) or list(done) != [2, 2])
            for c in cs:
                N.check(lib.parquet_destroy(c))

        th = [threading.Thread(target=f, args=(t,)) for t in range(2) for f in (batch, contexts)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert len(bad) == 20 and not any(bad), bad
        # a capture, an instantiation and two destructions per graph, and the rounds
        assert setting("fake_graph_calls").value == 4 * (2 + 4) + 2 * 10 + 4 * 10
        assert setting("fake_overlaps").value == 0, setting("fake_overlaps").value
    """)


@pytest.mark.parametrize("batch,widths", [(33, (3, 65, 7)), (2 ** 20 + 33, (3, 8192, 5)), (4194240, (2, 2100, 2050)),
                                          (40, (2, 4194240, 3))])
def test_perceptron_grids(fake_hip, batch, widths):
    """Every launch of the forward and backward pass within the limits of a grid (a
    dimension below 2^32 work items, the second and third at most 65535 workgroups),
    with a workgroup for every 32 x 32 tile."""
    run(fake_hip, f"""
        batch, widths = {batch}, {widths}
        w, nl, a = (c_int32 * len(widths))(*widths), {len(widths) - 1}, c_void_p(0x100000)
        N.check(lib.mlp_forward(w, nl, a, a, a, a, batch, None))
        N.check(lib.mlp_backward(w, nl, a, a, a, a, a, a, a, batch, None))
        n = setting("fake_launches").value
        dims = [list(d) for d in ((ctypes.c_uint * 6) * 4096).in_dll(fake, "fake_dims")[:n]]
        for d in dims:
            assert all(0 < d[i] * d[3 + i] < 2 ** 32 for i in range(3)), d
            assert max(d[1:3]) <= 65535, d

        def up(x, k):
            return -(-x // k)

        fwd = [up(o, 32) * up(batch, 32) for o in widths[1:]]
        bwd = [up(o, 32) * up(i, 256) + up(o, 512) + (up(i, 32) * up(batch, 32) if l else 0)
               for l, (i, o) in enumerate(zip(widths, widths[1:]))][::-1]
        got = [d for d in dims if d[3] == 512]
        assert len(got) == 2 * nl
        for d, need in zip(got, fwd + bwd):
            assert need <= d[0] * d[1] <= need + d[0], (d, need)       # one more: the loss
    """)


@pytest.mark.parametrize("fill,status", [(255, "PQ_ERR_NONFINITE"), (1, "PQ_ERR_SINGULAR")])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_times_of_an_iteration_that_fails(fake_hip, fill, status, prec):
    """A call that an error ends before its last iteration reports that iteration's
    times (1 ms an event pair here). fill: the results' bytes, NaN or a positive
    count of unresolved blocks."""
    run(fake_hip, f"""
        setting("fake_host_fill").value = {fill}
        pp = N.make_params(ModelParams(Lx=2, Ly=1, Nv=4, U=1.0, beta=2.0, mu_mode=0, alpha=0.6), "{prec}")
        need, c, done, st = c_size_t(), c_void_p(), c_int32(), N.PqIterStats()
        N.check(lib.parquet_query_workspace(byref(pp), byref(need)))
        ws = room(need.value)
        N.check(lib.parquet_init(byref(pp), ws, need, c_void_p(16), byref(c)))
        assert lib.parquet_iterate(c, 3, 0.0, byref(st), byref(done), None) == N.{status}
        assert done.value == 1 and st.iteration == 1
        assert st.ms_total == 1.0 and [st.ms_stage[i] for i in (0, 1, 3, 4, 5, 6)] == [1.0] * 6
        assert sum(st.n_bse_launch) > 0 and sum(st.ms_bse_kernel) == 0.25 * sum(st.n_bse_launch)
        N.check(lib.parquet_destroy(c))
    """)
