"""max_dt and advance_cfl wait for the GPU, so they are refused while the
forest's stream is being captured into a graph.  A refused call leaves the
forest as it was: what follows outside the capture gives the values of a forest
that never saw one, bit for bit.  The workspace starts as 0x7f bytes, so that
reduction slots or ghost slabs which only the captured (never executed) work
would have filled cannot pass for clear ones."""
import ctypes

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _cases(name):
    if name == "line":
        return W.sod(64)
    if name == "dam":
        return W.dam_break(3, 2)
    if name == "mhd":
        return W.mhd_blast(2, 4, 1)
    return W.blast(W.blast_scheme(3, 2), radius=0.12)


def _hip(name, *args):
    from paper_2004_03275_amd import _native as N

    fn = getattr(N.lib(), name)  # a dependency of the library
    fn.restype = ctypes.c_int
    return fn(*args)


def _program(g):
    dt = g.max_dt()
    g.advance(0.5 * dt)
    t, n = g.advance_cfl(3, float("inf"), 0.0)
    return dt, t, n, g.max_dt(), g.get_state()


@pytest.mark.parametrize("calls", [("max_dt",), ("advance_cfl",), ("advance_cfl", "max_dt")])
@pytest.mark.parametrize("name", ["line", "dam", "mhd", "blast"])
def test_a_refused_call_changes_nothing(name, calls):
    import torch

    from paper_2004_03275_amd import _native as N
    from paper_2004_03275_amd.forest import GpuForest

    f, U = _cases(name)

    def forest():
        g = GpuForest(f)
        size = g.workspace.numel()
        g.close()
        del g
        torch.cuda.synchronize()
        t = torch.full((size,), 0x7f, dtype=torch.uint8, device="cuda:0")
        torch.cuda.synchronize()
        at = t.data_ptr()
        del t  # its memory is the next workspace
        g = GpuForest(f)
        assert g.workspace.data_ptr() == at
        g.set_state(U)
        return g

    h = forest()
    ref = _program(h)
    h.close()
    del h
    g = forest()
    st = ctypes.c_void_p(g.stream.cuda_stream)
    assert _hip("hipStreamBeginCapture", st, ctypes.c_int(1)) == 0  # thread-local
    try:
        for c in calls:
            with pytest.raises(N.AmrvError):
                g.max_dt() if c == "max_dt" else g.advance_cfl(2, float("inf"), 0.0)
    finally:
        graph = ctypes.c_void_p()
        rc = _hip("hipStreamEndCapture", st, ctypes.byref(graph))
        if graph.value:
            _hip("hipGraphDestroy", graph)
        _hip("hipGetLastError")
    assert rc == 0  # nothing was enqueued: the caller's capture and the stream stay usable
    got = _program(g)
    assert got[:4] == ref[:4]
    assert np.array_equal(got[4], ref[4])
    g.close()
