"""The pinned words that max_dt and advance_cfl leave their results in: more
forests alive than a page holds, words reused after a forest is closed, several
threads on streams of their own, and the reduction that amrv_max_dt hands on to
advance_cfl and clears for its next call.  Bar: the first forest's values, bit
for bit (all run the same program)."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _program(g, U):
    g.set_state(U)
    out = [g.max_dt(), g.max_dt()]
    g.advance(0.5 * out[0])
    out.append(g.max_dt())
    t, n = g.advance_cfl(3, float("inf"), 0.0)
    out += [t, n, g.max_dt()]
    g.set_state(U)
    out.append(g.max_dt())
    assert out[0] == out[1] == out[6] and n == 3
    return out


@pytest.mark.parametrize("make", [lambda: W.sod(64), lambda: W.orszag_tang(2)])
def test_many_forests_and_threads(make):
    import torch

    from paper_2004_03275_amd.forest import GpuForest

    f, U = make()
    first = GpuForest(f)
    want = _program(first, U)
    forests = [GpuForest(f) for _ in range(140)]
    for g in forests:
        assert _program(g, U) == want
    for g in forests[::2]:
        g.close()
    more = [GpuForest(f) for _ in range(20)]
    for g in more + forests[1::2]:
        assert _program(g, U) == want
    for g in more + forests[1::2]:
        g.close()
    got = [None] * 4

    def work(i):
        s = torch.cuda.Stream()
        for _ in range(10):
            g = GpuForest(f, stream=s)
            got[i] = _program(g, U)
            g.close()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(r == want for r in got)
    assert _program(first, U) == want
    first.close()
