"""Device-timed steps (amrv_advance_cfl) on each way the step's clock can run:
inside the stage kernels (1D, 2D), from a launch of its own (a launch per leaf,
MHD with coarse-fine faces, 3D), launched directly and replayed from a graph of
several steps, and steps at or after t_end that do nothing.

Bar: the host-timed run (max_dt, advance) bit for bit, since the arithmetic is
the same; 2D/3D MHD evaluates the damping factor exp(-dt ch^2/cp^2) on the
device, whose last-place difference (2.2e-16 per step on psi alone) may grow by
at most the step count times the stages' amplification: 1e-12 of max|U|."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _case(name):
    if name == "line":
        return W.sod(256, 4)
    if name == "kh":
        return W.kh(3)
    if name == "ot":
        return W.orszag_tang(3)
    if name == "dam":
        return W.dam_break(3, 2)
    if name == "mhd_amr":
        return W.mhd_blast(2, 4, 2)
    if name == "mhd3":
        return W.mhd_blast(3, 4, 1)
    s = W.blast_scheme(3, 2)
    return W.blast(s, radius=0.12)


@pytest.mark.parametrize("sched", [(1, 1, 0), (2, 0, 0), (0, 1, 0)])
@pytest.mark.parametrize("name,steps", [("line", 90), ("kh", 90), ("ot", 90), ("dam", 90), ("mhd_amr", 90),
                                        ("mhd3", 12), ("blast", 12)])
def test_device_timed_equals_host_timed(name, steps, sched):
    from paper_2004_03275_amd.forest import GpuForest

    f, U = _case(name)
    h = GpuForest(f)
    h.set_schedule(*sched)
    h.set_state(U)
    t, times = 0.0, [0.0]
    for _ in range(steps):
        dt = h.max_dt()
        h.advance(dt)
        t += dt
        times.append(t)
    ref = h.get_state()
    bar = 1e-12 * np.abs(ref).max() if name in ("ot", "mhd_amr", "mhd3") else 0.0
    g = GpuForest(f)
    g.set_schedule(*sched)
    g.set_state(U)
    td, n, left = 0.0, 0, steps
    for k in (1, 2, 3, 30, 30, 19, steps):  # direct, then a graph with a remainder
        k = min(k, left)
        if k == 0:
            break
        td, taken = g.advance_cfl(k, float("inf"), td)
        assert taken == k
        left -= k
    assert left == 0 and abs(td - t) <= 1e-12 * t
    assert np.abs(g.get_state() - ref).max() <= bar
    # an end time between two steps: the rest of the steps do nothing, and later calls neither
    m = steps - 3
    t_end = 0.5 * (times[m] + times[m + 1])
    h.set_state(U)
    t = 0.0
    while t < t_end:
        dt = min(h.max_dt(), t_end - t)
        h.advance(dt)
        t += dt
    ref = h.get_state()
    g.set_state(U)
    td, n = g.advance_cfl(steps + 8, t_end, 0.0)
    assert n == m + 1 and abs(td - t_end) <= 1e-12 * t_end
    assert np.abs(g.get_state() - ref).max() <= bar
    td, n = g.advance_cfl(5, t_end, td)
    assert n == 0 and np.abs(g.get_state() - ref).max() <= bar
    h.close()
    g.close()
