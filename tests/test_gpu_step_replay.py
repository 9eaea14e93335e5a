"""Device-timed steps in 3D replayed from the graph of eight steps (taken by a
call of eight steps or more on a forest that has run 64 of them directly to the
same end time): coarse-fine faces with the stage kernel's own restriction, and
MHD, whose time steps come from a launch of their own.  Replays follow direct
remainders, host-timed steps, a new state and a change of schedule.

Bar: as for direct steps, the host-timed run bit for bit; MHD, whose damping
factor is evaluated on the device, 1e-12 of max|U| (test_gpu_step_clock.py)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _case(name):
    if name == "blast":
        return W.blast(W.blast_scheme(3, 2), radius=0.12)
    if name == "blast_split":
        return W.blast(W.blast_scheme(3, 2), radius=0.12)
    if name == "mhd":
        return W.mhd_blast(3, 4, 1)
    return W.mhd_blast(3, 2, 2)


@pytest.mark.parametrize("sched", [(1, 1, 0), (2, 0, 0)])
@pytest.mark.parametrize("name", ["blast", "blast_split", "mhd", "mhd_amr"])
def test_replayed_steps_equal_host_timed_ones(name, sched):
    from paper_2004_03275_amd.forest import GpuForest

    f, U = _case(name)
    exact = name.startswith("blast")
    forests = []
    for _ in range(2):
        g = GpuForest(f)
        if name == "blast_split":
            g.set_variant(1)
        g.set_schedule(*sched)
        g.set_state(U)
        forests.append(g)
    h, g = forests

    def host(steps):
        t = 0.0
        for _ in range(steps):
            dt = h.max_dt()
            h.advance(dt)
            t += dt
        return t

    def check(want, got):
        ref = h.get_state()
        assert abs(want - got) <= 1e-12 * want
        assert np.abs(g.get_state() - ref).max() <= (0.0 if exact else 1e-12 * np.abs(ref).max())

    def device(steps):
        t, taken = g.advance_cfl(steps, float("inf"), 0.0)
        assert taken == steps
        return t

    check(host(64), device(64))
    check(host(19), device(19))  # two graphs and three direct steps
    dt = h.max_dt()
    h.advance(0.5 * dt)
    g.advance(0.5 * g.max_dt())
    check(host(8), device(8))  # after a host-timed step
    h.set_state(U)
    g.set_state(U)
    check(host(17), device(17))  # after a new state
    g.set_schedule(1, 0, 0)
    check(host(9), device(9))  # the graph was dropped
    h.close()
    g.close()
