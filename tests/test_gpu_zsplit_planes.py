"""The two-launch 3D MHD stage update shares a leaf's planes out over 2 to 16
workgroups by the number of leaves: each split, coarse-fine faces, all
schedules.  Bar: bit for bit the one-launch kernel (variant 1), which evaluates
the same expressions plane after plane."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,levels", [(2, 1), (5, 1), (3, 2), (7, 1)])
@pytest.mark.parametrize("flux,limiter", [(W.HLLC, W.CADA), (W.HLL, W.VANLEER)])
def test_equals_the_one_launch_kernel(base, levels, flux, limiter):
    from paper_2004_03275_amd.forest import GpuForest

    s = W.mhd_blast_scheme(3, base, levels, limiter, flux)
    f, U = W.mhd_blast(3, radius=0.2, scheme=s)

    def steps(variant, sched):
        g = GpuForest(f)
        g.set_variant(variant)
        g.set_schedule(*sched)
        g.set_state(U)
        for _ in range(2):
            g.advance(0.1 * g.max_dt())
        out = g.get_state()
        g.close()
        return out

    ref = steps(1, (1, 1, 0))
    for sched in [(1, 1, 0), (1, 0, 0), (2, 1, 0)] + ([(0, 1, 0)] if base == 2 else []):
        assert np.array_equal(steps(2, sched), ref), sched
