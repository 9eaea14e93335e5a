"""The 2D stage kernel (one 576-thread workgroup per CU that walks its leaves)
at its edges: fewer leaves than CUs, a count that is no multiple of the XCDs or
the CUs, more leaves than CUs, coarse-fine faces, a queue with few workgroups,
every flux and limiter.  Bar: bit for bit the split variant, which evaluates
the same expressions with one 256-thread workgroup per leaf."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _case(name, flux, limiter):
    if name.startswith("kh"):
        s = W.kh_scheme(int(name[2:]))
        s.flux, s.limiter = flux, limiter
        return W.kh(int(name[2:]), scheme=s)
    if name.startswith("ot"):
        s = W.ot_scheme(int(name[2:]))
        s.flux, s.limiter = flux, limiter
        return W.orszag_tang(int(name[2:]), scheme=s)
    if name == "dam":
        s = W.dam_break_scheme(7, 3, flux)
        s.limiter = limiter
        return W.dam_break(scheme=s)
    s = W.mhd_blast_scheme(2, 9, 3, limiter, flux)
    return W.mhd_blast(2, scheme=s)


@pytest.mark.parametrize("name,flux", [("kh3", W.HLLC), ("kh17", W.HLLC), ("kh17", W.TVDLF), ("kh17", W.HLL),
                                       ("ot17", W.HLL), ("ot17", W.TVDLF), ("dam", W.HLL), ("dam", W.TVDLF),
                                       ("mhd", W.HLLC)])
@pytest.mark.parametrize("limiter", [W.MINMOD, W.VANLEER, W.MC, W.KOREN, W.CADA])
def test_equals_the_split_variant(name, flux, limiter):
    from paper_2004_03275_amd.forest import GpuForest

    f, U = _case(name, flux, limiter)

    def steps(variant, sched):
        g = GpuForest(f)
        g.set_variant(variant)
        g.set_schedule(*sched)
        g.set_state(U)
        for _ in range(3):
            g.advance(g.max_dt())
        out = g.get_state()
        g.close()
        return out

    ref = steps(1, (1, 1, 0))
    for sched in [(1, 1, 0), (1, 0, 0), (2, 1, 0), (2, 0, 3)]:
        assert np.array_equal(steps(0, sched), ref), sched
