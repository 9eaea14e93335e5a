"""Restriction, prolongation and fine fluxes in one launch (1D and 2D forests):
refined lines against the oracle, bit for bit, through both drivers (quadtrees:
the parity tests)."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [16, 30, 256])
@pytest.mark.parametrize("base,levels", [(2, 2), (3, 3)])
def test_refined_line(nx, base, levels):
    from paper_2004_03275_amd import forest as F

    s = W.sod_scheme(nx)
    s.base_blocks = (base, 1, 1)
    s.max_level = levels
    f = W.refined_forest(s, lambda lvl, ijk: lvl < levels and ijk[0] == (base << (lvl - 1)) // 2)
    x = W.cell_centres(f)[0]
    left = x < 0.5
    U = W.state_from_primitive(f, np.where(left, 1.0, 0.125), [np.zeros_like(x)], np.where(left, 1.0, 0.1))
    R, _ = oracle.run(f, U, steps=6)
    for dev in (False, True):
        G, _ = F.run(f, U, steps=6, device_dt=dev)
        assert np.array_equal(G, R)
