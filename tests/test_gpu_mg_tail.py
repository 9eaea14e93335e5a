"""The multigrid's coarse tail at the edges of its parts: grids of at most 64
cells (one wave), the level above the coarse matrix as the whole grid, one and
two levels in between, and sweep counts other than two.  Bar: the M-matrix
bound of the solve, max|phi - exact| <= max|r| / lambda (doubled for the
residual's rounding), and the same answer from a second solve with another
lambda in between (the coarse matrix follows lambda)."""
import numpy as np
import pytest

from oracle import rd as R
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nd,n", [(2, 4), (2, 8), (2, 16), (2, 32), (2, 128), (3, 4), (3, 8), (3, 16), (3, 32)])
@pytest.mark.parametrize("bc", [R.PERIODIC, R.NEUMANN])
@pytest.mark.parametrize("pre,post,nf", [(2, 2, 1), (1, 3, 2), (3, 1, 2)])
def test_tail_solves_within_the_residual_bound(nd, n, bc, pre, post, nf):
    import torch

    from paper_2004_03275_amd import multigrid as M

    lam = np.array([30.0, 700.0])[:nf]
    rng = W.uniform01(7 + n + nd, nf * n ** nd).reshape((nf,) + (n,) * nd)
    f = 2.0 * rng - 1.0 + np.cos(2 * np.pi * W.rd_cell_centres(nd, n, 1.0)[0])
    mg = M.GpuMultigrid(nd, n, bc, 1.0, nfields=nf, pre=pre, post=post)
    ft = torch.tensor(f, device="cuda:0").contiguous()
    phi = torch.zeros_like(ft)
    _, res, fmax = mg.solve(ft, phi, lam, tol=1e-10, max_cycles=80)
    got = phi.cpu().numpy()
    for i in range(nf):
        exact = R.helmholtz_solve(f[i], lam[i], 1.0, bc)
        assert res[i] <= 1e-10 * fmax[i]
        assert np.abs(got[i] - exact).max() <= 2.0 * res[i] / lam[i] + 1e-12 * np.abs(exact).max()
    other = torch.zeros_like(ft)
    mg.solve(ft, other, lam * 5.0, tol=1e-10, max_cycles=80)
    again = torch.zeros_like(ft)
    mg.solve(ft, again, lam, tol=1e-10, max_cycles=80)
    mg.close()
    assert torch.equal(again, phi) and not torch.equal(other, phi)
