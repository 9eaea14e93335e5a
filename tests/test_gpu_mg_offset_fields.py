"""Fields of the 3D multigrid that start 8 bytes past a 16-byte boundary (a
contiguous slice at an odd offset), on a grid whose finest level is in split
order.  Bar: the aligned fields' results bit for bit."""
import numpy as np
import pytest

from oracle import rd as R
import workloads as W

pytestmark = pytest.mark.gpu


def test_offset_fields_give_the_same_results():
    import torch

    from paper_2004_03275_amd import multigrid as M

    n = 32
    x = [1.0 + 0.1 * W.uniform01(3 + i, n ** 3).reshape((n,) * 3) for i in range(2)]
    p = R.SCHNAKENBERG_PARAMS

    def field(values, odd):
        values = np.ascontiguousarray(values).ravel()
        t = torch.empty(values.size + 1, dtype=torch.float64, device="cuda:0")[odd:odd + values.size]
        t.copy_(torch.from_numpy(values))
        assert t.is_contiguous() and (t.data_ptr() % 16 != 0) == bool(odd)
        return t

    def program(odd):
        mg = M.GpuMultigrid(3, n, R.NEUMANN, 1.0, nfields=2)
        f, phi = field(np.stack(x), odd), field(np.zeros((2,) + (n,) * 3), odd)
        mg.solve(f, phi, [30.0, 700.0], tol=1e-8)
        out = [phi.clone()]
        for scheme in (R.IMEX, R.SPLIT):
            u, v = field(x[0], odd), field(x[1], odd)
            mg.rd_step(u, v, 1e-3, scheme, p, 2, tol=1e-8)
            out += [u.clone(), v.clone()]
        torch.cuda.synchronize()
        mg.close()
        return out

    for a, b in zip(program(1), program(0)):
        assert torch.equal(a, b)
