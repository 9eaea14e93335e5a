"""The training step's split over workgroups (32 rows each, then the sums over
the rows, 1,024 staged at a time) against the CPU reference: the gradient of
the last batch at the edges of the split, lr = 0 so the weights stay.  Bar as for the single batch:
relative L2 error 1e-3 (binary32 accumulation order; bfloat16 rounding points
identical)."""
import ctypes

import numpy as np
import pytest

from oracle import mlp as M
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n", [(32, 32), (32, 33), (96, 70), (1024, 1024),
                                     (1056, 1030), (2048, 2048), (2080, 2049), (4096, 4096), (4096, 5)])
def test_gradient_of_split_batches(batch, n):
    import torch

    from paper_2004_03275_amd import _native as N

    X, y = W.mlp_random_features(31, n)
    w0 = W.mlp_init(6)
    order = np.random.default_rng(3).permutation(n).astype(np.int32)
    nbatch = (n + batch - 1) // batch
    dev = torch.device("cuda:0")
    Xd, yd, od = torch.from_numpy(X.view(np.int16)).to(dev), torch.from_numpy(y).to(dev), torch.from_numpy(order).to(dev)
    w = torch.from_numpy(w0.copy()).to(dev)
    m, v, grad = torch.zeros_like(w), torch.zeros_like(w), torch.zeros_like(w)
    loss = torch.zeros(nbatch, dtype=torch.float32, device=dev)
    ws = torch.empty(int(N.lib().amrv_mlp_train_workspace_bytes(batch)), dtype=torch.uint8, device=dev)
    cfg = N.TrainCfg(0.0, 0.9, 0.999, 1e-8, 2.0, 1.5, 0)
    torch.cuda.synchronize()
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    N.check(N.lib().amrv_mlp_train(p(Xd), p(yd), p(od), n, batch, 0, nbatch, p(w), p(m), p(v), ctypes.byref(cfg),
                                   p(ws), ws.numel(), None, p(loss), p(grad)))
    torch.cuda.synchronize()
    last = order[(nbatch - 1) * batch:]
    gr, lr = M.grad_bf16(w0, X[last], y[last], 2.0, 1.5)
    rel = np.linalg.norm(grad.cpu().numpy() - gr) / np.linalg.norm(gr)
    print(f"[mlp] batch {batch} n {n}: grad rel err {rel:.2e}", flush=True)
    assert rel <= 1e-3
    assert abs(float(loss[-1]) - lr) <= 1e-4 * max(1.0, lr)
    assert np.array_equal(w.cpu().numpy(), w0)
