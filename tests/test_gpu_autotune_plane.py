"""The autotuner tries the 2D stage kernel's own shape, one workgroup per CU,
with the queue too; it keeps the state whichever schedule it takes."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_one_workgroup_per_cu_is_tried():
    import torch

    from paper_2004_03275_amd.forest import GpuForest

    f, U = W.kh(6)
    g = GpuForest(f)
    g.set_state(U)
    g.autotune(1)
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    rows = g.autotune_report().splitlines()
    for x in (0, 1):
        assert any(r.startswith(f"sched=2 xcd={x} wgs={ncu} variant=0:") for r in rows), rows
    assert np.array_equal(g.get_state(), U)
    g.close()
