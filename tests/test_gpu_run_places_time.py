"""The backward of small blocks takes no longer on a small array than on a larger one: the last kernel's workgroups, one per region of
the array, are made as many as CUs by smaller regions."""
import numpy as np
import pytest
import torch

import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# 520 000 slots against four million: 1.00, 1.07, 1.09; 3.7, 3.1, 3.2 with regions of 2^14 slots on both
@pytest.mark.parametrize("d,Z,F,B", [(128, 1, 26, 8000), (128, 2, 26, 33_000), (16, 2, 26, 50_000)])
def test_small_arrays_fill_the_gpu(d, Z, F, B):
    ids = P.to_dev(np.random.default_rng(B).integers(0, B // 2, size=(B, F)))
    G = torch.randn(B, F, d, device=DEV)
    took = []
    for m in (520_000, 4_000_000):
        h, _ = P.both_hashes(3, m, d, Z, 0)
        grad = torch.zeros(m, device=DEV)
        work = torch.empty(robe.robe_workspace_bytes(h, B, F, B * F), dtype=torch.uint8, device=DEV)
        times = []
        for _ in range(15):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(4):
                robe.robe_backward(h, G, ids, None, B, F, grad, workspace=work)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end) * 250)
        took.append(float(np.median(times)))
    print(d, Z, B * F, "%.0f / %.0f us" % tuple(took), flush=True)
    assert took[0] < 1.5 * took[1]
