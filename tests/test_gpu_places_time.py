"""Single-hot lookups of blocks of one or two floats, by place against gathered: the same ids on an array of as many slots as
blocks are read and on one of a slot more, which differ in nothing else that counts.  Where the device turns the lists down
such a call must take little longer than one that has none; where it serves them, clearly less (had it turned them down, the result
would be the same bits).  Times are medians of calls in turn, both sides far from the line."""
import numpy as np
import pytest
import torch

import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P
from tests.launches import kernels

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _by_place_over_gathered(d, Z, F, B, ids):
    m = B * F * (d // Z)
    A, I, out = torch.randn(m + 1, device=DEV), P.to_dev(ids), torch.empty(B, F, d, device=DEV)
    calls = []
    for slots, launches in ((m, 8), (m + 1, 5)):
        h, _ = P.both_hashes(3, slots, d, Z, 0)
        call = lambda h=h, a=A[:slots]: robe.robe_forward(h, a, I, None, B, F, out=out)  # noqa: E731
        assert kernels(call) == launches
        calls.append(call)
    times = ([], [])
    for _ in range(15):
        for call, took in zip(calls, times):
            call()
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(4):
                call()
            end.record()
            torch.cuda.synchronize()
            took.append(start.elapsed_time(end))
    ratio = float(np.median(times[0]) / np.median(times[1]))
    print(d, Z, B * F, m, f"{np.median(times[0]) * 250:.0f} / {np.median(times[1]) * 250:.0f} us", flush=True)
    return ratio


def _uniform(B, F, each):
    return np.random.default_rng(B).integers(0, each, size=(B, F))


# (d, Z, F, B, ids of a table): fewer ids than are worth the lists.  1.07, 1.06, 1.05; 1.43, 1.46, 1.51 when the kernel that places the
# entries also gathered 64 rows a wavefront and all of the last samples were gathered
@pytest.mark.parametrize("d,Z,F,B,each", [(128, 1, 26, 15_900, 1200), (128, 2, 26, 33_000, 2400), (128, 1, 26, 30_000, 1200)])
def test_lists_turned_down_cost_little(d, Z, F, B, each):
    assert _by_place_over_gathered(d, Z, F, B, _uniform(B, F, each)) < 1.2


# (rows of 512 chunks: as many lines as would do with 128 lie in windows of few entries.  1.01, 1.03; served all the same 1.29, 1.50)
@pytest.mark.parametrize("d,Z,F,B,each", [(512, 1, 26, 3840, 820), (512, 1, 26, 3840, 540)])
def test_wide_rows_are_served_where_it_pays(d, Z, F, B, each):
    assert _by_place_over_gathered(d, Z, F, B, _uniform(B, F, each)) < 1.2


# (twice the ids that are worth it and more, each several times: 0.66, 0.76, 0.64)
@pytest.mark.parametrize("d,Z,F,B,each", [(128, 1, 26, 15_900, 4000), (128, 2, 26, 33_000, 8000), (64, 1, 26, 34_000, 8000)])
def test_lists_served_pay(d, Z, F, B, each):
    assert _by_place_over_gathered(d, Z, F, B, _uniform(B, F, each)) < 0.9
