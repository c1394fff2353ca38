"""Samples of about 2^23 floats or tables, where the kernels that walk rows change from 32-bit distances to 64-bit ones:
forward of lookups and bags (bit for bit) and the direct backward (exact on small integers), in both row orders,
against the shape-generic kernels, which have one form."""
import numpy as np
import pytest
import torch

import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
M = 777_777
ORDERS = (robe.ROWS_MEMORY, robe.ROWS_BY_TABLE, robe.ROWS_BY_TABLE_ALWAYS)


def _generic(**asked):
    return robe.options(fwd_elems=-1, bwd_elems=-1, **asked)


@pytest.mark.parametrize("F", [65_535, 65_536, 65_537])
@pytest.mark.parametrize("Z,B,sign", [(32, 2, 1), (8, 3, 0), (512, 3, 1)])
def test_samples_of_two_to_the_23_floats(F, Z, B, sign):
    d = 128
    h, _ = P.both_hashes(F, M, d, Z, sign)
    rng = np.random.default_rng(F)
    A = torch.randn(M, device=DEV)
    I = P.to_dev(rng.integers(0, 300, size=(B, F)))
    sizes = rng.integers(0, 4, size=B * F)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    T, O = P.to_dev(rng.integers(0, 300, size=int(off[-1]))), P.to_dev(off)
    for ids, offsets in ((I, None), (T, O)):
        want = robe.robe_forward(h, A, ids, offsets, B, F, options=_generic())
        for order in ORDERS:
            got = robe.robe_forward(h, A, ids, offsets, B, F, options=robe.options(row_order=order))
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (offsets is None, order)
        G = torch.randint(-2, 3, (B, F, d), device=DEV).float()
        sums = []
        for opt in [_generic(backward_route=robe.ROUTE_DIRECT)] + [robe.options(backward_route=robe.ROUTE_DIRECT, tile_combine=t, row_order=o)
                                                                   for t in (1, 2) for o in ORDERS]:
            ga = torch.zeros(M, device=DEV)
            robe.robe_backward(h, G, ids, offsets, B, F, ga, options=opt)
            sums.append(ga)
        assert all(torch.equal(s, sums[0]) for s in sums[1:]), offsets is None


@pytest.mark.parametrize("F", [2**23 - 1, 2**23, 2**23 + 1])
def test_samples_of_two_to_the_23_tables(F):
    """Narrow rows: the line is crossed by the floats of d = 1 and by the tables alike."""
    h, _ = P.both_hashes(F, M, 1, 4, 0)
    A = torch.randn(M, device=DEV)
    I = torch.randint(0, 300, (2, F), device=DEV)
    want = robe.robe_forward(h, A, I, None, 2, F, options=_generic())
    for order in ORDERS:
        got = robe.robe_forward(h, A, I, None, 2, F, options=robe.options(row_order=order))
        assert torch.equal(got.view(torch.int32), want.view(torch.int32)), order
