"""Tokens that the sort of a window cannot tell apart: it looks at 26 of 31 key bits and takes the two highest values of
those for one.  Runs are found by the whole key, so that such tokens cut each other's runs and nothing else:
parity with the oracle on small-integer gradients, exact in any order, through the atomics, the records, the direct
scatter's windows and blocks larger than embeddings (whose keys are array offsets), for lane groups of 16 to 64."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

LOW = 2**26


def _plain_keys(m, d, Z, sign):
    """A hash whose token part is the token: Bh = 1, Dh = 0, and one table."""
    h, H = P.both_hashes(5, m, d, Z, sign)
    c = list(H.coef)
    c[0:4] = [1, 1, c[2], 0]
    h.Ah, h.Bh, h.Dh = 1, 1, 0
    assert list(h.coef) == c
    return h, dataclasses.replace(H, coef=tuple(c))


def _ids(n, most, step=1):
    """Equal in 26 bits, or 2^26 - 2 and 2^26 - 1 there, in turn."""
    rng = np.random.default_rng(n)
    low = np.array([5, LOW - 2, LOW - 1, LOW - 3, 6])[rng.integers(0, 5, size=n)]
    return ((low + LOW * rng.integers(0, most, size=n)) * step).astype(np.int64)


@pytest.mark.parametrize("sign", [0, 1])
@pytest.mark.parametrize("d,Z", [(16, 16), (32, 8), (48, 24), (64, 16), (128, 32)])
def test_tokens_that_agree_in_26_bits(d, Z, sign):
    m = 300_007
    h, H = _plain_keys(m, d, Z, sign)
    for n in (61, 130, 5000):
        for most in (2, 31):
            ids = _ids(n, most).reshape(n, 1)
            G = np.random.default_rng(d).integers(-2, 3, size=(n, 1, d)).astype(np.float32)
            ref, _ = oracle.backward(H, G, ids, None, n, 1)
            for asked in (dict(backward_route=robe.ROUTE_COMBINE), dict(backward_route=robe.ROUTE_REGIONS, region_records=1), dict(reproducible=1),
                          dict(backward_route=robe.ROUTE_DIRECT, tile_combine=2)):
                ga = torch.zeros(m, device="cuda:0")
                robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), None, n, 1, ga, options=robe.options(**asked))
                assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref), (n, most, asked)


@pytest.mark.parametrize("sign", [0, 1])
def test_offsets_that_agree_in_26_bits(sign):
    """Z > d: the sort looks at the low bits of an array offset, the windows at its 26 lowest."""
    m, d, Z, n = 2**27 + 2**20, 16, 64, 5000
    h, H = _plain_keys(m, d, Z, sign)
    ids = _ids(n, 2, step=Z // d).reshape(n, 1)
    G = np.random.default_rng(d).integers(-2, 3, size=(n, 1, d)).astype(np.float32)
    ref, _ = oracle.backward(H, G, ids, None, n, 1)
    ga = torch.zeros(m, device="cuda:0")
    robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), None, n, 1, ga, options=robe.options(backward_route=robe.ROUTE_COMBINE))
    got = ga.cpu().numpy()
    assert np.array_equal(got.astype(np.float64), ref)
