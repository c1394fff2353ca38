"""Combine kernels whose rows take a whole wavefront (lane groups of 64) and those next to them (groups of 32):
parity with the oracle on small-integer gradients, exact in any order, with atomics and with records, signs, bags,
tables of mixed dimensions, runs that fill windows, end at their edges or stay alone, a last window of one token."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

M = 300_007


def _ids(n, seed):
    rng = np.random.default_rng(seed)
    ids = rng.zipf(1.3, size=n).astype(np.int64) % 10**6
    ids[: n // 4] = 3                                       # runs over many windows
    ids[n // 4: n // 2] = np.arange(n // 2 - n // 4)       # tokens that occur once
    return ids


# d: lane groups of 64 with 1, 2, 2 (lanes past d idle), 4 and 8 elements, of 32 with 3
@pytest.mark.parametrize("d,Z", [(64, 16), (128, 32), (100, 10), (200, 8), (512, 64), (96, 32)])
@pytest.mark.parametrize("sign", [0, 1])
@pytest.mark.parametrize("n", [1, 64, 65, 4161])
def test_rows_of_a_wavefront_match_the_oracle(d, Z, sign, n):
    h, H = P.both_hashes(d + Z, M, d, Z, sign)
    F = 1 if n < 100 else 3
    B = n // F
    ids = _ids(B * F, n)
    rng = np.random.default_rng(n)
    for bags in (False, True):
        off = np.concatenate([[0], np.sort(rng.integers(0, B * F + 1, size=B * F - 1)), [B * F]]).astype(np.int64) if bags else None
        use = ids if bags else ids.reshape(B, F)
        G = rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)
        ref, _ = oracle.backward(H, G, use, off, B, F)
        for opt in (dict(backward_route=robe.ROUTE_COMBINE), dict(backward_route=robe.ROUTE_REGIONS, region_records=1)):
            ga = torch.zeros(M, dtype=torch.float32, device="cuda:0")
            robe.robe_backward(h, P.to_dev(G), P.to_dev(use), P.to_dev(off) if bags else None, B, F, ga, options=robe.options(**opt))
            assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref), (bags, opt)


@pytest.mark.parametrize("sign", [0, 1])
@pytest.mark.parametrize("dims", [(16, 128, 64, 16), (512, 16, 256), (100, 20, 60)])
def test_mixed_rows_of_a_wavefront_match_the_oracle(dims, sign):
    Z = 20 if 100 in dims else 16
    h, H = P.both_hashes(sum(dims), M, max(dims), Z, sign)
    F, B = len(dims), 1501
    ids = _ids(B * F, 5).reshape(B, F)
    G = np.random.default_rng(1).integers(-2, 3, size=(B, sum(dims))).astype(np.float32)
    ref, _ = oracle.backward_mixed(H, dims, G, ids, None, B)
    for opt in (dict(backward_route=robe.ROUTE_COMBINE), dict(backward_route=robe.ROUTE_REGIONS, region_records=1)):
        ga = torch.zeros(M, dtype=torch.float32, device="cuda:0")
        robe.robe_backward_mixed(h, list(dims), P.to_dev(G), P.to_dev(ids), None, B, ga, options=robe.options(**opt))
        assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref), opt
