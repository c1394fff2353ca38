"""The direct single-hot scatter with the duplicates of a tile of 64 lookups combined: parity with the
oracle on small-integer gradients (exact in any order), over rows of one to eight lane groups, tables of
one, two and many tokens (runs within a group, across groups, over the whole tile), batches that end
inside a tile and inside a group, blocks larger than embeddings and the sign hash."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sign", [0, 1])
@pytest.mark.parametrize("d,Z", [(8, 8), (16, 4), (20, 5), (32, 1), (16, 64), (48, 16), (96, 32), (128, 32)])
def test_tiles_match_the_oracle(d, Z, sign):
    m = 50_021
    h, H = P.both_hashes(d + Z, m, d, Z, sign)
    opt = robe.options(backward_route=robe.ROUTE_DIRECT, tile_combine=2)
    rng = np.random.default_rng(d)
    for B, F in ((1, 1), (63, 1), (64, 2), (131, 3), (17, 5)):
        ids = np.stack([rng.integers(0, (1, 2, 40, 10**6, 5)[f], size=B) for f in range(F)], axis=1).astype(np.int64)
        G = rng.integers(-3, 4, size=(B, F, d)).astype(np.float32)
        ref, _ = oracle.backward(H, G, ids, None, B, F)
        ga = torch.zeros(m, dtype=torch.float32, device="cuda:0")
        robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), None, B, F, ga, options=opt)
        assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref), (B, F)
