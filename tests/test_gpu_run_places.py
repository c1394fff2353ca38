"""The backward of small blocks, whose runs are moved by the place they write: parity with the oracle slot by slot on small-integer
gradients (exact in any order).  Arrays of a power of two slots and around it, a last region of one slot, more runs than
there is room for (the rest goes by atomics), and one token so frequent that its runs crowd a window."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,Z,sign,elems,ids_of", [(2**20, 128, 1, 1, 2**23, "few"), (2**20 + 1, 512, 2, 0, 2**23, "few"), (2**24 - 1, 100, 2, 1, 2**24, "many"),
                                                     (600_007, 128, 2, 1, 2**26 + 2**22, "distinct"), (2**21 + 5, 128, 1, 0, 2**26 + 2**20, "distinct"),
                                                     (2**23, 16, 1, 0, 2**23, "one")])
def test_every_slot_gets_its_sum(m, d, Z, sign, elems, ids_of):
    h, H = P.both_hashes(m + d, m, d, Z, sign)
    rng = np.random.default_rng(m % 1009 + d)
    F = 4
    B = -(-elems // (d * F)) + 1
    n = B * F
    ids = {"few": lambda: rng.integers(0, 3000, size=n), "many": lambda: rng.integers(0, n, size=n), "distinct": lambda: rng.permutation(n),
           "one": lambda: np.zeros(n)}[ids_of]().astype(np.int64).reshape(B, F)
    G = rng.integers(-1, 2, size=(B, F, d)).astype(np.float32)
    ref, S = oracle.backward(H, G, ids, None, B, F, threads=8)
    assert S.max() < 2**24
    ga = torch.full((m,), 3.0, device="cuda:0")
    robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), None, B, F, ga)
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref + 3.0)
