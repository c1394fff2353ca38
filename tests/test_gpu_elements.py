"""The backward of small blocks (Z <= 2 on large batches: runs by the place they write): parity with the
oracle slot by slot on small-integer gradients, whose float32 sums are exact in any order.  Cases cover
row widths that are and are not powers of two, the widest and the narrowest rows of the route, blocks
larger than embeddings, array lengths at both ends of its range and past it, tokens repeated thousands
of times, bags, the sign hash, unaligned arrays and the fused rules."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# (m, d, Z, sign, bags); 2^23 gradient elements or a few more each
CASES = [
    (1_000_003, 128, 1, 0, False),
    (25_000_001, 128, 1, 1, True),
    (3600 * 2**14, 128, 2, 0, False),      # the most regions the route takes, and one slot more
    (3600 * 2**14 + 1, 128, 2, 0, False),
    (5, 100, 1, 0, False),                 # (too small an array for the route: sorted atomics)
    (700_001, 100, 2, 1, False),           # lanes past the row stay idle
    (700_002, 512, 1, 0, True),            # the widest rows
    (300_007, 16, 2, 1, False),            # (the same)
    (300_006, 2, 8, 0, False),             # (the same, blocks larger than embeddings)
]


@pytest.mark.parametrize("m,d,Z,sign,bags", CASES)
def test_small_blocks_match_the_oracle(m, d, Z, sign, bags):
    print(m, d, Z, sign, bags, flush=True)
    h, H = P.both_hashes(m + d, m, d, Z, sign)
    rng = np.random.default_rng(m % 1009 + d)
    F = 3
    n = -(-(2**23 + 1000) // (d * F)) * F
    ids = rng.integers(0, 10**6, size=n, dtype=np.int64)
    ids[rng.random(n) < 0.3] = 11
    if bags:
        B = n // (4 * F)
        off = np.sort(rng.integers(0, n + 1, size=B * F + 1))
        off[0], off[-1] = 0, n
    else:
        B, off = n // F, None
    G = rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)
    dG, dids, doff = P.to_dev(G), P.to_dev(ids), P.to_dev(off)
    ref, _ = oracle.backward(H, G, ids, off, B, F, threads=8)
    assert np.abs(ref).max() < 2**24
    buf = torch.full((m + 1,), 3.0, device=DEV)
    for shift in (0, 1):                              # an unaligned gradient array
        ga = buf[shift:m + shift]
        ga.fill_(3.0)
        robe.robe_backward(h, dG, dids, doff, B, F, ga)
        assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref + 3.0)
    P._check_fused(h, H, G, ids, off, B, F, m)
    M = np.random.default_rng(1).standard_normal(m).astype(np.float32)
    Md = torch.from_numpy(M.copy()).to(DEV)
    robe.robe_backward_sgd(h, dG, dids, doff, B, F, Md, 1.0)
    assert np.array_equal(Md.cpu().numpy(), M - ref.astype(np.float32))


# (m, d, Z, sign, bags, elements): the smallest array with a last region of five slots, the narrowest rows, and rows of more
# runs than there is room for (2^26 floats on arrays this small): the rest is added with atomics
MORE = [
    (31 * 2**14 + 5, 100, 1, 0, False, 2**23),
    (31 * 2**14 + 5, 128, 1, 0, False, 2**26 + 2**22),
    (600_007, 128, 2, 1, True, 2**26 + 2**22),
    (1_000_003, 4, 1, 0, False, 2**23),
    (1_000_003, 8, 2, 1, True, 2**23),
    (1_000_003, 16, 2, 1, False, 2**23),
]


@pytest.mark.parametrize("m,d,Z,sign,bags,elems", MORE)
def test_small_blocks_at_the_edges_of_their_room(m, d, Z, sign, bags, elems):
    h, H = P.both_hashes(m + d, m, d, Z, sign)
    rng = np.random.default_rng(m % 1009 + d)
    F = 3
    n = -(-(elems + 1000) // (d * F)) * F
    ids = rng.permutation(n).astype(np.int64)               # all distinct: a run for every token
    ids[:5000] = 7
    B, off = n // F, None
    if bags:
        B = n // (4 * F)
        off = np.sort(rng.integers(0, n + 1, size=B * F + 1))
        off[0], off[-1] = 0, n
    need = robe.robe_workspace_bytes(h, B, F, n)
    assert need > robe.robe_workspace_bytes(h, B, F, n, robe.options(backward_route=robe.ROUTE_COMBINE))
    # (without room for all the fused step goes through a gradient array)
    assert (robe.robe_fused_workspace_bytes(h, B, F, n) >= need + 4 * m) == (n * d - 5000 * d > 2**26)
    G = rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)
    dG, dids, doff = P.to_dev(G), P.to_dev(ids), P.to_dev(off)
    ref, _ = oracle.backward(H, G, ids, off, B, F, threads=8)
    assert np.abs(ref).max() < 2**24
    ga = torch.full((m,), 3.0, device=DEV)
    robe.robe_backward(h, dG, dids, doff, B, F, ga)
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref + 3.0)
    P._check_fused(h, H, G, ids, off, B, F, m)
    M = np.random.default_rng(1).standard_normal(m).astype(np.float32)
    Md = torch.from_numpy(M.copy()).to(DEV)
    robe.robe_backward_sgd(h, dG, dids, doff, B, F, Md, 1.0)
    assert np.array_equal(Md.cpu().numpy(), M - ref.astype(np.float32))
