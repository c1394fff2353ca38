"""The bag forward that gives a lane group four bags at a time, which large launches of short bags take:
the same bits as the oracle's sums in token order within the float32 bound, and exactly the same as the
one-bag kernel's, over lane groups of several widths, empty bags, bags longer than a lane group, launches
that end inside a group's four, bounds out of order, blocks larger than embeddings, signs and bfloat16."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("d,Z,sign", [(100, 10, 1), (128, 32, 0), (32, 4, 1), (16, 64, 0), (200, 100, 0), (64, 16, 1), (48, 16, 0)])
def test_short_bags(d, Z, sign):
    m, F = 30_011, 3
    h, H = P.both_hashes(d, m, d, Z, sign)
    G = {100: 64, 128: 32, 32: 8, 16: 4, 200: 64, 64: 16, 48: 16}[d]     # (below 16 lanes: the one-bag kernel)
    rows = 8192 * 4 * (64 // G) + 5                  # a few past the least that the kernel takes
    B = -(-rows // F)
    rng = np.random.default_rng(d)
    sizes = rng.poisson(1.5, size=B * F)
    sizes[rng.integers(0, B * F, 20)] = 150
    sizes[-3:] = 0
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    assert n <= 4 * B * F
    ids = rng.integers(0, 10**6, size=n, dtype=np.int64)
    M = rng.standard_normal(m).astype(np.float32)
    A, I = P.to_dev(M), P.to_dev(ids)
    got = robe.robe_forward(h, A, I, P.to_dev(off), B, F).cpu().numpy().reshape(B * F, d)
    want = oracle.forward(H, M, ids, off, B, F).reshape(B * F, d)
    bound = 1e-5 * oracle.forward(H, np.full(m, np.abs(M).max(), np.float32), ids, off, B, F).reshape(B * F, d)
    assert np.all(np.abs(got - want) <= np.maximum(np.abs(bound), 1e-4))
    assert not got[sizes == 0].any()
    # the one-bag kernel, on as few of the bags as it keeps: the same bits
    few = 40
    part = robe.robe_forward(h, A, I[:off[few * F]], P.to_dev(off[:few * F + 1]), few, F).cpu().numpy().reshape(few * F, d)
    assert np.array_equal(part.view(np.int32), got[:few * F].view(np.int32))
    b16 = robe.robe_array_to_bf16(A)
    full = robe.robe_forward_bf16(h, b16, I, P.to_dev(off), B, F).cpu().numpy().reshape(B * F, d)
    part = robe.robe_forward_bf16(h, b16, I[:off[few * F]], P.to_dev(off[:few * F + 1]), few, F).cpu().numpy().reshape(few * F, d)
    assert np.array_equal(part.view(np.int32), full[:few * F].view(np.int32))
    # bounds out of order and out of range are clamped bag by bag
    bad = off.copy()
    bad[5], bad[9], bad[17], bad[30] = n + 50, -7, 2, n
    got = robe.robe_forward(h, A, I, P.to_dev(bad), B, F).cpu().numpy().reshape(B * F, d)
    for k in range(40):
        a = min(max(int(bad[k]), 0), n)
        b = min(max(int(bad[k + 1]), a), n)
        if b - a > 2000:
            continue
        one = robe.robe_forward(h, A, I[a:b], torch.tensor([0] * (k % F + 1) + [b - a] * (F - k % F), device=DEV), 1, F)
        assert np.array_equal(one.cpu().numpy().reshape(F, d)[k % F].view(np.int32), got[k].view(np.int32)), k
