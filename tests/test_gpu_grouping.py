"""The grouping sort (one pass by the top key bits, then every tile by the next inside LDS) under the combine
kernels: parity with the oracle on small-integer gradients, exact in any order, over token counts around the
tiles, around the change from 8 to 10 bits (2^18, 450 000 in bags), around the last that it takes (2^21), single-hot lookups and bags,
signs, blocks larger than embeddings, one token for all lookups.  Reproducible calls repeat their bits; the
workspace is the plain sort's, so that the built-in one takes what it took with that.  Which sort a call takes is
seen in its launches."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P
from tests.launches import kernels

pytestmark = pytest.mark.gpu

M = 300_007


def _problem(n, F, d, bags, kind):
    rng = np.random.default_rng(n + F)
    B = -(-n // F)
    ids = rng.zipf(1.2, size=B * F if not bags else n).astype(np.int64) % 10**7 if kind == "zipf" else np.full(B * F if not bags else n, 7, np.int64)
    off = None
    if bags:
        cut = np.sort(rng.integers(0, n + 1, size=B * F - 1))
        off = np.concatenate([[0], cut, [n]]).astype(np.int64)
    return B, ids, off, rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)


@pytest.mark.parametrize("n,F,kind", [(1, 1, "zipf"), (4095, 3, "zipf"), (4097, 1, "zipf"), (70_001, 26, "zipf"), (2**18, 2, "zipf"), (2**18 + 1, 1, "zipf"),
                                      (300_000, 7, "same"), (450_001, 3, "zipf"), (2**21, 8, "zipf"), (2**21 + 8, 8, "zipf")])
@pytest.mark.parametrize("d,Z,sign", [(16, 16, 0), (8, 2, 1), (8, 32, 1)])
def test_grouped_tokens_match_the_oracle(n, F, kind, d, Z, sign):
    h, H = P.both_hashes(n + Z, M, d, Z, sign)
    opt = robe.options(backward_route=robe.ROUTE_COMBINE)
    for bags in (False, True):
        B, ids, off, G = _problem(n, F, d, bags, kind)
        ref, _ = oracle.backward(H, G, ids if bags else ids.reshape(B, F), off, B, F)
        ga = torch.zeros(M, dtype=torch.float32, device="cuda:0")
        robe.robe_backward(h, P.to_dev(G), P.to_dev(ids if bags else ids.reshape(B, F)), P.to_dev(off) if bags else None, B, F, ga, options=opt)
        assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref), bags


@pytest.mark.parametrize("n", [200_000, 700_000])
def test_reproducible_calls_repeat_their_bits(n):
    h, H = P.both_hashes(n, 5_000_011, 64, 16, 1)
    opt = robe.options(reproducible=1)
    B, ids, _, G = _problem(n, 10, 64, False, "zipf")
    G = (G * np.float32(0.37)).astype(np.float32)
    runs = []
    for _ in range(3):
        ga = torch.zeros(5_000_011, dtype=torch.float32, device="cuda:0")
        robe.robe_backward(h, P.to_dev(G), P.to_dev(ids.reshape(B, 10)), None, B, 10, ga, options=opt)
        runs.append(ga.cpu().numpy())
    assert np.array_equal(runs[0].view(np.int32), runs[1].view(np.int32)) and np.array_equal(runs[0].view(np.int32), runs[2].view(np.int32))
    ref, S = oracle.backward(H, G, ids.reshape(B, 10), None, B, 10)
    assert np.all(np.abs(runs[0] - ref) <= 1e-5 * S + 1e-30)


def test_the_built_in_workspace_holds_two_million_tokens():
    n, d = 2_000_000, 32
    h, H = P.both_hashes(3, M, d, 16, 0)
    assert robe.robe_workspace_bytes(h, n, 1, n, robe.options(backward_route=robe.ROUTE_COMBINE)) <= 2**25
    B, ids, _, G = _problem(n, 1, d, False, "zipf")
    ref, _ = oracle.backward(H, G, ids.reshape(B, 1), None, B, 1)
    ga = torch.zeros(M, dtype=torch.float32, device="cuda:0")
    args = (h, P.to_dev(G), P.to_dev(ids.reshape(B, 1)), None, B, 1, ga)
    robe.robe_backward_noalloc(*args)
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref)
    assert kernels(lambda: robe.robe_backward_noalloc(*args)) == 5


# count, scatter, local, combine; bags: their tokens' keys or rows before; above 2^18 tokens: offsets
@pytest.mark.parametrize("n,bags,sign,launches", [(2**18, False, 0, 4), (2**18, True, 1, 5), (2**18 + 2, False, 1, 5), (2**18 + 2, True, 0, 6),
                                                  (450_000, True, 0, 6), (450_002, True, 0, 6), (450_002, True, 1, 6), (2**21, True, 1, 6)])
def test_the_plain_sorts_workspace_is_enough(n, bags, sign, launches):
    """... to the byte, and nothing behind it is written."""
    F, d = 2, 16
    h, H = P.both_hashes(n, M, d, 16, sign)
    B, ids, off, G = _problem(n, F, d, bags, "zipf")
    use = ids if bags else ids.reshape(B, F)
    ref, _ = oracle.backward(H, G, use, off, B, F)
    opt = robe.options(backward_route=robe.ROUTE_COMBINE)
    size = robe.robe_workspace_bytes(h, B, F, n, robe.options(backward_route=robe.ROUTE_COMBINE, key_bits=24))
    ws = torch.full((size + 512,), 255, dtype=torch.uint8, device="cuda:0")
    ga = torch.zeros(M, dtype=torch.float32, device="cuda:0")
    args = (h, P.to_dev(G), P.to_dev(use), P.to_dev(off) if bags else None, B, F, ga)
    robe.robe_backward(*args, workspace=ws[:size], options=opt)
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref)
    assert (ws[size:] == 255).all()
    assert kernels(lambda: robe.robe_backward(*args, workspace=ws[:size], options=opt)) == launches
