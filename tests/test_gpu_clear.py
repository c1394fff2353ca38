"""The fused step in two steps clears its gradient array beside the first kernel of the sort: parity with the oracle,
exact on small integers, from a workspace full of NaN, for keys hashed in the sort and keys written before it, both
sorts, arrays that are no whole number of vectors or shorter than a workgroup's share, mixed dimensions, and small
blocks, the rows of whose runs do not all fit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu


def _nan(n):
    return torch.full((n,), 255, dtype=torch.uint8, device="cuda:0")


@pytest.mark.parametrize("m", [67, 8191, 300_007])
@pytest.mark.parametrize("key_bits", [0, 24])
@pytest.mark.parametrize("bags", [False, True])
def test_two_steps_clear_their_gradient(m, key_bits, bags):
    d, Z, F, B = 64, 16, 3, 1501
    h, H = P.both_hashes(m, m, d, Z, 1)
    rng = np.random.default_rng(m)
    ids = rng.integers(0, 50, size=B * F).astype(np.int64)
    off = np.concatenate([[0], np.sort(rng.integers(0, B * F + 1, size=B * F - 1)), [B * F]]).astype(np.int64) if bags else None
    use = ids if bags else ids.reshape(B, F)
    G = rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)
    A = rng.integers(-50, 50, size=m).astype(np.float32)
    opt = robe.options(backward_route=robe.ROUTE_COMBINE, fused_route=robe.ROUTE_TWO_STEP, key_bits=key_bits)
    ref, _ = oracle.backward(H, G, use, off, B, F)
    array = P.to_dev(A)
    need = robe.robe_fused_workspace_bytes(h, B, F, B * F, opt)
    robe.robe_backward_sgd(h, P.to_dev(G), P.to_dev(use), P.to_dev(off) if bags else None, B, F, array, 1.0, workspace=_nan(need), options=opt)
    assert np.array_equal(array.cpu().numpy().astype(np.float64), A - ref)


def test_two_steps_of_mixed_dimensions_clear_their_gradient():
    m, dims, Z, B = 300_007, (16, 64, 32), 16, 1501
    h, H = P.both_hashes(m, m, max(dims), Z, 0)
    rng = np.random.default_rng(3)
    ids = rng.integers(0, 50, size=(B, len(dims))).astype(np.int64)
    G = rng.integers(-2, 3, size=(B, sum(dims))).astype(np.float32)
    ref, _ = oracle.backward_mixed(H, dims, G, ids, None, B)
    opt = robe.options(backward_route=robe.ROUTE_COMBINE, fused_route=robe.ROUTE_TWO_STEP)
    array, state = torch.zeros(m, device="cuda:0"), torch.zeros(m, device="cuda:0")
    need = robe.robe_fused_mixed_workspace_bytes(h, list(dims), B, ids.size, opt)
    robe.robe_backward_adagrad_mixed(h, list(dims), P.to_dev(G), P.to_dev(ids), None, B, array, state, 0.01, 1e-8, workspace=_nan(need), options=opt)
    assert np.array_equal(state.cpu().numpy(), np.float32(ref) * np.float32(ref))       # (integers below 2^12: squares are exact)


@pytest.mark.parametrize("n,d,bags", [(540_000, 128, False), (540_000, 128, True), (2**21 + 2**17, 32, False)])
def test_runs_without_room_clear_their_gradient(n, d, bags):
    """More than 2^26 elements of blocks of one float on a small array, nearly every id another one: the runs whose rows find no
    room are added with atomics, so the step goes through a gradient array."""
    m, F = 600_011, 2
    h, H = P.both_hashes(n, m, d, 1, 0)
    rng = np.random.default_rng(n)
    B = n // F
    ids = rng.integers(0, 10**9, size=n).astype(np.int64)
    off = np.concatenate([[0], np.sort(rng.integers(0, n + 1, size=n - 1)), [n]]).astype(np.int64) if bags else None
    use = ids if bags else ids.reshape(B, F)
    G = rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)
    need = robe.robe_fused_workspace_bytes(h, B, F, n)
    assert need > robe.robe_fused_workspace_bytes(h, B, F, n, robe.options(backward_route=robe.ROUTE_COMBINE))      # the route of small blocks
    assert need >= robe.robe_workspace_bytes(h, B, F, n) + 4 * m and len(np.unique(ids)) * d > 2**26 + 2**20
    ref, _ = oracle.backward(H, G, use, off, B, F, threads=8)
    array = torch.zeros(m, device="cuda:0")
    robe.robe_backward_sgd(h, P.to_dev(G), P.to_dev(use), P.to_dev(off) if bags else None, B, F, array, 1.0, workspace=_nan(need))
    assert np.array_equal(array.cpu().numpy().astype(np.float64), -ref)
