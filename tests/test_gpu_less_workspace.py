"""Calls that ask for no route and bring less workspace than the query names: what a direct scatter (or,
for large scatters of small blocks, the sort alone) can do without is done without; the rest is refused.
Small-integer gradients make every float32 sum exact, so results are compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
M = 300_007
BYTES = torch.uint8


def problem(m, d, Z, n, bags, seed=1):
    h, H = P.both_hashes(seed, m, d, Z, 0)
    rng = np.random.default_rng(n + d)
    F = 2
    ids = rng.integers(0, 5000, size=n, dtype=np.int64)
    B, off = n // F, None
    if bags:
        B = n // (4 * F)
        off = np.sort(rng.integers(0, n + 1, size=B * F + 1))
        off[0], off[-1] = 0, n
    G = rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)
    return h, H, ids, off, B, F, G


def workspaces(size):
    """None at all, too small a one, and (if it is read) one off its alignment."""
    buf = torch.empty(size + 512, dtype=BYTES, device=DEV)
    return [buf[:0], buf[:256], buf[4:4 + size]]


@pytest.mark.parametrize("d,Z,n,bags", [(16, 4, 120_000, True), (128, 32, 200_000, False), (128, 1, 2**17, False), (128, 2, 2**17, True)])
def test_backward_scatters_directly(d, Z, n, bags):
    h, H, ids, off, B, F, G = problem(M, d, Z, n, bags)
    need = robe.robe_workspace_bytes(h, B, F, n)
    assert need > 0 and n * d < 2**25
    ref, _ = oracle.backward(H, G, ids, off, B, F, threads=8)
    for ws in workspaces(need):
        ga = torch.zeros(M, device=DEV)
        robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, F, ga, workspace=ws)
        assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref)
        for asked in ({"backward_route": robe.ROUTE_COMBINE}, {"reproducible": 1}):      # asked for by name, it is refused
            with pytest.raises(robe.RobeError, match="workspace"):
                robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, F, ga, workspace=ws, options=robe.options(**asked))


def test_large_scatters_of_small_blocks_sort_with_atomics():
    n, d = 2**18 + 2, 128
    h, H, ids, off, B, F, G = problem(1_000_003, d, 1, n, False)
    combine = robe.robe_workspace_bytes(h, B, F, n, robe.options(backward_route=robe.ROUTE_COMBINE))
    ref, _ = oracle.backward(H, G, ids, off, B, F, threads=8)
    ga = torch.zeros(h.m, device=DEV)
    robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), None, B, F, ga, workspace=torch.empty(combine, dtype=BYTES, device=DEV))
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref)
    with pytest.raises(robe.RobeError, match="workspace"):
        robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), None, B, F, ga, workspace=torch.empty(combine - 256, dtype=BYTES, device=DEV))


def test_mixed_dimensions_scatter_directly():
    m, dims, B = M, [16, 64, 32, 64], 12_000
    h, H = P.both_hashes(3, m, 64, 8, 0)
    rng = np.random.default_rng(0)
    ids = rng.integers(0, 5000, size=(B, 4), dtype=np.int64)
    ids = np.concatenate([ids] * 4)
    B *= 4
    G = rng.integers(-2, 3, size=(B, sum(dims))).astype(np.float32)
    ref, _ = oracle.backward_mixed(H, dims, G, ids, None, B)
    need = robe.robe_mixed_workspace_bytes(h, dims, B, ids.size)
    off = np.arange(ids.size + 1)
    assert need > 0
    for ws in workspaces(need):
        ga = torch.zeros(m, device=DEV)
        robe.robe_backward_mixed(h, dims, P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, ga, workspace=ws)
        assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("m,d,Z,n,bags", [(21_000_003, 128, 32, 140_000, False), (1_000_003, 32, 8, 80_000, True), (1_000_003, 128, 1, 2**17, False)])
def test_the_fused_step_takes_two_steps_in_a_gradient_array(m, d, Z, n, bags):
    h, H, ids, off, B, F, G = problem(m, d, Z, n, bags)
    assert n * d < 2**25
    array = torch.randn(m, device=DEV)
    args = (P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, F)
    got = []
    for ws in (None, torch.empty(-(-4 * m // 256) * 256, dtype=BYTES, device=DEV)):
        a, s = array.clone(), torch.ones(m, device=DEV)
        robe.robe_backward_adagrad(h, *args, a, s, 0.1, 1e-8, workspace=ws)
        b = array.clone()
        robe.robe_backward_sgd(h, *args, b, 0.5, workspace=ws)
        got.append([a, s, b])
    for x, y in zip(*got):
        assert torch.equal(x, y)
    with pytest.raises(robe.RobeError, match="workspace"):
        robe.robe_backward_sgd(h, *args, array, 0.5, workspace=torch.empty(256, dtype=BYTES, device=DEV))
