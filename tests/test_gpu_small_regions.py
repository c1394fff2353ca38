"""The reduce kernel for regions with few records (one wavefront per region, no copy of the region in
LDS): parity with the oracle, slot by slot.  Small-integer gradients make every float32 sum exact, so the
comparison is bit for bit; cases cover array lengths that are no multiple of a vector or a granule,
blocks that wrap to slot 0 or pass through a short last region, overlapping blocks, blocks from one
float to longer than 64 slots, a token repeated until its region holds more records than the kernel
takes, the sign hash, tables of mixed dimensions and all three rules."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_mixed_dims as MD
from tests import test_gpu_parity as P
from tests.test_gpu_gather import tokens_near_the_array_end

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# (m, d, Z, sign, region_shift) of 2304 tokens and, where C = 1, 12000 copies of one more: few enough
# records for the kernel (see problem)
CASES = [
    (12_000_003, 32, 32, 0, 0),        # odd tail, C = 1: the repeated token overfills its region
    (12_000_001, 32, 32, 1, 10),       # the sign, small regions
    (2**21 + 5, 8, 64, 0, 0),          # blocks larger than embeddings
    (10_000_002, 128, 32, 0, 13),
    (3 * 2**22 + 7, 16, 16, 1, 0),     # the array ends in a region shorter than a block
    (58_000_003, 128, 1, 0, 14),       # one float per block
    (20_000_001, 96, 3, 1, 0),         # odd blocks, shorter than a vector
    (10_000_019, 200, 100, 0, 15),     # longer than 64 slots
    (2**26 + 3, 128, 32, 0, 0),        # taken by default
]


def problem(m, d, Z, sign):
    h, H = P.both_hashes(m + d, m, d, Z, sign)
    rng = np.random.default_rng(m % 7919)
    F, B = 3, 768
    copies = 12000 if d == Z else 0
    C, z = max(1, d // Z), min(d, Z)            # the rule that picks the kernel
    weight = max(1 if z <= 32 else 1 + z // 64, 3 if C == 1 and m < 150_000_000 else 1)
    assert (B * F + copies) * C * weight * 8192 <= m * min(78, 30 + m // 4_000_000)
    ids = rng.integers(0, 10**6, size=B * F + copies, dtype=np.int64)
    for k, (x, f) in enumerate(tokens_near_the_array_end(H, F, 6, rng)):
        ids[3 * k + f] = x
    ids[60:120:3] = ids[60]                     # a repeated token of table 0
    offsets = np.arange(B * F + 1, dtype=np.int64)
    if copies:                                  # the first bag takes the copies as well
        ids[B * F:] = ids[0]
        ids = np.concatenate([ids[B * F:], ids[:B * F]])
        offsets[1:] += copies
    G = rng.integers(-3, 4, size=(B, F, d)).astype(np.float32)
    return h, H, ids, offsets, B, F, G


@pytest.mark.parametrize("m,d,Z,sign,shift", CASES)
def test_small_regions_match_the_oracle(m, d, Z, sign, shift):
    print(m, d, Z, sign, shift, flush=True)
    h, H, ids, off, B, F, G = problem(m, d, Z, sign)
    ref, _ = oracle.backward(H, G, ids, off, B, F, threads=8)
    opt = robe.options(backward_route=robe.ROUTE_REGIONS, region_records=1, region_shift=shift)
    start = np.full(m, 2.0, dtype=np.float32)
    ga = torch.from_numpy(start).to(DEV)
    robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, F, ga, options=opt)
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref + 2.0)
    # an unaligned gradient array
    odd = torch.from_numpy(np.concatenate([start[:1], start])).to(DEV)[1:]
    robe.robe_backward(h, P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, F, odd, options=opt)
    assert np.array_equal(odd.cpu().numpy(), ga.cpu().numpy())
    fused = robe.options(fused_route=robe.ROUTE_REGIONS, region_records=1, region_shift=shift)
    P._check_fused(h, H, G, ids, off, B, F, m, options=fused)
    # SGD at a rate of one: the array minus an exact sum of integers, rounded once
    M = np.random.default_rng(1).standard_normal(m).astype(np.float32)
    Md = torch.from_numpy(M.copy()).to(DEV)
    robe.robe_backward_sgd(h, P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, F, Md, 1.0, options=fused)
    assert np.array_equal(Md.cpu().numpy(), M - ref.astype(np.float32))
    # real-valued gradients: the same bits twice
    Gr = torch.randn(B, F, d, device=DEV)
    repro = robe.options(reproducible=1, region_records=1, region_shift=shift)
    got = []
    for _ in range(2):
        g = torch.zeros(m, device=DEV)
        robe.robe_backward(h, Gr, P.to_dev(ids), P.to_dev(off), B, F, g, options=repro)
        got.append(g.cpu().numpy().view(np.int32))
    assert np.array_equal(got[0], got[1])


def test_small_regions_mixed_dimensions():
    m, Z, dims = 8_000_009, 16, [16, 64, 32, 48, 16]
    h, H = MD.hashes(5, m, Z, 1, max(dims))
    rng = np.random.default_rng(3)
    B, F = 700, len(dims)
    ids = rng.integers(0, 5000, size=(B, F), dtype=np.int64)
    G = rng.integers(-3, 4, size=(B, sum(dims))).astype(np.float32)
    ref, _ = oracle.backward_mixed(H, dims, G, ids, None, B)
    ga = torch.zeros(m, dtype=torch.float32, device=DEV)
    robe.robe_backward_mixed(h, dims, MD.dev(G), MD.dev(ids), None, B, ga,
                             options=robe.options(backward_route=robe.ROUTE_REGIONS, region_records=1))
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref)
    MD._fused_mixed_check(h, H, dims, G, ids, None, B, m, robe.options(fused_route=robe.ROUTE_REGIONS))


@pytest.mark.parametrize("m,d,Z,sign,shift", [(10_000_002, 128, 32, 0, 0), (12_000_001, 32, 32, 1, 10), (2**26 + 3, 128, 32, 1, 0)])
def test_reproducible_bits_do_not_depend_on_the_buffers_alignment(m, d, Z, sign, shift):
    h, H, ids, off, B, F, _ = problem(m, d, Z, sign)
    G = torch.randn(B, F, d, device=DEV, generator=torch.Generator(DEV).manual_seed(1))
    opt = robe.options(reproducible=1, region_records=1, region_shift=shift)
    start = torch.randn(m, device=DEV, generator=torch.Generator(DEV).manual_seed(2))
    got = []
    for pad in (0, 1, 2, 3):
        bufs = [torch.empty(m + pad, device=DEV)[pad:] for _ in range(3)]
        bufs[0].zero_()
        robe.robe_backward(h, G, P.to_dev(ids), P.to_dev(off), B, F, bufs[0], options=opt)
        bufs[1].copy_(start)
        bufs[2].fill_(0.5)
        robe.robe_backward_adagrad(h, G, P.to_dev(ids), P.to_dev(off), B, F, bufs[1], bufs[2], 0.1, 1e-8, options=opt)
        got.append([b.clone().view(torch.int32) for b in bufs])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
