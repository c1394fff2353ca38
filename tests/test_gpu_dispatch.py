"""The size rules that pick a backward route by default: results on both sides of each line agree with
the oracle bit for bit (small-integer gradients), the workspace query covers both kinds of input, and
the allocation-free call still takes every problem that it can scatter directly."""
import numpy as np
import pytest
import torch

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

DEV = "cuda:0"


# (d, Z, tokens) around the lines for bags (65536 tokens, 650 thousand of requests and tokens) and for
# single-hot lookups (1.2 million requests and a thousand per float of a row, a million more than the tokens cost)
SIZES = [(16, 4, 65_535), (16, 4, 65_536), (16, 4, 113_043), (16, 4, 113_044), (128, 32, 113_020), (128, 32, 113_030), (32, 128, 60_000),
         (100, 10, 65_535), (100, 10, 83_199), (100, 10, 83_200), (16, 16, 900_000)]
MORE_SIZES = [(16, 16, 2**21 - 1), (16, 16, 2**21), (8, 8, 2**22 - 1), (8, 8, 2**22),
              (16, 1, 90_000), (16, 1, 95_000), (16, 1, 64_000), (4, 1, 125_000), (4, 1, 135_000), (6, 2, 900_000), (12, 4, 140_000), (12, 4, 145_000), (3, 3, 2_000_000), (3, 3, 12_000_000)]        # around 2^25 gradient elements


def pays(d, Z, n, bags):
    Z = min(d, Z)
    requests = n * (d // Z) * (Z + 15) // 16
    lanes = {3: 1, 4: 4, 6: 2, 8: 8, 12: 4}.get(d, 16)
    return (n * d >= 2**25 or (bags and lanes >= 4 and n >= 65_536 and requests + n >= 650_000) or
            (lanes >= 8 and requests >= 1_200_000 + 1000 * d + (300_000 if Z <= 2 else 0) and requests >= 1_000_000 + (2 * n if d < 16 else n + n // 4)))


@pytest.mark.parametrize("d,Z,n", SIZES + MORE_SIZES)
def test_the_workspace_query_covers_single_hot_and_bags(d, Z, n):
    h = robe.robe_init_hash(1, 1_000_003, d, Z, 1)
    single = robe.robe_workspace_bytes(h, n, 1, n)
    forced = robe.robe_workspace_bytes(h, n, 1, n, robe.options(backward_route=robe.ROUTE_COMBINE))
    assert single in (0, forced)
    assert (single > 0) == (pays(d, Z, n, True) or pays(d, Z, n, False))


@pytest.mark.parametrize("m", [1_000_003, 20_971_519, 20_971_520, 25_000_000, 2**25, 2**25 + 1, 2**26, 250_000_000])
@pytest.mark.parametrize("d,Z,sign", [(128, 32, 0), (128, 32, 1), (128, 1, 0), (64, 16, 1), (100, 10, 0), (16, 64, 0)])
def test_the_fused_query_covers_single_hot_and_bags(m, d, Z, sign):
    # a call without a workspace says how much it needs and launches nothing
    import ctypes
    h = robe.robe_init_hash(1, m, d, Z, sign)
    L, fake = robe.lib(), ctypes.c_void_p(4096)
    for n in (1, 49_999, 50_000, 65_535, 65_536, 78_000, 113_000, 114_000, 1 << 18, 1 << 20, (1 << 20) + 1, 1_700_000, 9_000_000):
        query = robe.robe_fused_workspace_bytes(h, n, 1, n)
        for offsets in (None, fake):
            rc = L.robe_backward_adagrad(ctypes.byref(h), fake, fake, offsets, n, n, 1, fake, fake, 0.1, 1e-8, None, 0, None, None)
            text = L.robe_last_error().decode()
            assert rc == robe.ROBE_EINVAL and text.startswith("workspace of"), text
            assert int(text.split()[2]) <= query, (n, offsets)


@pytest.mark.gpu
@pytest.mark.parametrize("bags", [False, True])
@pytest.mark.parametrize("d,Z,n", SIZES)
def test_both_sides_of_the_size_rule_match_the_oracle(d, Z, n, bags):
    m = 300_007
    h, H = P.both_hashes(n + d, m, d, Z, 1)
    rng = np.random.default_rng(n)
    ids = rng.integers(0, 2000, size=n, dtype=np.int64)
    ids[rng.random(n) < 0.3] = 7
    if bags:
        B, F = n // 6, 2
        off = np.sort(rng.integers(0, n + 1, size=B * F + 1))
        off[0], off[-1] = 0, n
    else:
        B, F, off = n, 1, None
    G = rng.integers(-2, 3, size=(B, F, d)).astype(np.float32)
    ref, _ = oracle.backward(H, G, ids, off, B, F, threads=8)
    for call in (robe.robe_backward, robe.robe_backward_noalloc):
        ga = torch.zeros(m, dtype=torch.float32, device=DEV)
        call(h, P.to_dev(G), P.to_dev(ids), P.to_dev(off), B, F, ga)
        assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref), call


@pytest.mark.gpu
def test_noalloc_takes_many_narrow_tokens():
    # 2.2 million tokens need more than the built-in workspace to sort, but go directly
    m, d, Z, n = 500_009, 4, 2, 2_200_000
    h, H = P.both_hashes(3, m, d, Z, 0)
    rng = np.random.default_rng(0)
    ids = rng.integers(0, 10**6, size=(n // 4, 4), dtype=np.int64)
    G = rng.integers(-2, 3, size=(n // 4, 4, d)).astype(np.float32)
    assert robe.robe_workspace_bytes(h, n // 4, 4, n) > robe.lib().robe_noalloc_max_workspace_bytes()
    ga = torch.zeros(m, dtype=torch.float32, device=DEV)
    robe.robe_backward_noalloc(h, P.to_dev(G), P.to_dev(ids), None, n // 4, 4, ga)
    ref, _ = oracle.backward(H, G, ids, None, n // 4, 4, threads=8)
    assert np.array_equal(ga.cpu().numpy().astype(np.float64), ref)
    with pytest.raises(robe.RobeError):      # asked for by name, the sorted route is refused as before
        robe.robe_backward_noalloc(h, P.to_dev(G), P.to_dev(ids), None, n // 4, 4, ga,
                                   options=robe.options(backward_route=robe.ROUTE_COMBINE))


@pytest.mark.gpu
@pytest.mark.parametrize("d,Z,n,bags,sorts", [(16, 4, 70_000, True, False), (128, 32, 200_000, False, False), (4, 1, 2**23 - 1, False, False),
                                              (128, 32, 2**18 - 1, True, False), (128, 32, 2**18, False, True), (128, 1, 2**18, True, True)])
def test_noalloc_sorts_from_two_to_the_25_elements_on(d, Z, n, bags, sorts):
    # the built-in workspace is shared by all streams: what scatters directly leaves it alone
    m = 500_009
    h = robe.robe_init_hash(1, m, d, Z, 0)
    begin, end, origin = (torch.cuda.Event(enable_timing=True) for _ in range(3))
    for e in (origin, begin, end):
        e.record()
    torch.cuda.synchronize()
    first = origin.elapsed_time(begin)
    opt = robe.options(probe_kernel=robe.PROBE_SORT, probe_begin=begin.cuda_event, probe_end=end.cuda_event)
    off = torch.arange(n + 1, device=DEV) if bags else None
    ga = torch.zeros(m, device=DEV)
    robe.robe_backward_noalloc(h, torch.ones(n, 1, d, device=DEV), torch.arange(n, device=DEV), off, n, 1, ga, options=opt)
    torch.cuda.synchronize()
    assert (origin.elapsed_time(begin) != first) == sorts            # recorded anew, just before the sort
    assert float(ga.sum(dtype=torch.float64)) == n * d


@pytest.mark.gpu
@pytest.mark.parametrize("n", [4096, 64 * 4096 - 1, 64 * 4096, 64 * 4096 + 1])
def test_sort_on_both_sides_of_its_tile_limit(n):
    from tests import test_gpu_sort as S
    rng = np.random.default_rng(n)
    keys = rng.integers(0, 2**31, size=n, dtype=np.uint64).astype(np.uint32)
    keys[rng.random(n) < 0.3] = 77
    for lo, hi in ((15, 31), (0, 8), (7, 31)):
        S.check(keys, lo, hi)
