"""What the calls accept, asked through the workspace queries: host arithmetic, no GPU."""
import math
import random

import pytest

import paper_2108_02191_amd as robe


def accepted(query, *args, **options):
    try:
        query(*args, robe.options(**options))
    except robe.RobeError as e:
        assert e.code == robe.ROBE_EINVAL
        return False
    return True


def _reproducible_shapes():
    yield 376_864_942, 512, 2, 0, 33_910, 11
    yield 25_000_000, 128, 1, 0, 700_000, 1
    yield 404_529_294, 512, 2, 0, 13_972, 27
    yield 133_675_900, 256, 8, 1, 259_352, 8
    yield 725_339_600, 96, 1, 0, 39_975, 13
    rng = random.Random(0)
    for _ in range(4000):
        d = rng.choice((8, 16, 32, 64, 96, 128, 256, 512))
        Z = rng.choice([z for z in (1, 2, 4, 8, 16, 32) if d % z == 0])
        m = int(math.exp(rng.uniform(math.log(10_000), math.log(2**30))))
        F = rng.randint(1, 40)
        yield m, d, Z, rng.randint(0, 1), int(math.exp(rng.uniform(math.log(50), math.log(4_000_000 / F)))), F


def test_the_default_sort_refuses_no_reproducible_call_that_a_longer_sort_takes():
    taken = 0
    for m, d, Z, sign, B, F in _reproducible_shapes():
        h = robe.robe_init_hash(1, m, d, Z, sign)
        for query in (robe.robe_workspace_bytes, robe.robe_fused_workspace_bytes):
            if accepted(query, h, B, F, B * F, reproducible=1, key_bits=24):
                taken += 1
                assert accepted(query, h, B, F, B * F, reproducible=1), (query.__name__, m, d, Z, sign, B, F)
    assert taken > 1000


def test_small_blocks_go_by_place_only_where_it_pays():
    """The runs moved by the place they write: arrays of 32 times 2^14 slots or more, rows of eight blocks (four if all is sure to fit), 2^16 tokens,
    2^23 gradient elements."""
    took = 0
    for m in (5, 16_384, 2**19 - 2**14, 2**19 - 2**14 + 1, 1_000_003, 25_000_000, 3600 * 2**14, 3600 * 2**14 + 1):
        for d in (2, 4, 8, 16, 100, 128, 512):
            for Z in (1, 2):
                h = robe.robe_init_hash(1, m, d, Z, 1)
                for n in (20_000, 65_535, 65_536, 400_000, 852_000, 2_200_000, 9_000_000):
                    need = robe.robe_workspace_bytes(h, n, 1, n)
                    if need in (0, robe.robe_workspace_bytes(h, n, 1, n, robe.options(backward_route=robe.ROUTE_COMBINE))):
                        continue
                    took += 1
                    assert 2**19 - 2**14 < m <= 3600 * 2**14 and n >= 65_536 and n * d >= 2**23, (m, d, Z, n)
                    assert d >= 8 * Z or (d >= 4 * Z and m <= 2**25 and n * d <= 2**25), (m, d, Z, n)
    assert took > 20


def test_small_blocks_take_a_bounded_workspace():
    """At most three floats per array slot (or 384 MiB) beside the sort's buffers, whatever the batch."""
    took = 0
    for m in (5, 16_384, 2**19 - 2**14, 2**19 - 2**14 + 1, 1_000_003, 25_000_000, 3600 * 2**14, 3600 * 2**14 + 1):
        for d in (2, 4, 8, 16, 100, 128, 512):
            for Z in (1, 2):
                h = robe.robe_init_hash(1, m, d, Z, 1) if Z <= m else None
                for n in (20_000, 65_535, 65_536, 400_000, 852_000, 3_500_000, 8_500_000, 30_000_000):
                    need = robe.robe_workspace_bytes(h, n, 1, n)
                    combine = robe.robe_workspace_bytes(h, n, 1, n, robe.options(backward_route=robe.ROUTE_COMBINE))
                    if need in (0, combine):
                        continue
                    took += 1
                    lists = combine + 9 * n + 2**22               # run starts and sign terms; counts per workgroup and region
                    assert need <= lists + max(12 * m, 3 * 2**27), (m, d, Z, n)
                    fused = robe.robe_fused_workspace_bytes(h, n, 1, n)
                    assert fused <= lists + max(12 * m, 3 * 2**27) + 4 * m + 256
    assert took > 50


def test_few_requests_a_token_are_not_sorted():
    """Bags and lookups whose direct scatter is quicker than the sort alone, on both sides of 2^25 elements."""
    for d, Z, n in ((8, 8, 70_000), (8, 8, 200_000), (16, 4, 70_000), (16, 16, 150_000), (32, 32, 100_000), (4, 2, 150_000)):
        assert robe.robe_workspace_bytes(robe.robe_init_hash(1, 4_000_000, d, Z, 0), n, 1, n) == 0, (d, Z, n)
    for d, Z, n in ((100, 10, 66_000), (64, 16, 80_000), (16, 4, 120_000), (128, 32, 120_000), (8, 8, 300_000), (4, 2, 2**23)):
        assert robe.robe_workspace_bytes(robe.robe_init_hash(1, 4_000_000, d, Z, 0), n, 1, n) > 0, (d, Z, n)


def test_long_blocks_and_single_ones_count_for_more_in_small_regions():
    """Regions of few records grow past 2^13 slots: seen in the workspace, which holds counts for each of them."""
    def grown(m, d, Z, n):
        h = robe.robe_init_hash(1, m, d, Z, 0)
        return (robe.robe_fused_workspace_bytes(h, n, 1, n) !=
                robe.robe_fused_workspace_bytes(h, n, 1, n, robe.options(region_shift=13, region_records=1)))
    m = 250_000_000
    for d, Z, blocks in ((128, 32, 40), (128, 16, 20), (128, 64, 30), (128, 128, 20)):
        assert grown(m, d, Z, blocks * m // 8192 * Z // d), (d, Z, blocks)
    for d, Z, blocks in ((128, 64, 42), (128, 128, 28)):
        assert not grown(m, d, Z, blocks * m // 8192 * Z // d), (d, Z, blocks)


def test_the_fused_step_takes_regions_by_rows_and_requests():
    def regions(m, d, Z, n):
        h = robe.robe_init_hash(1, m, d, Z, 0)
        need = [robe.robe_fused_workspace_bytes(h, n, 1, n, robe.options(fused_route=r)) for r in (robe.ROUTE_AUTO, robe.ROUTE_REGIONS, robe.ROUTE_TWO_STEP)]
        assert need[0] in need[1:] and need[1] != need[2]
        return need[0] == need[1]
    for m, d, Z, n in ((25_000_000, 128, 32, 100_000), (25_000_000, 64, 16, 200_000), (25_000_000, 32, 4, 200_000), (60_000_000, 128, 32, 50_000),
                       (33_000_000, 128, 128, 200_000), (40_000_000, 128, 32, 1_700_000), (2**26, 16, 16, 100)):
        assert regions(m, d, Z, n), (m, d, Z, n)
    for m, d, Z, n in ((20_000_000, 128, 32, 400_000), (25_000_000, 128, 32, 50_000), (25_000_000, 16, 4, 400_000), (25_000_000, 32, 4, 400_000),
                       (33_000_000, 128, 128, 400_000), (25_000_000, 128, 32, 2**20 + 1), (34_000_000, 16, 16, 150_000), (34_000_000, 64, 64, 100_000)):
        assert not regions(m, d, Z, n), (m, d, Z, n)


def test_the_shorter_sort_takes_the_plain_sorts_workspace():
    """Tokens are sorted on 16 bits up to 2^21 of them: a caller whose buffer holds the 24-bit sort has room enough."""
    for m, d, Z in ((25_000_000, 128, 32), (1_000_003, 16, 4), (25_000_000, 100, 10), (25_000_000, 128, 1), (2**26, 64, 16)):
        for n in (1000, 2**18, 2**18 + 1, 300_000, 852_000, 2**21, 2**21 + 1):
            for sign in (0, 1):
                h = robe.robe_init_hash(1, m, d, Z, sign)
                for asked in ({}, {"backward_route": robe.ROUTE_COMBINE}, {"backward_route": robe.ROUTE_COMBINE, "fused_route": robe.ROUTE_TWO_STEP}):
                    for query in (robe.robe_workspace_bytes, robe.robe_fused_workspace_bytes):
                        assert query(h, n, 1, n, robe.options(**asked)) == query(h, n, 1, n, robe.options(key_bits=24, **asked)), (m, d, Z, n, sign, asked)
