"""Single-hot lookups of small blocks that gather every distinct token once and copy its row: the bits of the
route that gathers every lookup (a requested row order keeps a call on it), over strided and consecutive lane
layouts, rows that four floats do not divide, outputs off 16- and 8-byte alignment, ids that never repeat,
always repeat, repeat in some tiles only, or differ by multiples of P (the same places), batches that end inside
a tile, one table and many, signs and the bfloat16 array.  Which route a call takes is seen in its launches."""
import numpy as np
import pytest
import torch

import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P
from tests.launches import kernels

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _ids(kind, n):
    rng = np.random.default_rng(n)
    if kind == "same":
        return np.full(n, -5, np.int64)
    if kind == "distinct":
        return rng.permutation(np.arange(n, dtype=np.int64) * 977 - 10**6)
    if kind == "patches":       # one id in a few long stretches, others that never repeat
        ids = np.arange(n, dtype=np.int64)
        ids[(ids // 50_000) % 3 == 0] = 7
        return ids
    ids = rng.zipf(1.3, size=n).astype(np.int64) % 10**9
    return ids + (rng.integers(0, 3, size=n) * (2**31 - 1) if kind == "congruent" else 0)


def _first_batch(d, Z, F):
    """The smallest batch whose lookups read lines enough, from the rule's two numbers."""
    lines = d // Z * (31 + Z) / 32
    return int(-(-21_000_000 // ((lines - 18) * F)))


@pytest.mark.parametrize("d,Z,F,kind,sign", [(512, 1, 3, "zipf", 0), (512, 4, 1, "zipf", 1), (128, 1, 26, "zipf", 1), (128, 2, 7, "congruent", 0),
                                             (100, 1, 5, "congruent", 1), (64, 1, 2, "zipf", 0), (192, 1, 40, "same", 0), (384, 2, 9, "distinct", 1),
                                             (33, 1, 4, "zipf", 0), (512, 1, 100, "zipf", 1), (128, 1, 4, "patches", 1), (384, 4, 3, "distinct", 0), (512, 2, 1, "patches", 0)])
def test_copied_rows_have_the_gathered_bits(d, Z, F, kind, sign):
    m = 777_777
    h, _ = P.both_hashes(d, m, d, Z, sign)
    B = _first_batch(d, Z, F) + 3
    n = B * F
    A = torch.randn(m, device=DEV)
    I = P.to_dev(_ids(kind, n).reshape(B, F))
    plain = robe.options(row_order=robe.ROWS_BY_TABLE)
    want = robe.robe_forward(h, A, I, None, B, F, options=plain)
    for off in (0, 1, 2):
        room = torch.full((n * d + 8,), 7.0, device=DEV)
        out = room[off:off + n * d].view(B, F, d)
        assert kernels(lambda: robe.robe_forward(h, A, I, None, B, F, out=out)) == 5
        robe.robe_forward(h, A, I, None, B, F, out=out)
        assert torch.equal(out.view(torch.int32), want.view(torch.int32)), off
        assert (room[:off] == 7.0).all() and (room[off + n * d:] == 7.0).all()
    b16 = robe.robe_array_to_bf16(A)
    got, want = robe.robe_forward_bf16(h, b16, I, None, B, F), robe.robe_forward_bf16(h, b16, I, None, B, F, options=plain)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("d,Z,F", [(128, 1, 26), (128, 2, 26), (128, 4, 5), (64, 1, 2), (512, 4, 1)])
def test_fewer_lines_and_requested_orders_take_the_plain_route(d, Z, F):
    h, _ = P.both_hashes(1, 777_777, d, Z, 0)
    B = _first_batch(d, Z, F)
    A = torch.zeros(h.m, device=DEV)
    I = torch.zeros((B + 1, F), dtype=torch.int64, device=DEV)
    out = torch.empty((B + 1, F, d), device=DEV)
    def launches(b, **asked):
        return kernels(lambda: robe.robe_forward(h, A, I[:b], None, b, F, out=out[:b], options=robe.options(**asked)))
    assert launches(B + 1) == 5
    assert launches(B - 1) == 1
    for asked in ({"row_order": robe.ROWS_MEMORY}, {"row_order": robe.ROWS_BY_TABLE}, {"tile_lookups": 64}, {"fwd_elems": -1}):
        assert launches(B + 1, **asked) == 1, asked


@pytest.mark.parametrize("d,Z,rows", [(32, 4, 1_700_000), (32, 2, 852_000), (16, 1, 2_000_000), (128, 8, 2_000_000)])
def test_rows_of_few_lines_take_the_plain_route(d, Z, rows):
    """Whatever their number: the lists cost more than the lines they save."""
    h, _ = P.both_hashes(1, 777_777, d, Z, 0)
    A, I = torch.zeros(h.m, device=DEV), torch.zeros((rows // 4, 4), dtype=torch.int64, device=DEV)
    out = torch.empty((rows // 4, 4, d), device=DEV)
    assert kernels(lambda: robe.robe_forward(h, A, I, None, rows // 4, 4, out=out)) == 1


def test_one_sample_has_no_room_for_the_lists():
    d, F = 128, 250_001
    h, _ = P.both_hashes(1, 777_777, d, 1, 0)
    A = torch.randn(h.m, device=DEV)
    I = P.to_dev(_ids("zipf", F).reshape(1, F))
    out = torch.empty((1, F, d), device=DEV)
    assert kernels(lambda: robe.robe_forward(h, A, I, None, 1, F, out=out)) == 1
    robe.robe_forward(h, A, I, None, 1, F, out=out)
    assert torch.equal(out, robe.robe_forward(h, A, I, None, 1, F, options=robe.options(row_order=robe.ROWS_MEMORY)))


def test_replays_repeat():
    """One launch captured into a graph, replayed on new ids each time."""
    m, d, F, B = 777_777, 128, 26, 7500
    h, _ = P.both_hashes(1, m, d, 1, 0)
    A = torch.randn(m, device=DEV)
    I = P.to_dev(_ids("zipf", B * F).reshape(B, F))
    out = torch.empty(B, F, d, device=DEV)
    robe.robe_forward(h, A, I, None, B, F, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        robe.robe_forward(h, A, I, None, B, F, out=out)
    plain = robe.options(row_order=robe.ROWS_BY_TABLE)
    for r in range(4):
        I.copy_(P.to_dev((_ids("zipf", B * F) * (r + 3) % 10**6).reshape(B, F)))
        out.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, robe.robe_forward(h, A, I, None, B, F, options=plain)), r
