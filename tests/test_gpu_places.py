"""Single-hot lookups of blocks of one or two floats on arrays that no L2 holds, served region by region of the array:
the bits of the route that gathers every lookup (a requested row order keeps a call on it).  Arrays of a power of two
slots and around it, a last region of one slot and of most of one, rows of one to eight elements a page (an odd number
too, where blocks of two lie across pages), ids that hardly repeat (no rows free for the tiles), always repeat, repeat
enough, crowd one table, or differ by multiples of P; signs and the bfloat16 array; one launch captured and replayed."""
import numpy as np
import pytest
import torch

import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P
from tests.launches import kernels
from tests.test_gpu_distinct import _first_batch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _ids(kind, B, F, seed=0):
    rng = np.random.default_rng(B + seed)
    n = B * F
    if kind == "same":
        return np.full((B, F), -5, np.int64)
    if kind == "distinct":
        return (rng.permutation(np.arange(n, dtype=np.int64)) * 977 - 10**6).reshape(B, F)
    if kind == "halves":        # every id of a table twice, most of them in different tiles
        return np.stack([rng.permutation(np.arange(B, dtype=np.int64) // 2) for _ in range(F)], 1)
    ids = rng.zipf(1.2, size=(B, F)).astype(np.int64) % 10**9
    return ids + (rng.integers(0, 3, size=(B, F)) * (2**31 - 1) if kind == "congruent" else 0)


CASES = [(2**23, 128, 1, 26, "zipf", 0), (2**23 + 1, 128, 2, 9, "zipf", 1), (2**23 + 16383, 512, 1, 3, "zipf", 1), (9_000_011, 64, 1, 2, "zipf", 0),
         (9_000_011, 64, 2, 30, "zipf", 1), (9_000_011, 192, 2, 7, "congruent", 0), (9_000_011, 320, 1, 5, "congruent", 1), (2**23, 448, 2, 4, "zipf", 0),
         (2**24 + 1, 128, 1, 5, "distinct", 1), (2**23, 128, 1, 5, "same", 0), (12_345_678, 128, 1, 26, "halves", 0), (12_345_678, 128, 2, 1, "halves", 1)]


@pytest.mark.parametrize("m,d,Z,F,kind,sign", CASES)
def test_served_rows_have_the_gathered_bits(m, d, Z, F, kind, sign):
    h, _ = P.both_hashes(d, m, d, Z, sign)
    B = _first_batch(d, Z, F) + 3
    n = B * F
    A = torch.randn(m, device=DEV)
    I = P.to_dev(_ids(kind, B, F))
    plain = robe.options(row_order=robe.ROWS_BY_TABLE)
    want = robe.robe_forward(h, A, I, None, B, F, options=plain)
    room = torch.full((n * d + 8,), 7.0, device=DEV)
    out = room[4:4 + n * d].view(B, F, d)
    assert kernels(lambda: robe.robe_forward(h, A, I, None, B, F, out=out)) == 8
    robe.robe_forward(h, A, I, None, B, F, out=out)
    assert torch.equal(out.view(torch.int32), want.view(torch.int32))
    assert (room[:4] == 7.0).all() and (room[4 + n * d:] == 7.0).all()
    b16 = robe.robe_array_to_bf16(A)
    got, want = robe.robe_forward_bf16(h, b16, I, None, B, F), robe.robe_forward_bf16(h, b16, I, None, B, F, options=plain)
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))


def _least(m, d, Z):
    """From how many distinct tokens on the lists are served."""
    C = d // Z
    if C <= 128:
        return m // 8 // C + 1
    return (m // 1024 * 5 // 8 + m * 3 // 64 // C if Z == 1 else m // 1024) + 1


@pytest.mark.parametrize("m,d,Z,F,kind,sign", CASES)
def test_the_cases_are_served_or_not(m, d, Z, F, kind, sign):
    """What the device decides by, from the ids alone: distinct tokens enough, and as many free rows (of those before the last
    samples, 5 words a lookup at the most)."""
    B = _first_batch(d, Z, F) + 3
    ids = _ids(kind, B, F)
    keep = B - 5 * B // d - 2
    tokens = len(np.unique(ids[:keep] % (2**31 - 1) + (np.arange(F) << 32)))
    free = keep * F - tokens
    assert (tokens >= _least(m, d, Z) and free >= _least(m, d, Z) + 64 * 32) == (kind not in ("same", "distinct")), (tokens, free)


# arrays of more than 100 M slots and outputs past 2 GiB, where sizes in bytes have the top bit of 32 set, up to the last size of the route
@pytest.mark.parametrize("m,d,Z,B,kind,sign", [(2**27 + 5, 128, 1, 170_000, "zipf", 1), (2**27 - 3, 128, 2, 165_000, "few", 0), (2**29 - 1, 128, 1, 322_638, "few", 0),
                                               (2**23 + 77, 512, 1, 80_659, "few", 1)])
def test_large_arrays_and_outputs(m, d, Z, B, kind, sign):
    F = 26
    n = B * F
    assert 2**31 < n * d * 4 < 2**32
    h, _ = P.both_hashes(d, m, d, Z, sign)
    A = torch.randn(m, device=DEV)
    if kind == "few":             # twice as many distinct tokens as are worth it, in most of the rows
        I = torch.randint(0, 2 * _least(m, d, Z) // F, (B, F), device=DEV)
    else:
        I = P.to_dev(_ids(kind, B, F))
    assert len(torch.unique(I + (torch.arange(F, device=DEV) << 32))) >= _least(m, d, Z)
    room = torch.full((n * d + 8,), 7.0, device=DEV)
    out = room[4:4 + n * d].view(B, F, d)
    assert kernels(lambda: robe.robe_forward(h, A, I, None, B, F, out=out)) == 8
    robe.robe_forward(h, A, I, None, B, F, out=out)
    want = robe.robe_forward(h, A, I, None, B, F, options=robe.options(row_order=robe.ROWS_BY_TABLE))
    for first in range(0, B, 50_000):                          # (a comparison holds copies)
        assert torch.equal(out[first:first + 50_000].view(torch.int32), want[first:first + 50_000].view(torch.int32))
    assert (room[:4] == 7.0).all() and (room[4 + n * d:] == 7.0).all()


@pytest.mark.parametrize("m,d,Z,off,launches", [(2**23 - 1, 128, 1, 0, 5), (2**23, 100, 1, 0, 5), (2**23, 128, 4, 0, 5), (2**23, 128, 1, 1, 5), (2**26, 128, 1, 0, 5),
                                                (2**23, 128, 1, 4, 8)])
def test_what_takes_the_route(m, d, Z, off, launches):
    F = 26
    h, _ = P.both_hashes(1, m, d, Z, 0)
    B = _first_batch(d, Z, F) + 1
    A, I = torch.zeros(m, device=DEV), torch.zeros((B, F), dtype=torch.int64, device=DEV)
    out = torch.empty(B * F * d + 8, device=DEV)[off:off + B * F * d].view(B, F, d)
    assert kernels(lambda: robe.robe_forward(h, A, I, None, B, F, out=out)) == launches


def test_replays_repeat():
    m, d, F, B = 9_000_011, 128, 26, 9000
    h, _ = P.both_hashes(1, m, d, 1, 1)
    A = torch.randn(m, device=DEV)
    I = P.to_dev(_ids("zipf", B, F))
    out = torch.empty(B, F, d, device=DEV)
    robe.robe_forward(h, A, I, None, B, F, out=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        robe.robe_forward(h, A, I, None, B, F, out=out)
    plain = robe.options(row_order=robe.ROWS_BY_TABLE)
    for r in range(4):
        I.copy_(P.to_dev(_ids("zipf" if r % 2 else "halves", B, F, r)))
        out.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, robe.robe_forward(h, A, I, None, B, F, options=plain)), r
