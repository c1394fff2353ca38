"""Forward kernels that hash a block's offset in one lane for all lanes that read the block (Z at least four
lanes' elements, or Z > d): the bits of the oracle (single-hot) and of the kernels that hash in every lane
(bags, whose sums are in token order on both), over rows of one to 64 lanes, one to 16 chunks, arrays little
longer than a block (most spans cross the end), batches that end inside a wavefront's rows, both row orders,
ids of every size, empty bags and bags longer than a lane group, signs and bfloat16."""
import numpy as np
import pytest

import oracle
import paper_2108_02191_amd as robe
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu


def _ids(rng, n):
    ids = rng.integers(0, 50, size=n, dtype=np.int64)
    wide = rng.random(n) < 0.3
    ids[wide] = rng.integers(-2**63, 2**63 - 1, size=int(wide.sum()), dtype=np.int64)
    return ids


@pytest.mark.parametrize("sign", [0, 1])
@pytest.mark.parametrize("d,Z,m", [(4, 16, 17), (16, 16, 31), (32, 16, 5003), (64, 64, 131), (128, 16, 40_009), (128, 32, 67),
                                   (128, 128, 1021), (256, 32, 9973), (256, 256, 259), (128, 512, 515), (2, 8, 4001)])
def test_block_offsets(d, Z, m, sign):
    h, H = P.both_hashes(d + Z, m, d, Z, sign)
    rng = np.random.default_rng(m)
    M = rng.standard_normal(m).astype(np.float32)
    A = P.to_dev(M)
    b16 = robe.robe_array_to_bf16(A)
    wide = b16.float().cpu().numpy() if hasattr(b16, "float") and b16.is_floating_point() else \
        (b16.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    lanes = robe.options(fwd_elems=2 if d <= 128 else 4, fwd_strided=1)
    for B, F, order in ((1, 1, 0), (3, 7, 0), (37, 5, 3), (129, 3, 3), (700, 13, 0)):
        opt = robe.options(row_order=order)
        ids = _ids(rng, B * F)
        I = P.to_dev(ids.reshape(B, F))
        got = robe.robe_forward(h, A, I, None, B, F, options=opt).cpu().numpy()
        want = oracle.forward(H, M, ids.reshape(B, F), None, B, F)
        assert np.array_equal(got.view(np.int32), want.view(np.int32).reshape(got.shape)), (B, F)
        got = robe.robe_forward_bf16(h, b16, I, None, B, F, options=opt).cpu().numpy()
        want = oracle.forward(H, wide, ids.reshape(B, F), None, B, F)
        assert np.array_equal(got.view(np.int32), want.view(np.int32).reshape(got.shape)), (B, F)
        sizes = rng.poisson(6.0, size=B * F)
        sizes[::5] = 0
        sizes[-1] = 150
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        T, O = P.to_dev(_ids(rng, int(off[-1]))), P.to_dev(off)
        for call, array in ((robe.robe_forward, A), (robe.robe_forward_bf16, b16)):
            got = call(h, array, T, O, B, F, options=opt).cpu().numpy()
            want = call(h, array, T, O, B, F, options=lanes).cpu().numpy()
            assert np.array_equal(got.view(np.int32), want.view(np.int32)), (B, F)
