"""GPU: the bitmap index and the CSC build at the edges of their workgroups: rows
past a 16-row block, words past a column quarter and a 64-word scan step, one and
several 1024-row blocks, columns with more entries of a block than its staged run,
entry counts that leave a wave's last lanes idle."""
import numpy as np
import pytest

import paper_1905_07931_amd as L1
from _helpers import bits_equal, csc_reference, h

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,d", [(1, 1, 1.0), (15, 33, 0.5), (17, 31, 0.3), (16, 2049, 0.9), (1024, 40, 0.6),
                                   (1025, 65, 0.5), (2050, 9, 1.0), (33, 10240, 0.2), (33, 10250, 0.2), (70, 4100, 0.01)])
def test_bitmap_and_csc_edges(N, K, d):
    rng = np.random.default_rng(N * 7 + K)
    mask = rng.random((N, K)) < d
    if N > 2 and d < 1:
        mask[1] = False
        mask[N - 2] = True
    rp = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    ci = np.nonzero(mask)[1].astype(np.int32)
    v = rng.standard_normal(max(len(ci), 1)).astype(np.float32)[:len(ci)]
    W = L1.CSR.from_host(rp, ci, v, K)
    kw = -(-K // 32)
    words = np.zeros((N, kw * 32), bool)
    words[:, :K] = mask
    words = words.reshape(N, kw, 32)
    want = (words * (1 << np.arange(32, dtype=np.int64))).sum(2).astype(np.uint32).view(np.int32)
    counts = words.sum(2)
    pos = rp[:-1, None] + np.cumsum(counts, 1) - counts
    bm = L1.csr_bitmap_build(W)
    assert bits_equal(h(bm.mask), np.ascontiguousarray(want.T))
    assert bits_equal(h(bm.pos), np.ascontiguousarray(pos.T.astype(np.int32)))
    cp, ri, pm = csc_reference(rp, ci, K)
    for csc in (L1.csc_build(W), L1.csc_build(W, bitmap=bm)):
        n = len(ci)
        assert bits_equal(h(csc.col_ptr), cp)
        assert bits_equal(h(csc.row_idx)[:n], ri) and bits_equal(h(csc.perm)[:n], pm)
        assert bits_equal(h(csc.vals_t)[:n], v[pm])
