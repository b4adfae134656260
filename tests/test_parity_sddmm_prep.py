"""GPU: the masked gradient's list of row pieces and column-range bounds, made in
one launch: row counts around the rows of one pass, long rows at both ends of a
pass, one and several column ranges, against 64-bit references and run to run."""
import numpy as np
import pytest

import paper_1905_07931_amd as L1
from _helpers import bits_equal, h, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,B", [(1, 300, 8), (15, 900, 32), (4095, 500, 8), (4096, 500, 8), (4097, 500, 8), (8200, 500, 12),
                                   (17, 4096, 512), (4099, 2600, 516), (1024, 500, 8), (1025, 500, 8), (2048, 500, 8),
                                   (32768, 400, 4), (32769, 400, 4), (41000, 300, 4)])
def test_row_pieces(N, K, B):
    check(N, K, B, 0)


@pytest.mark.parametrize("N,K,B", [(1025, 500, 8), (2048, 500, 8), (2049, 500, 12), (4095, 500, 8), (4096, 500, 8)])
def test_row_pieces_up_to_4096_rows(N, K, B):
    # beyond 16 entries a row a workgroup lists 1024 rows here too, and one lists all of them below
    check(N, K, B, 16)


def check(N, K, B, least):
    rng = np.random.default_rng(N)
    n = rng.integers(least, least + 4, N)
    for i in (0, 1, 1023, 1024, 2047, 4095, 4096, 4097, 8191, 32767, 32768, N // 2, N - 1):
        if i < N:
            n[i] = K - i % 7
    rp = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(K, c, replace=False)) for c in n]).astype(np.int32)
    W = L1.CSR.from_host(rp, ci, np.ones(len(ci), np.float32), K)
    X, dY = rng.random((K, B)).astype(np.float32), rng.standard_normal((N, B)).astype(np.float32)
    gv = h(L1.sddmm_masked_wgrad(W, t(dY), t(X)))[:len(ci)]
    rows = np.repeat(np.arange(N), n)
    a, x = dY[rows].astype(np.float64), X[ci].astype(np.float64)
    # a lane's chain over its share of the batch, then six levels of a tree and the ranges' sums
    bound = (B / 64 + 12) * 2.0 ** -24 * (np.abs(a) * x).sum(axis=1)
    assert (np.abs(gv - (a * x).sum(axis=1)) <= bound).all()
    assert bits_equal(h(L1.sddmm_masked_wgrad(W, t(dY), t(X)))[:len(ci)], gv)
