"""The largest layer the int32 CSR layout holds: N = K = 46340, so a full
result has N*K = 2,147,395,600 entries, just below 2^31.  Row pointers and
output positions then come within 0.01 % of the int32 range; the whole row
pointer array and the entries at both ends of the output (positions near 0
and near 2^31) are checked exactly.  About 26 GB of device memory each."""
import numpy as np
import pytest

import oracle
import paper_1905_07931_amd as L1

from _helpers import cuda, h

pytestmark = pytest.mark.gpu

N = K = 46340
ZEROS = [(0, 0), (1, K - 1), (N // 2, 123), (N - 1, K - 1)]


def _expected_row_ptr():
    cnt = np.full(N, K, np.int64)
    for i, _ in ZEROS:
        cnt[i] -= 1
    return np.concatenate([[0], np.cumsum(cnt)])


def _check_structure(out, val):
    rp = h(out.row_ptr).astype(np.int64)
    exp = _expected_row_ptr()
    assert np.array_equal(rp, exp)
    assert rp[-1] == N * K - len(ZEROS) and rp[-1] < 2 ** 31
    for i, k0 in ZEROS:
        ci = h(out.col_idx[int(rp[i]):int(rp[i + 1])])
        assert np.array_equal(ci, np.delete(np.arange(K, dtype=np.int32), k0)), i
        assert np.all(h(out.vals[int(rp[i]):int(rp[i + 1])]) == val), i
    # a full row in the middle of the array
    i = N // 3
    assert np.array_equal(h(out.col_idx[int(rp[i]):int(rp[i + 1])]), np.arange(K, dtype=np.int32))


def test_recompress_at_the_int32_limit():
    import torch
    Z = torch.full((N, K), 0.5, device=cuda())
    for i, k in ZEROS:
        Z[i, k] = 0.0
    out = L1.csr_recompress(Z)
    torch.cuda.synchronize()
    del Z
    _check_structure(out, np.float32(0.5))
    del out
    torch.cuda.empty_cache()


def test_prox_recompress_at_the_int32_limit():
    # an empty W and G = -1 everywhere: z = eta, kept with value S_t(eta), t = eta*lam;
    # G = 0 at the chosen positions gives z = 0 there, dropped
    import torch
    eta, lam = 0.01, 0.5
    W = L1.CSR.from_host(np.zeros(N + 1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32), K,
                         device=cuda())
    G = torch.full((N, K), -1.0, device=cuda())
    for i, k in ZEROS:
        G[i, k] = 0.0
    out = L1.prox_l1_recompress(W, G, eta, lam)
    torch.cuda.synchronize()
    del G
    Zr, _ = oracle.prox_dense(np.zeros(2, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32),
                              np.full((1, 1), -1.0, np.float32), eta, lam, 1)
    _check_structure(out, Zr[0, 0])
    del out
    torch.cuda.empty_cache()


def test_csc_build_beyond_one_launch_of_the_emit_pass():
    # 13108.x row blocks x 320 words x 4 column groups of 256 threads: more than the 2^32 threads
    # of one launch; entries at both ends and in every row block's last row.  36 GB of bitmap index.
    import torch
    n, k = 13108 * 1024 + 5, 10240
    rows = np.unique(np.concatenate([np.arange(1023, n, 1024), [0, 1, n - 2, n - 1]]))
    cols = (rows.astype(np.int64) * 7919) % k
    cols[0], cols[-1] = k - 1, 0
    rp = np.zeros(n + 1, np.int32)
    rp[rows + 1] = 1
    rp = np.cumsum(rp, dtype=np.int32)
    vals = np.arange(1, len(rows) + 1, dtype=np.float32)
    W = L1.CSR.from_host(rp, cols.astype(np.int32), vals, k, device=cuda())
    csc = L1.csc_build(W)
    order = np.lexsort((rows, cols))
    assert np.array_equal(h(csc.col_ptr), np.concatenate([[0], np.cumsum(np.bincount(cols, minlength=k))]))
    assert np.array_equal(h(csc.row_idx), rows[order]) and np.array_equal(h(csc.perm), order)
    assert np.array_equal(h(csc.vals_t), vals[order])
    del W, csc
    torch.cuda.empty_cache()


def test_row_product_of_nearly_a_whole_launch():
    # 4095 x 4097 workgroups, 2^24 - 1 (a launch's most): none can be added for long rows.  17 GB of Y.
    import torch
    n, k, b = 4095 * 4, 400, 4097 * 64 - 1
    rp = np.zeros(n + 1, np.int32)
    rp[1], rp[8], rp[n // 2], rp[n] = 300, 5, 2, 7  # one long row
    rp = np.cumsum(rp, dtype=np.int32)
    ci = np.concatenate([np.arange(300), np.arange(5), [7, 399], np.arange(7)]).astype(np.int32)
    v = np.random.default_rng(1).standard_normal(len(ci)).astype(np.float32)
    W = L1.CSR.from_host(rp, ci, v, k, device=cuda())
    X = torch.zeros((k, b), device=cuda())
    cols = torch.tensor([0, 63, 64, b // 2, b - 65, b - 1], device=cuda())
    X[:, cols] = torch.rand((k, 6), device=cuda(), generator=torch.Generator("cuda").manual_seed(2))
    Y = torch.full((n, b), 3.0, device=cuda())
    L1.csr_spmm_fwd(W, X, Y)
    x, got = h(X[:, cols]).astype(np.float64), h(Y[:, cols])
    ref, m = np.zeros((n, 6)), np.zeros((n, 6))
    rows = np.repeat(np.arange(n), np.diff(rp))
    np.add.at(ref, rows, v[:, None] * x[ci])
    np.add.at(m, rows, np.abs(v)[:, None] * x[ci])
    assert (np.abs(got - ref) <= 304 * 2.0 ** -24 * m).all()
    assert not bool((Y[-1] == 3.0).any()) and not bool((Y[1] != 0).any())
    del X, Y
    torch.cuda.empty_cache()
