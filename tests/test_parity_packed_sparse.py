"""GPU: products over dense patterns on packed operands (csr_spmm_fwd, csr_spmm_bwd_t
and sddmm_masked_wgrad with the packed workspace) against 64-bit references: tile and
step edges, power-law and empty rows, split reductions, operands outside the parts'
range, and the same bits from the planned calls."""
import numpy as np
import pytest

import paper_1905_07931_amd as L1
from paper_1905_07931_amd import synth
from _helpers import bits_equal, h, t

pytestmark = pytest.mark.gpu


def layer(N, K, B, density, seed=0, pattern="uniform", empty=True):
    rng = np.random.default_rng(seed)
    if pattern == "zipf":
        rp, ci = synth.zipf_pattern(rng, N, K, int(density * N * K))
    else:
        mask = rng.random((N, K)) < density
        if empty:
            mask[N // 3] = False
            mask[:, K // 2] = False
            mask[N - 1] = True
        rp = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
        ci = np.nonzero(mask)[1].astype(np.int32)
    v = (rng.standard_normal(len(ci)) * 0.1).astype(np.float32)
    dense = np.zeros((N, K))
    dense[np.repeat(np.arange(N), np.diff(rp)), ci] = v
    X, dY = rng.random((K, B)).astype(np.float32), rng.standard_normal((N, B)).astype(np.float32)
    return L1.CSR.from_host(rp, ci, v, K), dense, rp, ci, X, dY


def bound(terms):
    # the terms left out of a product (2^-22), then a rounding per summed term
    return 2.0 ** -22 + (terms / 16 + 96) * 2.0 ** -24


SHAPES = [(1024, 1024, 384, 0.4, "uniform"), (1025, 1281, 333, 0.3, "uniform"), (1537, 1000, 1001, 0.25, "zipf"),
          (2049, 2305, 130, 0.3, "uniform"), (300, 4097, 515, 0.5, "uniform")]


@pytest.mark.parametrize("N,K,B,d,pattern", SHAPES)
def test_packed_products(N, K, B, d, pattern):
    W, dense, rp, ci, X, dY = layer(N, K, B, d, seed=N + B, pattern=pattern)
    assert L1.workspace_bytes(L1.OP_SPMM_PACKED, N, K, W.nnz, B) > 0
    assert L1.workspace_bytes(L1.OP_SPMM_PACKED, K, N, W.nnz, B) > 0
    Xd, dYd = t(X), t(dY)
    Y = L1.csr_spmm_fwd(W, Xd)
    assert (np.abs(h(Y) - dense @ X) <= bound(6 * K) * (np.abs(dense) @ np.abs(X))).all()
    csc = L1.csc_build(W)
    dX = L1.csr_spmm_bwd_t(W, dYd, csc)
    assert (np.abs(h(dX) - dense.T @ dY) <= bound(6 * N) * (np.abs(dense).T @ np.abs(dY))).all()
    for got, ref in ((h(Y), dense @ X), (h(dX), dense.T @ dY)):  # (two parts are at some 5e-6)
        assert np.linalg.norm(got - ref) <= 8e-7 * np.linalg.norm(ref)
    # again, planned, and into padded rows: the same bits
    import torch
    assert bits_equal(h(L1.csr_spmm_planned(W, Xd, L1.csr_spmm_plan(W, B))), h(Y))
    assert bits_equal(h(L1.csr_spmm_bwd_t_planned(W, dYd, csc, L1.csr_spmm_bwd_t_plan(W, csc, B))), h(dX))
    wide = torch.full((N, B + 3), 7.0, device="cuda")
    L1.csr_spmm_fwd(W, Xd, wide[:, :B])
    assert bits_equal(h(wide[:, :B].contiguous()), h(Y)) and bool((wide[:, B:] == 7.0).all())


@pytest.mark.parametrize("N,K,B,d,pattern", [(1024, 2048, 256, 0.4, "uniform"), (2049, 3001, 97, 0.3, "uniform"),
                                             (2177, 2050, 333, 0.25, "zipf"), (600, 1300, 530, 0.4, "uniform")])
def test_packed_masked_gradient(N, K, B, d, pattern):
    W, dense, rp, ci, X, dY = layer(N, K, B, d, seed=B, pattern=pattern)
    assert L1.workspace_bytes(L1.OP_SDDMM_PACKED, N, K, W.nnz, B) > 0
    import torch
    gv = torch.full((W.nnz + 5,), 3.0, device="cuda")  # entries past the pattern stay
    L1.sddmm_masked_wgrad(W, t(dY), t(X), gv)
    rows = np.repeat(np.arange(N), np.diff(rp))
    ref = (dY.astype(np.float64) @ X.astype(np.float64).T)[rows, ci]
    m = (np.abs(dY).astype(np.float64) @ np.abs(X).astype(np.float64).T)[rows, ci]
    assert (np.abs(h(gv)[:W.nnz] - ref) <= bound(6 * B) * m).all()
    assert np.linalg.norm(h(gv)[:W.nnz] - ref) <= 3e-7 * np.linalg.norm(ref)
    assert bool((gv[W.nnz:] == 3.0).all())


def test_packed_products_odd_values():
    # values no three bf16 parts hold: the stored entries alone are summed, so an
    # infinity meets only the rows that store its column
    N, K, B = 1024, 1100, 500
    W, dense, rp, ci, X, dY = layer(N, K, B, 0.4, seed=9)
    assert L1.workspace_bytes(L1.OP_SPMM_PACKED, N, K, W.nnz, B) > 0
    X[17, 5], X[1000, 299], X[40, 130] = np.inf, np.nan, 3e38
    X[:, 200] *= np.float32(2.0 ** -115)
    got = h(L1.csr_spmm_fwd(W, t(X))).astype(np.float64)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = np.zeros((N, B), np.float64)
        for i in range(N):
            s = slice(rp[i], rp[i + 1])
            ref[i] = (dense[i, ci[s]][:, None] * X[ci[s]].astype(np.float64)).sum(axis=0)
        ref = ref.astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    m = np.abs(dense) @ np.where(np.isfinite(X), np.abs(X.astype(np.float64)), 0)
    assert (np.abs(got[ok] - ref[ok]) <= 1e-4 * m[ok] + 2.0 ** -149 * K).all()


def test_packed_products_small_beside_large():
    # rows of normal values that meet zeros alone, beside others of 2^-80 to 2^-145
    N, K, B = 1024, 2048, 256
    W, dense, rp, ci, X, dY = layer(N, K, B, 0.4, seed=11)
    assert L1.workspace_bytes(L1.OP_SPMM_PACKED, N, K, W.nnz, B) > 0
    assert L1.workspace_bytes(L1.OP_SDDMM_PACKED, N, K, W.nnz, B) > 0
    small = np.exp2(-np.linspace(80, 145, N)).astype(np.float32)
    rows = np.repeat(np.arange(N), np.diff(rp))
    W.vals.copy_(t(np.where(ci % 2 == 1, small[rows], np.float32(1)) * h(W.vals)))
    dense[rows, ci] = h(W.vals)
    Xf = (X * np.float32(2.0 ** 27)).astype(np.float32)
    Xf[0::2] = 0
    got, x = h(L1.csr_spmm_fwd(W, t(Xf))).astype(np.float64), Xf.astype(np.float64)
    assert (np.abs(got - dense @ x) <= bound(6 * K) * (np.abs(dense) @ x)).all()
    dY[:, 1::2] *= small[:, None]
    Xg = (X * np.float32(2.0 ** 27)).astype(np.float32)
    Xg[:, 0::2] = 0
    gv = h(L1.sddmm_masked_wgrad(W, t(dY), t(Xg))).astype(np.float64)[:W.nnz]
    a, x = dY.astype(np.float64), Xg.astype(np.float64)
    assert (np.abs(gv - (a @ x.T)[rows, ci]) <= bound(6 * B) * (np.abs(a) @ x.T)[rows, ci]).all()


@pytest.mark.parametrize("N,K,B,d,pattern", [(1025, 1281, 333, 0.3, "uniform"), (300, 4097, 515, 0.5, "uniform"),
                                             (2049, 2305, 130, 0.3, "uniform")])
def test_packed_products_flagged_blocks(N, K, B, d, pattern):
    # values that no parts hold, at the edges of groups and 256-index blocks, in the weights and
    # in X: added once, over the stored entries alone, and the entries beside them as exact as ever
    W, dense, rp, ci, X, dY = layer(N, K, B, d, seed=N, pattern=pattern)
    assert L1.workspace_bytes(L1.OP_SPMM_PACKED, N, K, W.nnz, B) > 0
    v = h(W.vals).copy()
    v[rp[31]], v[rp[32]], v[rp[N] - 1], v[rp[N // 2] + 3] = 2.0 ** 30, -(2.0 ** 29), 2.0 ** 35, 2.0 ** 31
    W.vals.copy_(t(v))
    rows = np.repeat(np.arange(N), np.diff(rp))
    dense[rows, ci] = v
    for k, b in [(0, 0), (255, 31), (256, 32), (K - 1, B - 1), (K // 3, 127), (512, 128), (K // 2, 64)]:
        X[k, b] = 2.0 ** 30
    X[257, 5], X[K - 2, B // 2] = np.inf, -np.inf
    x = np.where(np.isfinite(X), X, 0).astype(np.float64)
    ref, m = dense @ x, np.abs(dense) @ np.abs(x)
    for k, b in [(257, 5), (K - 2, B // 2)]:
        st = dense[:, k] != 0
        ref[st, b] = np.sign(dense[st, k]) * X[k, b]
    got = h(L1.csr_spmm_fwd(W, t(X))).astype(np.float64)
    ok = np.isfinite(ref)
    assert not np.isnan(got).any() and np.array_equal(got[~ok], ref[~ok])
    assert (np.abs(got[ok] - ref[ok]) <= (bound(6 * K) + K * 2.0 ** -24) * m[ok]).all()


def test_flagged_blocks_cost_little():
    # one infinity is the work of its own block: the call takes no multiple of its time
    import torch
    N, K, B = 4096, 4096, 512
    W, _, _, _, X, _ = layer(N, K, B, 0.2, seed=1)
    Xd, Y = t(X), torch.empty((N, B), device="cuda")

    def us():
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            L1.csr_spmm_fwd(W, Xd, Y)
            b.record()
            torch.cuda.synchronize()
            times.append(1e3 * a.elapsed_time(b))
        return min(times)

    us()
    plain = us()
    Xd[K // 2, B // 2] = float("inf")
    assert us() < 6 * plain


def test_plain_workspace_gives_the_planned_bits():
    # nearly full: the packed operands fit the tiled kernel's workspace, which still takes that kernel
    import torch
    N, K, B = 2048, 2048, 512
    W, dense, rp, ci, X, dY = layer(N, K, B, 0.9, seed=4)
    n = L1.workspace_bytes(L1.OP_SPMM, N, K, W.nnz, B)
    assert 0 < n < L1.workspace_bytes(L1.OP_SPMM_PACKED, N, K, W.nnz, B)
    Xd, s = t(X), torch.cuda.current_stream().cuda_stream
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    Y = [torch.empty((N, B), device="cuda") for _ in range(2)]
    a = (N, K, W.nnz, W.row_ptr.data_ptr(), W.col_idx.data_ptr(), W.vals.data_ptr())
    assert L1.lib().csr_spmm_fwd(*a, Xd.data_ptr(), B, B, Y[0].data_ptr(), B, ws.data_ptr(), n, s) == L1.OK
    assert L1.lib().csr_spmm_plan(*a, B, ws.data_ptr(), n, s) == L1.OK
    assert L1.lib().csr_spmm_planned(*a, Xd.data_ptr(), B, B, Y[1].data_ptr(), B, ws.data_ptr(), n, s) == L1.OK
    assert bits_equal(h(Y[0]), h(Y[1]))


def test_packed_workspace_is_given_back_and_can_be_refused(monkeypatch):
    import torch
    N, K, B = 1024, 1024, 384
    W, dense, rp, ci, X, dY = layer(N, K, B, 0.4, seed=6)
    Xd, dYd = t(X), t(dY)
    big = L1.workspace_bytes(L1.OP_SPMM_PACKED, N, K, W.nnz, B)
    packed = h(L1.csr_spmm_fwd(W, Xd))
    # beyond the bound no buffer outlives its call
    monkeypatch.setattr(L1, "_ws_cache", {})
    monkeypatch.setattr(L1, "_WS_KEEP", big - 1)
    assert bits_equal(h(L1.csr_spmm_fwd(W, Xd)), packed)
    L1.dense_wgrad(dYd, Xd)
    assert all(b.numel() < big for b in L1._ws_cache.values())
    # and where there is no memory for one, the calls run without it
    real = L1._empty_bytes

    def scarce(nbytes, device, stream):
        if nbytes >= (1 << 20):
            raise torch.OutOfMemoryError("no memory for packed operands")
        return real(nbytes, device, stream)

    monkeypatch.setattr(L1, "_ws_cache", {})
    monkeypatch.setattr(L1, "_empty_bytes", scarce)
    plain = L1.workspace_bytes(L1.OP_SPMM, N, K, W.nnz, B)
    if plain < (1 << 20):
        Y = h(L1.csr_spmm_fwd(W, Xd))
        assert (np.abs(Y - dense @ X) <= bound(6 * K) * (np.abs(dense) @ np.abs(X))).all()
    G = h(L1.dense_wgrad(dYd, Xd, precision=L1.BF16X3)).astype(np.float64)
    ref, m = dY.astype(np.float64) @ X.T.astype(np.float64), np.abs(dY).astype(np.float64) @ X.T
    assert (np.abs(G - ref) <= 1e-4 * m).all()


def test_captured_planned_product_keeps_its_memory():
    # a graph of a planned product, replayed after a larger call on its stream: neither
    # does the replay write to memory that was handed on, nor the other way round
    import torch
    N, K, B = 1024, 1024, 384
    W, dense, rp, ci, X, dY = layer(N, K, B, 0.4, seed=6)
    W2, _, _, _, X2, _ = layer(2048, 2305, 384, 0.4, seed=7)
    need = L1.workspace_bytes(L1.OP_SPMM_PACKED, N, K, W.nnz, B)
    assert 0 < need < L1.workspace_bytes(L1.OP_SPMM_PACKED, 2048, 2305, W2.nnz, B)
    Xd, X2d = t(X), t(X2)
    Y = torch.empty((N, B), device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        plan = L1.csr_spmm_plan(W, B)
        L1.csr_spmm_planned(W, Xd, plan, Y)
        want = Y.clone()
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        L1.csr_spmm_planned(W, Xd, plan, Y)
    with torch.cuda.stream(s):
        L1.csr_spmm_fwd(W2, X2d)
        others = [torch.full((need,), 7, dtype=torch.uint8, device="cuda") for _ in range(4)]
        for _ in range(3):
            Y.zero_()
            g.replay()
            assert torch.equal(Y, want)
            assert all(bool((o == 7).all()) for o in others)
            for o in others:
                o.fill_(7)
    s.synchronize()


def test_packed_products_take_all_six_terms():
    # one stored value meets one nonzero of X: exact only with each of the six part products
    N, K, B = 1024, 2048, 256
    W, dense, rp, ci, X, dY = layer(N, K, B, 0.4, seed=11)
    assert min(L1.workspace_bytes(op, N, K, W.nnz, B) for op in (L1.OP_SPMM_PACKED, L1.OP_SDDMM_PACKED)) > 0
    hi, mid, lo = 1.0, 1 + 2.0 ** -9, 1 + 2.0 ** -9 + 2.0 ** -18
    v, x = np.zeros(len(ci), np.float32), np.zeros((K, B), np.float32)
    dy, xg = np.zeros((N, B), np.float32), np.zeros((K, B), np.float32)
    want, wantg = np.zeros((N, B)), np.zeros(len(ci))
    for n, (a, b) in enumerate([(hi, hi), (mid, hi), (hi, mid), (mid, mid), (lo, hi), (hi, lo)]):
        i, col = 150 * n + 1, 40 * n + 7  # (row 341 is empty)
        p = rp[i] + 30 * n + 2  # this row's value stands alone in its column of X and of the batch
        v[p], x[ci[p], col], want[i, col] = a, b, a * b
        dy[i, col], xg[ci[p], col], wantg[p] = a, b, a * b
    assert np.count_nonzero(x) == 6
    W.vals.copy_(t(v))
    assert np.array_equal(h(L1.csr_spmm_fwd(W, t(x))), want.astype(np.float32))
    assert np.array_equal(h(L1.sddmm_masked_wgrad(W, t(dy), t(xg)))[:W.nnz], wantg.astype(np.float32))
