"""GPU: the weight gradient from packed bf16 parts (dense_wgrad / dense_wgrad_prox
with the packed workspace) against 64-bit references, at tile edges, ragged
sizes, split reductions and operands outside the parts' range."""
import numpy as np
import pytest

import paper_1905_07931_amd as L1
from _helpers import bits_equal, h, t

pytestmark = pytest.mark.gpu


def operands(N, K, B, seed=0, pad=0):
    rng = np.random.default_rng(seed)
    dY = rng.standard_normal((N, B + pad)).astype(np.float32)
    X = rng.random((K, B + pad)).astype(np.float32)
    return dY, X


def bound(B, prec):
    """|error| / sum |a b|: the terms left out (2^-22 with three parts, 3 (1 + 2^-7) 2^-16 with
    two) and an fp32 rounding per instruction and per product inside one."""
    terms = 6 if prec == L1.F32 else 3
    left_out = 2.0 ** -22 if prec == L1.F32 else 3 * (1 + 2.0 ** -7) * 2.0 ** -16
    return left_out + (terms * (-(-B // 16)) + 16 + 64) * 2.0 ** -24


# one tile exactly, one row / column / index past tiles and steps, less than a
# tile, a partial last band of tile rows, split reductions (B >= 512) of 24, 2 and,
# on both sides of the last split, 128 and 129 tiles
@pytest.mark.parametrize("N,K,B,pad", [(128, 128, 160, 0), (129, 257, 161, 0), (127, 1, 175, 3), (1, 300, 320, 0),
                                       (1153, 2177, 333, 0), (2049, 2100, 97, 1), (300, 1000, 1024, 0),
                                       (65, 129, 4097, 2), (1100, 1300, 777, 0),
                                       (1024, 2048, 515, 0), (300, 5500, 516, 1)])
@pytest.mark.parametrize("prec", [L1.F32, L1.BF16X3])
def test_packed_wgrad(N, K, B, pad, prec):
    dYh, Xh = operands(N, K, B, seed=N + K + B, pad=pad)
    dY, X = t(dYh)[:, :B], t(Xh)[:, :B]
    assert L1.workspace_bytes(L1.OP_WGRAD_PACKED, N, K, 0, B) > 0
    got = h(L1.dense_wgrad(dY, X, precision=prec)).astype(np.float64)
    a, x = dYh[:, :B].astype(np.float64), Xh[:, :B].astype(np.float64)
    err = np.abs(got - a @ x.T)
    assert (err <= bound(B, prec) * (np.abs(a) @ np.abs(x).T)).all()
    # that bound holds for two parts as well: three are some ten times closer (2-norm)
    rel = np.linalg.norm(got - a @ x.T) / np.linalg.norm(a @ x.T)
    assert rel <= 8e-7 if prec == L1.F32 else rel <= 2e-5


def test_packed_wgrad_takes_all_six_products():
    # one batch index meets one: the entry is exact only with each of hi hi, hi mid, mid hi, mid
    # mid, hi lo and lo hi
    N, K, B = 130, 260, 322
    hi, mid, lo = 1.0, 1 + 2.0 ** -9, 1 + 2.0 ** -9 + 2.0 ** -18  # of 1, 2 and 3 parts
    dYh, Xh = np.zeros((N, B), np.float32), np.zeros((K, B), np.float32)
    for b, a, x in [(3, hi, hi), (40, mid, hi), (70, hi, mid), (255, mid, mid), (256, lo, hi), (321, hi, lo)]:
        dYh[b % N, b], Xh[b % K, b] = a, x
    got = h(L1.dense_wgrad(t(dYh), t(Xh)))
    assert np.array_equal(got, (dYh.astype(np.float64) @ Xh.astype(np.float64).T).astype(np.float32))
    assert got[255 % N, 255 % K] == np.float32(mid * mid) and got[256 % N, 256 % K] == np.float32(lo)


def test_packed_is_deterministic_and_needs_its_workspace():
    N, K, B = 300, 1000, 1024
    dY, X = (t(v) for v in operands(N, K, B))
    assert bits_equal(h(L1.dense_wgrad(dY, X)), h(L1.dense_wgrad(dY, X)))
    # a workspace of the older size is still taken: the fp32 tiles
    import ctypes as C
    import torch
    need = L1.workspace_bytes(L1.OP_DENSE_WGRAD, N, K, 0, B)
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    dW = torch.empty((N, K), device="cuda")
    rc = L1.lib().dense_wgrad(N, K, B, C.c_void_p(dY.data_ptr()), B, C.c_void_p(X.data_ptr()), B,
                              C.c_void_p(dW.data_ptr()), K, L1.F32, C.c_void_p(ws.data_ptr()), need,
                              C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == L1.OK
    ref = h(dY).astype(np.float64) @ h(X).astype(np.float64).T
    assert np.abs(h(dW) - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("scale_a,scale_x", [(2.0 ** -95, 2.0 ** 20), (2.0 ** -112, 2.0 ** 40), (2.0 ** 75, 2.0 ** -40)])
def test_packed_wgrad_scales(scale_a, scale_x):
    # inside the parts' range, below it and above it: the error stays relative to the products
    N, K, B = 200, 300, 320
    dYh, Xh = operands(N, K, B, seed=3)
    dYh *= np.float32(scale_a)
    Xh *= np.float32(scale_x)
    got = h(L1.dense_wgrad(t(dYh), t(Xh))).astype(np.float64)
    a, x = dYh.astype(np.float64), Xh.astype(np.float64)
    assert (np.abs(got - a @ x.T) <= (2.0 ** -22 + B * 2.0 ** -24) * (np.abs(a) @ np.abs(x).T)).all()


@pytest.mark.parametrize("prec", [L1.F32, L1.BF16X3])
def test_packed_wgrad_small_beside_large(prec):
    # every row of dY holds normal values and others some 2^-80 to 2^-145 (down to subnormals
    # of a few bits) that alone meet nonzeros of X: the error stays relative to their products
    N, K, B = 130, 260, 322
    dYh, Xh = operands(N, K, B, seed=8)
    dYh[:, 1::2] *= np.exp2(-np.linspace(80, 145, N))[:, None].astype(np.float32)
    Xh[:, 0::2] = 0
    Xh[:, 1::2] *= np.float32(2.0 ** 27)
    got = h(L1.dense_wgrad(t(dYh), t(Xh), precision=prec)).astype(np.float64)
    a, x = dYh.astype(np.float64), Xh.astype(np.float64)
    assert (np.abs(got - a @ x.T) <= bound(B, prec) * (np.abs(a) @ np.abs(x).T)).all()


@pytest.mark.parametrize("prec", [L1.F32, L1.BF16X3])
def test_packed_wgrad_nonfinite(prec):
    # infinities and NaN reach exactly the entries that multiply them
    N, K, B = 260, 390, 322
    dYh, Xh = operands(N, K, B, seed=5)
    dYh[7, 11], dYh[200, 300], Xh[5, 3] = np.inf, -np.inf, np.nan
    dYh[31, 40] = 3.4e38  # hi would round to infinity
    Xh[9, 11] = 0.0       # inf * 0
    got = h(L1.dense_wgrad(t(dYh), t(Xh), precision=prec))
    with np.errstate(invalid="ignore", over="ignore"):
        a, x = dYh.astype(np.float64), Xh.astype(np.float64)
        # column by column: a BLAS product may spread NaN
        ref = np.stack([(a * x[k]).sum(axis=1) for k in range(K)], axis=1).astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    m = np.abs(np.where(np.isfinite(a), a, 0)) @ np.abs(np.where(np.isfinite(x), x, 0)).T
    assert (np.abs(got[ok] - ref[ok].astype(np.float64)) <= 1e-4 * m[ok]).all()


@pytest.mark.parametrize("N,K,B,pad", [(129, 257, 161, 0), (300, 1000, 1024, 0), (65, 129, 4097, 2), (300, 5500, 516, 1)])
def test_packed_wgrad_flagged_blocks(N, K, B, pad):
    # values that no parts hold at the edges of groups and 256-index blocks: added once, and
    # the entries beside them as exact as ever
    if B < 320 or not L1.workspace_bytes(L1.OP_WGRAD_PACKED, N, K, 0, B):
        precs = [L1.F32]
    else:
        precs = [L1.F32, L1.BF16X3]
    dYh, Xh = operands(N, K, B, seed=N, pad=pad)
    for i, b in [(0, 0), (31, min(255, B - 1)), (32, min(256, B - 1)), (N - 1, B - 1), (N // 2, B // 2)]:
        dYh[i, b] = 2.0 ** 30
    for k, b in [(K - 1, 0), (K // 2, B - 1), (32, B // 2), (127, 31), (128, 32)]:
        Xh[k, b] = -(2.0 ** 40)
    Xh[K // 3, 5], dYh[N // 3, 7] = np.inf, -np.inf
    a, x = dYh[:, :B].astype(np.float64), Xh[:, :B].astype(np.float64)
    fa, fx = np.where(np.isfinite(a), a, 0), np.where(np.isfinite(x), x, 0)
    ref = fa @ fx.T
    ref[:, K // 3] = np.sign(a[:, 5]) * np.inf
    ref[N // 3, :] = -np.inf
    ref[N // 3, K // 3] = -np.inf if a[N // 3, 5] < 0 else np.nan
    for prec in precs:
        got = h(L1.dense_wgrad(t(dYh)[:, :B], t(Xh)[:, :B], precision=prec)).astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        ok = np.isfinite(ref)
        assert (np.abs(got[ok] - ref[ok]) <= (bound(B, prec) + 2 * B / 16 * 2.0 ** -24) * (np.abs(fa) @ np.abs(fx).T)[ok]).all()


@pytest.mark.parametrize("N,K,B", [(1153, 2177, 333), (300, 1000, 1024), (300, 5500, 516)])
@pytest.mark.parametrize("prec", [L1.F32, L1.BF16X3])
def test_packed_prox_equals_the_calls(N, K, B, prec):
    # the fused update and dense_wgrad + prox_l1_recompress: the same bits
    rng = np.random.default_rng(1)
    mask = rng.random((N, K)) < 0.1
    rp = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    ci = np.nonzero(mask)[1].astype(np.int32)
    W = L1.CSR.from_host(rp, ci, rng.standard_normal(len(ci)).astype(np.float32), K)
    dY, X = (t(v) for v in operands(N, K, B, seed=2))
    lam = float(np.sqrt(B / 3.0))
    Z, out = L1.dense_wgrad_prox_recompress(W, dY, X, 0.01, lam, precision=prec)
    ref = L1.prox_l1_recompress(W, L1.dense_wgrad(dY, X, precision=prec), 0.01, lam)
    for a, b in zip(out.to_host(), ref.to_host()):
        assert bits_equal(a, b)
