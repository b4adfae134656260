"""GPU: the wave-per-position convolution kernels at the batches where their lane
mapping changes (64 lanes x 1, 2 or 4 floats, partly filled), odd position counts,
strides and padding, channels without entries and past one staging pass, against
64-bit references; a one-image slice of the batch (the thread-per-output kernels)
gives the same bits."""
import numpy as np
import pytest

import paper_1905_07931_amd as L1
from _helpers import bits_equal, h, t

pytestmark = pytest.mark.gpu


def reference(g, w, X, dY):
    """Forward and input gradient in float64, entry by entry."""
    n, (OH, OW) = w.shape[0], g.out_hw
    B = X.shape[1]
    x = np.zeros((g.C, g.H + 2 * g.PH, g.W + 2 * g.PW, B))
    x[:, g.PH:g.PH + g.H, g.PW:g.PW + g.W] = X.reshape(g.C, g.H, g.W, B)
    d = dY.reshape(n, OH * OW * B)
    y, dx = np.zeros((n, OH * OW * B)), np.zeros_like(x)
    k = 0
    for c in range(g.C):
        for i in range(g.KH):
            for j in range(g.KW):
                win = (c, slice(i, i + g.SH * (OH - 1) + 1, g.SH), slice(j, j + g.SW * (OW - 1) + 1, g.SW))
                y += np.outer(w[:, k], x[win].reshape(-1))
                dx[win] += (w[:, k] @ d).reshape(OH, OW, B)
                k += 1
    return y.reshape(-1, B), dx[:, g.PH:g.PH + g.H, g.PW:g.PW + g.W].reshape(-1, B)


@pytest.mark.parametrize("B", [47, 48, 64, 71, 96, 129, 192, 250, 256, 260])
@pytest.mark.parametrize("geom", [(3, 7, 9, 3, 3, 1, 1, 0, 0), (2, 9, 8, 5, 3, 2, 1, 2, 1), (4, 5, 5, 5, 5, 1, 1, 0, 0)])
def test_conv_wave(B, geom):
    g = L1.ConvGeom(*geom)
    n, K = 7, g.filter_cols
    rng = np.random.default_rng(B + K)
    mask = rng.random((n, K)) < 0.4
    mask[2] = False
    mask[:, 0:g.KH * g.KW] = False  # an input channel without entries
    rp = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    ci = np.nonzero(mask)[1].astype(np.int32)
    v = rng.standard_normal(len(ci)).astype(np.float32)
    dense = np.zeros((n, K))
    dense[np.nonzero(mask)] = v
    OH, OW = g.out_hw
    X, dY = rng.random((g.in_rows, B)).astype(np.float32), rng.standard_normal((n * OH * OW, B)).astype(np.float32)
    W = L1.CSR.from_host(rp, ci, v, K)
    csc = L1.csc_build(W)
    Y = h(L1.csr_conv_fwd(g, W, t(X)))
    dX = h(L1.csr_conv_bwd_data(g, n, csc, t(dY), nnz=W.nnz))
    y, dx = reference(g, dense, X.astype(np.float64), dY.astype(np.float64))
    my, mdx = reference(g, np.abs(dense), np.abs(X).astype(np.float64), np.abs(dY).astype(np.float64))
    assert (np.abs(Y - y) <= K * 2.0 ** -24 * my).all()
    assert (np.abs(dX - dx) <= n * g.KH * g.KW * 2.0 ** -24 * mdx).all()
    assert bits_equal(h(L1.csr_conv_fwd(g, W, t(X[:, :1]))), Y[:, :1].copy())
    assert bits_equal(h(L1.csr_conv_bwd_data(g, n, csc, t(dY[:, :1]), nnz=W.nnz)), dX[:, :1].copy())


def test_conv_wave_many_entries():
    # more entries per channel than one staging pass (2048) holds
    g = L1.ConvGeom(250, 4, 4, 3, 3)
    n, K, B = 3, g.filter_cols, 64
    rng = np.random.default_rng(0)
    w = rng.standard_normal((n, K)).astype(np.float32)
    W = L1.CSR.from_host((np.arange(n + 1) * K).astype(np.int32), np.tile(np.arange(K, dtype=np.int32), n), w.reshape(-1), K)
    X = rng.random((g.in_rows, B + 1)).astype(np.float32)
    dY = rng.standard_normal((n * 4, B + 1)).astype(np.float32)
    Y = h(L1.csr_conv_fwd(g, W, t(X)))
    y, _ = reference(g, w.astype(np.float64), X.astype(np.float64), dY.astype(np.float64))
    my, _ = reference(g, np.abs(w).astype(np.float64), X.astype(np.float64), dY.astype(np.float64))
    assert (np.abs(Y - y) <= K * 2.0 ** -24 * my).all()
    g2 = L1.ConvGeom(2, 6, 6, 5, 5)  # backward: 100 output channels x 25 positions per input channel
    n2 = 100
    w2 = rng.standard_normal((n2, g2.filter_cols)).astype(np.float32)
    W2 = L1.CSR.from_host((np.arange(n2 + 1) * g2.filter_cols).astype(np.int32),
                          np.tile(np.arange(g2.filter_cols, dtype=np.int32), n2), w2.reshape(-1), g2.filter_cols)
    d2 = rng.standard_normal((n2 * 4, 96)).astype(np.float32)
    x2 = np.zeros((g2.in_rows, 96))
    dX = h(L1.csr_conv_bwd_data(g2, n2, L1.csc_build(W2), t(d2), nnz=W2.nnz))
    _, dx = reference(g2, w2.astype(np.float64), x2, d2.astype(np.float64))
    _, mdx = reference(g2, np.abs(w2).astype(np.float64), x2, np.abs(d2).astype(np.float64))
    assert (np.abs(dX - dx) <= n2 * 25 * 2.0 ** -24 * mdx).all()


@pytest.mark.parametrize("geom,n,B", [((52, 11, 11, 1, 1, 1, 1, 0, 0), 7, 1000), ((42, 13, 11, 3, 3, 2, 1, 1, 1), 9, 1020),
                                      ((400, 5, 3, 1, 1, 1, 1, 0, 0), 1, 1024)])
def test_conv_wave_mapped_slices(geom, n, B):
    # inputs beyond 24 MB: the (channel, slice) items are dealt to the XCDs by slice; counts of
    # slices and channels that are no multiple of 8, fewer slices than XCDs
    g = L1.ConvGeom(*geom)
    assert g.in_rows * B * 4 > 24e6
    rng = np.random.default_rng(n)
    dense = rng.standard_normal((n, g.filter_cols)) * (rng.random((n, g.filter_cols)) < 0.3)
    dense = dense.astype(np.float32).astype(np.float64)
    rp = np.concatenate([[0], np.cumsum((dense != 0).sum(1))]).astype(np.int32)
    ci = np.nonzero(dense)[1].astype(np.int32)
    W = L1.CSR.from_host(rp, ci, dense[dense != 0].astype(np.float32), g.filter_cols)
    OH, OW = g.out_hw
    X = rng.random((g.in_rows, B)).astype(np.float32)
    none = np.zeros((n * OH * OW, B))
    y, _ = reference(g, dense, X.astype(np.float64), none)
    my, _ = reference(g, np.abs(dense), X.astype(np.float64), none)
    import torch
    Y = torch.full((n * OH * OW, B + 4), 3.0, device="cuda")
    L1.csr_conv_fwd(g, W, t(X), Y[:, :B])
    assert (np.abs(h(Y)[:, :B] - y) <= g.filter_cols * 2.0 ** -24 * my).all() and bool((Y[:, B:] == 3.0).all())


@pytest.mark.parametrize("geom,B,density", [((8, 40, 40, 1, 1, 1, 1, 0, 0), 48, 0.3), ((8, 40, 40, 1, 1, 1, 1, 0, 0), 64, 0.3),
                                            ((12, 40, 41, 1, 1, 2, 1, 0, 0), 64, 0.3), ((8, 13, 11, 2, 2, 1, 1, 1, 0), 48, 0.6),
                                            ((8, 40, 40, 1, 1, 1, 1, 0, 0), 47, 0.3), ((8, 40, 40, 1, 1, 1, 1, 0, 0), 96, 0.3),
                                            ((8, 40, 40, 1, 1, 1, 1, 0, 0), 116, 0.3), ((8, 40, 40, 1, 1, 1, 1, 0, 0), 336, 0.3),
                                            ((12, 40, 41, 1, 1, 2, 1, 0, 0), 100, 0.3), ((8, 40, 40, 1, 1, 1, 1, 0, 0), 352, 0.2),
                                            ((8, 40, 40, 1, 1, 1, 1, 0, 0), 98, 0.3)])
def test_conv_backward_few_entries(geom, B, density):
    # batches that leave lanes idle, few entries a channel and many positions: a thread per output (four
    # batch columns), beside sizes on the wave's side of the line and a batch that has no vectors
    g = L1.ConvGeom(*geom)
    n = 9
    rng = np.random.default_rng(B)
    dense = (rng.standard_normal((n, g.filter_cols)) * (rng.random((n, g.filter_cols)) < density)).astype(np.float32)
    rp = np.concatenate([[0], np.cumsum((dense != 0).sum(1))]).astype(np.int32)
    W = L1.CSR.from_host(rp, np.nonzero(dense)[1].astype(np.int32), dense[dense != 0], g.filter_cols)
    OH, OW = g.out_hw
    dY = rng.standard_normal((n * OH * OW, B)).astype(np.float32)
    none = np.zeros((g.in_rows, B))
    _, dx = reference(g, dense.astype(np.float64), none, dY.astype(np.float64))
    _, m = reference(g, np.abs(dense).astype(np.float64), none, np.abs(dY).astype(np.float64))
    dX = h(L1.csr_conv_bwd_data(g, n, L1.csc_build(W), t(dY), nnz=W.nnz))
    assert (np.abs(dX - dx) <= n * g.KH * g.KW * 2.0 ** -24 * m).all()
