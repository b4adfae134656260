"""GPU: the row kernel's long rows (beyond 256 entries and a share of their layer's
mean length, taken by workgroups of their own) around that length, with more of them
than one LDS list holds, in every slice of the search, among empty rows, past the row
count that is searched, at batches on both sides of each vector width, against 64-bit
references and run to run."""
import numpy as np
import pytest

import paper_1905_07931_amd as L1
from _helpers import bits_equal, h, t

pytestmark = pytest.mark.gpu


def check(lengths, K, B, seed):
    rng = np.random.default_rng(seed)
    lengths = np.asarray(lengths)
    rp = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(K, n, replace=False)) for n in lengths] or [[]]).astype(np.int32)
    v = rng.standard_normal(len(ci)).astype(np.float32)
    X = rng.random((K, B)).astype(np.float32)
    N = len(lengths)
    W = L1.CSR.from_host(rp, ci, v, K)
    Xd = t(X)
    import ctypes as C
    import torch
    Y = torch.full((N, B + 1), 5.0, device="cuda")  # without a workspace: the row kernel
    rc = L1.lib().csr_spmm_fwd(N, K, W.nnz, W.row_ptr.data_ptr(), W.col_idx.data_ptr(), W.vals.data_ptr(), Xd.data_ptr(),
                               B, B, Y.data_ptr(), B + 1, None, 0, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == L1.OK
    got = h(Y)
    assert (got[:, B] == 5.0).all()
    rows = np.repeat(np.arange(N), lengths)
    ref, m = np.zeros((N, B)), np.zeros((N, B))
    np.add.at(ref, rows, v[:, None].astype(np.float64) * X[ci])
    np.add.at(m, rows, np.abs(v)[:, None].astype(np.float64) * X[ci])
    bound = (lengths[:, None] + 4) * 2.0 ** -24 * m
    assert (np.abs(got[:, :B] - ref) <= bound).all()
    Z = torch.empty((N, B + 1), device="cuda")
    L1.lib().csr_spmm_fwd(N, K, W.nnz, W.row_ptr.data_ptr(), W.col_idx.data_ptr(), W.vals.data_ptr(), Xd.data_ptr(), B, B,
                          Z.data_ptr(), B + 1, None, 0, C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert bits_equal(h(Z)[:, :B].copy(), got[:, :B].copy())


@pytest.mark.parametrize("B", [1, 33, 64, 65, 128, 132, 260])
def test_lengths_around_the_split(B):
    check([0, 255, 256, 257, 1, 300, 0, 1000, 64, 8, 9, 320, 259], 1000, B, B)


def test_more_long_rows_than_a_list():
    check([257] * 2100 + [3] * 5, 300, 7, 1)


def test_one_long_row_among_many():
    check([0] * 1500 + [2000] + [1] * 1500, 2000, 96, 2)


def test_past_the_scanned_rows():
    n = np.zeros(32769, np.int64)
    n[[0, 7, 32768]] = [300, 1, 270]
    check(n, 300, 3, 3)


@pytest.mark.parametrize("B", [64, 100])
def test_even_rows_keep_a_wave(B):
    # many rows of some 300 entries: only the one past their mean by half is split
    check([300] * 1500 + [440, 0, 455, 1000, 256, 257] + [290] * 900, 1000, B, B)


def test_few_rows_around_their_mean():
    # 12 rows, mean 400: the line lies at 300 entries
    check([299, 300, 301, 257, 400, 480, 500, 460, 440, 463, 500, 400], 600, 40, 6)


@pytest.mark.parametrize("N", [859, 860, 900, 1093, 1094])
def test_rows_between_the_lines(N):
    # N * 128 columns on both sides of 110,000 and 140,000, a mean of about 290: 9/8 of it and 16 between
    rng = np.random.default_rng(N)
    n = rng.integers(255, 300, N)
    n[::29] = rng.integers(320, 360, len(n[::29]))
    n[::97] = 700
    check(n, 900, 128, N)


@pytest.mark.parametrize("N,B", [(n, 5) for n in (2047, 2048, 2049, 2081, 8192, 8193, 8225, 20000, 32768)] +
                         [(n, b) for n in (2049, 2081, 4095, 4096, 4097, 4129, 8192) for b in (257, 260)] + [(8193, 257)])
def test_long_rows_in_every_slice(N, B):
    # the rows are looked at in slices of 32 (of every 256 from 2049 rows, of every 512 from 8193; past 256
    # columns of every 64 from 2049, of every 128 from 4097): long ones at the slices' edges, and in the
    # last, partial, one
    n = np.zeros(N, np.int64)
    n[np.unique(np.concatenate([np.arange(0, N, 32 * 7), np.arange(31, N, 32 * 7), np.arange(224, N, 256),
                                np.arange(480, N, 512), [N - 1, N - 2]]))] = 260
    n[::97] = 257
    n[5] = 256
    check(n, 300, B, N)
