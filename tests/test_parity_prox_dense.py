"""GPU: prox_adaptive_recompress with the dense result kept in the workspace gives
the bits of the two-pass route (a workspace without room for it): W', m', v' at
slab and word remainders, with more rows than the compaction prefixes itself,
views whose rows are not 16-byte aligned, NaN and infinite gradients, and a
result without a nonzero."""
import numpy as np
import pytest

import paper_1905_07931_amd as L1
from _helpers import bits_equal, h, t

pytestmark = pytest.mark.gpu


def run(solver, N, K, G, m, v, W, lam, pad):
    import torch
    def mat(a):
        full = torch.full((N, K + pad), 7.0, device="cuda")
        full[:, :K] = t(a)
        return full[:, :K]
    st = L1.AdaptiveState(solver, mat(v), mat(m) if solver == L1.SOLVER_ADAM else None, t=3)
    out = L1.CSR(N, K, torch.zeros(N + 1, dtype=torch.int32, device="cuda"),
                 torch.full((N * K,), -1, dtype=torch.int32, device="cuda"), torch.full((N * K,), 9.0, device="cuda"), None)
    out = L1.prox_adaptive_recompress(W, mat(G), st, 1e-2, lam, out=out)
    states = [h(st.v)] + ([h(st.m)] if solver == L1.SOLVER_ADAM else [])
    return [h(out.row_ptr), h(out.col_idx), h(out.vals)] + states, out.validate_shapes()


@pytest.mark.parametrize("solver", [L1.SOLVER_RMSPROP, L1.SOLVER_ADAM])
@pytest.mark.parametrize("N,K,lam,pad", [
    (1, 1, 1e-3, 0), (3, 31, 1e-3, 0), (5, 33, 1.0, 1), (7, 1025, 0.5, 3), (130, 4099, 0.5, 0),
    (64, 4100, 0.0, 4), (9, 9000, 1e6, 0), (16500, 70, 0.5, 2), (257, 2048, 0.5, 0)])
def test_bits_of_the_two_passes(solver, N, K, lam, pad, monkeypatch):
    rng = np.random.default_rng(N * 7 + K)
    dense = (rng.standard_normal((N, K)) * 0.05 * (rng.random((N, K)) < 0.2)).astype(np.float32)
    rows, cols = np.nonzero(dense)
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=N))]).astype(np.int32)
    W = L1.CSR.from_host(rp, cols.astype(np.int32), dense[rows, cols], K)
    G = rng.standard_normal((N, K)).astype(np.float32)
    if N > 100:
        G[3, 5], G[4, K - 1], G[N - 1, 0] = np.nan, np.inf, -np.inf
    m, v = G * np.float32(0.3), rng.random((N, K)).astype(np.float32)
    kept, nnz = run(solver, N, K, G, m, v, W, lam, pad)
    real = L1.workspace_bytes
    asked = []
    def without(op, *a):
        asked.append(op)
        return 0 if op == L1.OP_PROX_DENSE else real(op, *a)
    monkeypatch.setattr(L1, "workspace_bytes", without)
    two, nnz2 = run(solver, N, K, G, m, v, W, lam, pad)
    assert L1.OP_PROX_DENSE in asked and nnz == nnz2 == kept[0][-1]
    for a, b in zip(kept, two):
        assert bits_equal(a, b)
