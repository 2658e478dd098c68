"""CholeskyQR2 at the edges of its blocks: 64-column diagonal blocks, the 32 x
32 tiles behind them, 16-row solves, the last block ragged, and the columns
(1024) up to which the rows of a solve stay in LDS.

Tolerance: |Q^T Q - I| <= 4 p u, the dot products of p terms on either side
with room, at least 1e-14; the same, relative, for what of Y lies outside Q.
"""
import ctypes

import numpy as np
import pytest

import paper_2410_19747_amd as T

pytestmark = pytest.mark.gpu


def _cholqr2(Y):
    import torch

    L = T.lib()
    p, l = Y.shape
    d = torch.from_numpy(np.ascontiguousarray(Y.T)).cuda()  # column-major
    guard = torch.full((64,), float("nan"), dtype=torch.float64, device="cuda")
    ws = torch.full((int(L.ttm_test_cholqr2_ws_bytes(p, l)) // 8 + 1,), float("nan"), dtype=torch.float64,
                    device="cuda")
    down = ctypes.c_int(-1)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = L.ttm_test_cholqr2(ptr(d), p, l, ctypes.byref(down), ptr(ws), ws.numel() * 8, None)
    assert rc == 0, rc
    assert torch.isnan(guard).all()
    return d.cpu().numpy().T, down.value


@pytest.mark.parametrize("p,l", [(1, 1), (17, 1), (15, 15), (63, 63), (80, 65), (97, 96), (128, 127), (129, 128),
                                 (130, 129), (300, 257), (520, 511), (513, 513), (1040, 1024), (1050, 1025)])
def test_orthonormal_at_block_edges(p, l):
    print("cholqr2 %dx%d" % (p, l), flush=True)
    rng = np.random.default_rng(1000 * p + l)
    Y = rng.standard_normal((p, l))
    if p < 4 * l:  # a square Gaussian matrix may be ill conditioned: cond 100
        u, _, vt = np.linalg.svd(Y, full_matrices=False)
        Y = (u * np.geomspace(1.0, 0.01, l)) @ vt
    Q, down = _cholqr2(Y)
    assert down == 0
    tol = max(1e-14, 4 * p * 2.0 ** -53)
    assert np.abs(Q.T @ Q - np.eye(l)).max() <= tol
    assert np.linalg.norm(Y - Q @ (Q.T @ Y)) <= tol * np.linalg.norm(Y)


@pytest.mark.parametrize("l,copy", [(2, 1), (64, 60), (64, 61), (64, 62), (64, 63), (65, 64), (128, 125), (200, 199)])
def test_breakdown_is_seen_in_every_pivot(l, copy):
    """A column that repeats the first: the pivot that vanishes is its own."""
    print("cholqr2 breakdown %d %d" % (l, copy), flush=True)
    rng = np.random.default_rng(l + copy)
    Y = rng.standard_normal((4 * l, l))
    Y[:, copy] = Y[:, 0]
    Q, down = _cholqr2(Y)
    assert down == 1
    assert np.isfinite(Q).all()


@pytest.mark.parametrize("l,rank", [(64, 3), (128, 40), (300, 20)])
def test_breakdown_stays_finite(l, rank):
    """Most pivots vanish: every one of them is replaced, and none makes the
    rows behind it grow."""
    print("cholqr2 rank %d of %d" % (rank, l), flush=True)
    rng = np.random.default_rng(l + rank)
    Y = rng.standard_normal((4 * l, rank)) @ (np.geomspace(1.0, 1e-6, rank)[:, None] * rng.standard_normal((rank, l)))
    Q, down = _cholqr2(Y)
    assert down == 1
    assert np.isfinite(Q).all()
