"""The capped swap SVD at full accuracy (the cap leading singular triplets by a
filtered subspace iteration, checked, with the full SVD where it refuses)
against LAPACK's truncation.

Tolerance of the truncated matrix: 200 u ||Theta|| over the relative gap at
the cut (Wedin's bound for a backward error of 32 u on either side, with
room); of the orthonormal factor: 64 l u, a Jacobi SVD's of l columns.
"""
import ctypes

import numpy as np
import pytest

import paper_2410_19747_amd as T

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _capped(M, cap, eps):
    import torch

    L = T.lib()
    m, n = M.shape
    d = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()  # column-major
    pt = torch.full((cap * n,), float("nan"), dtype=torch.float64, device="cuda")
    xt = torch.full((m * cap,), float("nan"), dtype=torch.float64, device="cuda")
    need = int(L.ttm_test_capped_svd_ws_bytes(m, n, cap))
    assert need > 0
    ws = torch.full((need // 8 + 1,), float("nan"), dtype=torch.float64, device="cuda")
    rank, refused, w = ctypes.c_int(0), ctypes.c_int(0), (ctypes.c_double * 3)()
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = L.ttm_test_capped_svd(p(d), m, n, cap, eps, p(pt), p(xt), ctypes.byref(rank), ctypes.byref(refused), w,
                               p(ws), ws.numel() * 8, None)
    assert rc == 0, rc
    if refused.value:
        return None
    r = rank.value
    return pt.cpu().numpy()[: r * n].reshape(r, n), xt.cpu().numpy()[: m * r].reshape(m, r), r, list(w)


def _with_values(m, n, s, seed):
    rng = np.random.default_rng(seed)
    k = min(m, n)
    a, _ = np.linalg.qr(rng.standard_normal((m, k)))
    b, _ = np.linalg.qr(rng.standard_normal((n, k)))
    return (a * s) @ b.T, a, b


@pytest.mark.parametrize("m,n,cap", [(160, 129, 32), (129, 400, 17), (256, 256, 64), (301, 277, 65), (512, 1000, 100),
                                     (1024, 600, 128), (530, 530, 130)])
def test_decaying_spectrum(m, n, cap):
    k = min(m, n)
    s = (1.0 + np.arange(k)) ** -1.5
    s[cap:] *= 0.9
    M, a, b = _with_values(m, n, s, m + n)
    got = _capped(M, cap, 1e-14)
    assert got is not None
    pt, xt, r, w = got
    assert r == cap
    assert np.abs(pt @ pt.T - np.eye(r)).max() <= 64 * 2 * cap * U
    gap = (s[cap - 1] - s[cap]) / s[cap - 1]
    want = (a[:, :r] * s[:r]) @ b[:, :r].T
    assert np.linalg.norm(xt @ pt - want) <= 200 * U / gap * np.linalg.norm(s)
    tail = (s[cap:] ** 2).sum()
    assert abs(w[0] - tail) <= 1e-9 * tail and abs(w[1] - (s ** 2).sum()) <= 1e-12 * w[1]


def test_rule_cuts_below_the_cap():
    m, n, cap, eps = 300, 320, 64, 1e-6
    s = 0.93 ** np.arange(300)
    M, a, b = _with_values(m, n, s, 3)
    tail = np.append(np.cumsum((s ** 2)[::-1])[::-1], 0.0)
    want = next(i for i in range(1, 300) if tail[i] < eps * tail[0])
    assert want > cap  # the cap binds
    got = _capped(M, cap, eps)
    assert got is not None and got[2] == cap
    s = 0.8 ** np.arange(300)
    s[100:] = s[100]
    M, a, b = _with_values(m, n, s, 4)
    tail = np.append(np.cumsum((s ** 2)[::-1])[::-1], 0.0)
    want = next(i for i in range(1, 300) if tail[i] < eps * tail[0])
    assert want < cap
    got = _capped(M, cap, eps)
    assert got is None or got[2] == want


def test_equal_values_at_the_cut():
    """sigma_r = sigma_{r+1}: any choice within the cluster is a best rank-r
    approximation."""
    m = n = 256
    cap = 40
    s = 0.9 ** np.arange(256)
    s[30:50] = s[30]
    M, _, _ = _with_values(m, n, s, 5)
    got = _capped(M, cap, 1e-14)
    assert got is not None
    pt, xt, r, w = got
    assert r == cap and np.abs(pt @ pt.T - np.eye(r)).max() <= 64 * 2 * cap * U
    best = np.sqrt((s[cap:] ** 2).sum())
    assert abs(np.linalg.norm(M - xt @ pt) - best) <= 200 * U * np.linalg.norm(s)


@pytest.mark.parametrize("kind", ["flat", "rank_between", "rank_below", "zero", "nan", "huge", "tiny"])
def test_refused_or_right(kind):
    """Matrices that the filter is not made for: refused, or as accurate."""
    m, n, cap = 200, 260, 32
    rng = np.random.default_rng(6)
    s = np.ones(200)
    if kind == "flat":
        M = rng.standard_normal((m, n))
    elif kind == "rank_between":
        s = 0.9 ** np.arange(200) * (np.arange(200) < 48)
        M = _with_values(m, n, s, 7)[0]
    elif kind == "rank_below":
        s = 0.9 ** np.arange(200) * (np.arange(200) < 20)
        M = _with_values(m, n, s, 8)[0]
    elif kind == "zero":
        M = np.zeros((m, n))
    else:
        M = _with_values(m, n, 0.9 ** np.arange(200), 9)[0]
        M = M * {"huge": 1e120, "tiny": 1e-120, "nan": 1.0}[kind]
        if kind == "nan":
            M[3, 5] = np.nan
    got = _capped(M, cap, 1e-14)
    if kind in ("zero", "nan", "rank_below"):
        assert got is None
    if got is not None:
        pt, xt, r, w = got
        sv = np.linalg.svd(M, compute_uv=False)
        assert r == cap
        assert abs(np.linalg.norm(M - xt @ pt) - np.linalg.norm(sv[r:])) <= 200 * U * np.linalg.norm(sv)


@pytest.mark.parametrize("m,n,cap,rate", [(256, 256, 40, 0.2), (200, 260, 33, 0.25), (300, 256, 64, 0.12),
                                          (512, 1024, 128, 0.06)])
def test_spectrum_steeper_than_the_grams_resolve(m, n, cap, rate):
    """Values 10^(-rate i): those at the end of the 2 cap sketch columns are
    below u of the first, so that a plain CholeskyQR breaks down; the kept ones
    are above the noise level, and the passes with a shift must find them."""
    s = 10.0 ** (-rate * np.arange(min(m, n)))
    M, _, _ = _with_values(m, n, s, 11)
    got = _capped(M, cap, 1e-30)
    assert got is not None
    pt, xt, r, w = got
    assert r == cap and np.abs(pt @ pt.T - np.eye(r)).max() <= 64 * 2 * cap * U
    best = np.sqrt((s[cap:] ** 2).sum())
    assert abs(np.linalg.norm(M - xt @ pt) - best) <= 200 * U * np.linalg.norm(s)
