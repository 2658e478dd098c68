"""The one-workgroup SVD of matrices with a short side of at most 128, against
LAPACK, at the edges of its tiles (32, 64 and 128 columns) and in each of its
forms: from the matrix itself, from the triangle of a tall matrix, and from
that of a wide one.

Tolerances: a backward-stable SVD's, p(k) u ||M|| with p(k) = 64 k (a column
takes part in at most about ten sweeps of k rotations, each with a few
roundings of its own norm, and in k reflections).
"""
import ctypes

import numpy as np
import pytest

import paper_2410_19747_amd as T

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _svd(M, eps=0.0, cap=0, right_pow=0):
    import torch

    L = T.lib()
    m, n = M.shape
    k = min(m, n)
    d = torch.from_numpy(np.ascontiguousarray(M)).cuda()
    left = torch.zeros(m * k, dtype=torch.float64, device="cuda")
    right = torch.zeros(k * n, dtype=torch.float64, device="cuda")
    sig = torch.zeros(k, dtype=torch.float64, device="cuda")
    ws = torch.full((int(L.ttm_test_svd_ws_bytes_bw(m, n, 0)) // 8 + 1,), float("nan"), dtype=torch.float64,
                    device="cuda")
    rank, sweeps = ctypes.c_int(0), ctypes.c_int(0)
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = L.ttm_test_svd_bw(p(d), m, n, eps, cap, 0, 1 - right_pow, right_pow, p(left), p(right), p(sig),
                           ctypes.byref(rank), ctypes.byref(sweeps), 0, p(ws), ws.numel() * 8, None)
    assert rc == 0, rc
    r = rank.value
    return (left.cpu().numpy()[: m * r].reshape(m, r), right.cpu().numpy()[: r * n].reshape(r, n),
            sig.cpu().numpy(), r)


def _matrix(kind, m, n, rng):
    if kind == "random":
        return rng.standard_normal((m, n))
    if kind == "ones":  # rank one: what a QR leaves after a few columns is far below any rounding error
        return np.ones((m, n))
    if kind in ("huge", "tiny"):  # squared norms near the ends of the range
        return rng.standard_normal((m, n)) * (1e150 if kind == "huge" else 1e-150)
    k = min(m, n)
    a, _ = np.linalg.qr(rng.standard_normal((m, k)))
    b, _ = np.linalg.qr(rng.standard_normal((n, k)))
    if kind == "graded":  # from 1 to below the rounding level of 1
        return (a * 10.0 ** -np.linspace(0, 18, k)) @ b.T
    s = np.ones(k)  # "deficient": a cluster, then exact zeros
    s[(k + 1) // 2:] = 0.0
    return (a * s) @ b.T


SIZES = [(1, 1), (2, 1), (1, 7), (3, 3), (16, 16), (31, 32), (32, 32), (33, 17), (40, 33), (64, 64), (63, 65), (65, 64),
         (96, 97), (127, 128), (128, 128), (1, 300), (300, 1), (129, 16), (20, 130), (500, 33), (64, 512), (1000, 65),
         (128, 1024), (513, 128), (127, 129), (95, 96), (96, 70), (97, 97), (96, 400), (400, 96), (97, 300)]


@pytest.mark.parametrize("right_pow", [0, 1])
@pytest.mark.parametrize("kind", ["random", "graded", "deficient", "ones", "huge", "tiny"])
@pytest.mark.parametrize("m,n", SIZES)
def test_small_svd(m, n, kind, right_pow):
    rng = np.random.default_rng(1000 * m + n)
    M = _matrix(kind, m, n, rng)
    left, right, s, r = _svd(M, right_pow=right_pow)
    k = min(m, n)
    ref = np.linalg.svd(M, compute_uv=False)
    tol = 64 * k * U
    assert np.abs(s - ref).max() <= tol * ref[0]
    assert (np.diff(s) <= 0).all()
    # only values above the rounding-noise level 8 sqrt(k) u ||M|| are kept
    # (u there is the spacing 2^-52)
    noise = 16 * np.sqrt(k) * U * np.linalg.norm(M)
    assert np.count_nonzero(ref > 2 * noise) <= r <= max(1, np.count_nonzero(ref > noise / 2))
    orth = right @ right.T if right_pow == 0 else left.T @ left
    assert np.abs(orth - np.eye(r)).max() <= tol
    rest = np.sqrt((ref[r:] ** 2).sum())
    assert np.linalg.norm(left @ right - M) <= rest + tol * np.linalg.norm(M)


@pytest.mark.parametrize("m,n,cap", [(32, 32, 5), (64, 64, 64), (100, 90, 40), (600, 128, 128), (128, 700, 1)])
def test_small_svd_cap_and_eps(m, n, cap):
    rng = np.random.default_rng(m + n)
    k = min(m, n)
    a, _ = np.linalg.qr(rng.standard_normal((m, k)))
    b, _ = np.linalg.qr(rng.standard_normal((n, k)))
    s = 0.9 ** np.arange(k)
    M = (a * s) @ b.T
    eps = 1e-6
    tail = np.append(np.cumsum((s ** 2)[::-1])[::-1], 0.0)
    want = min(next(i for i in range(1, k + 1) if tail[i] < eps * tail[0] or tail[i] == 0), cap)
    left, right, sig, r = _svd(M, eps=eps, cap=cap)
    assert r == want
    assert np.linalg.norm(left @ right - (a[:, :r] * s[:r]) @ b[:, :r].T) <= 64 * k * U * 10 * np.linalg.norm(s)
