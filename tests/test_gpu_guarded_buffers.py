"""CholeskyQR2 and the capped SVD inside larger buffers filled with NaN: at
ragged sizes no word before or behind the matrix, the results or the workspace
is written, and none that was not written is read.

Tolerances: those of the tests of the same kernels (4 p u, at least 1e-14; 200 u
over the gap at the cut).
"""
import ctypes

import numpy as np
import pytest

import paper_2410_19747_amd as T

pytestmark = pytest.mark.gpu

PAD = 96  # doubles before and behind


class _Guarded:
    def __init__(self, doubles, values=None):
        import torch

        self.n = doubles
        self.t = torch.full((PAD + doubles + PAD,), float("nan"), dtype=torch.float64, device="cuda")
        if values is not None:
            self.t[PAD:PAD + doubles] = torch.from_numpy(np.ascontiguousarray(values).reshape(-1)).cuda()

    @property
    def ptr(self):
        return ctypes.c_void_p(self.t.data_ptr() + 8 * PAD)

    def get(self):
        g = self.t.cpu().numpy()
        assert np.isnan(g[:PAD]).all() and np.isnan(g[PAD + self.n:]).all()
        return g[PAD:PAD + self.n]


@pytest.mark.parametrize("p,l", [(1, 1), (17, 1), (80, 65), (97, 96), (128, 127), (130, 129), (300, 257), (513, 513),
                                 (1050, 1025)])
def test_cholqr2_stays_inside(p, l):
    L = T.lib()
    rng = np.random.default_rng(p + l)
    u, _, vt = np.linalg.svd(rng.standard_normal((p, l)), full_matrices=False)
    Y = (u * np.geomspace(1.0, 0.01, l)) @ vt
    d, ws = _Guarded(p * l, Y.T), _Guarded(int(L.ttm_test_cholqr2_ws_bytes(p, l)) // 8)
    down = ctypes.c_int(-1)
    rc = L.ttm_test_cholqr2(d.ptr, p, l, ctypes.byref(down), ws.ptr, ws.n * 8, None)
    assert (rc, down.value) == (0, 0)
    ws.get()
    Q = d.get().reshape(l, p).T
    assert np.abs(Q.T @ Q - np.eye(l)).max() <= max(1e-14, 4 * p * 2.0 ** -53)


def _capped(m, n, s, cap, eps, seed):
    L = T.lib()
    rng = np.random.default_rng(seed)
    k = min(m, n)
    a, _ = np.linalg.qr(rng.standard_normal((m, k)))
    b, _ = np.linalg.qr(rng.standard_normal((n, k)))
    M = (a * s) @ b.T
    d, pt, xt = _Guarded(m * n, M.T), _Guarded(cap * n), _Guarded(m * cap)
    ws = _Guarded(int(L.ttm_test_capped_svd_ws_bytes(m, n, cap)) // 8)
    assert ws.n > 0
    rank, refused, w = ctypes.c_int(0), ctypes.c_int(-1), (ctypes.c_double * 3)()
    rc = L.ttm_test_capped_svd(d.ptr, m, n, cap, eps, pt.ptr, xt.ptr, ctypes.byref(rank), ctypes.byref(refused), w,
                               ws.ptr, ws.n * 8, None)
    assert (rc, refused.value) == (0, 0)
    ws.get()
    assert np.array_equal(d.get().reshape(n, m).T, M)
    r = rank.value
    P, X = pt.get()[:r * n].reshape(r, n), xt.get()[:m * r].reshape(m, r)
    gap = (s[r - 1] - s[r]) / s[r - 1]
    want = (a[:, :r] * s[:r]) @ b[:, :r].T
    assert np.linalg.norm(X @ P - want) <= 200 * 2.0 ** -53 / gap * np.linalg.norm(s)
    tail = (s[r:] ** 2).sum()
    assert abs(w[0] - tail) <= 1e-9 * tail
    return r


# the last: 64-column block pairs (8192 rows, more than 256 columns)
@pytest.mark.parametrize("m,n,cap", [(129, 131, 32), (301, 277, 65), (150, 300, 33), (600, 8192, 140)])
def test_capped_svd_stays_inside(m, n, cap):
    s = (1.0 + np.arange(min(m, n))) ** -1.5
    s[cap:] *= 0.9
    assert _capped(m, n, s, cap, 1e-14, m + n) == cap


@pytest.mark.parametrize("m,n,cap,eps", [(300, 320, 64, 1e-5), (260, 300, 65, 1e-4), (400, 257, 60, 1e-5)])
def test_rank_below_the_cap_is_accepted(m, n, cap, eps):
    """The rule of Eq. (eps) cuts below the cap, well clear of every check: the
    capped SVD has to find that rank, not to leave it to the full one."""
    s = (1.0 + np.arange(min(m, n))) ** -2.0
    tail = np.append(np.cumsum((s ** 2)[::-1])[::-1], 0.0)
    want = next(i for i in range(1, len(s)) if tail[i] < eps * tail[0])
    assert 1 < want < cap
    assert _capped(m, n, s, cap, eps, m) == want
