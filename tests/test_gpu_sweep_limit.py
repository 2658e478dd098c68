"""svd_max_sweeps refuses no product that the block Jacobi method alone
carries within it: the SVDs in one workgroup, the capped ones and the
randomized ones, whose sweeps are others, fall back on it.

Tolerance: two truncations of the same products by backward-stable SVDs, 1e-12
relative (the bound of the parity tests).
"""
import ctypes

import numpy as np
import pytest

import oracle as O
import ttm_inputs as I

pytestmark = pytest.mark.gpu


def _host(packed):
    return [c.detach().cpu().numpy() for c in packed.cores()]


def _least_limit(T, A, B, chi, tol):
    """The least svd_max_sweeps at which every SVD of the product converges by
    the block method alone."""
    for limit in range(1, 41):
        try:
            return limit, T._run("block", A, B, chi, tol, svd_max_sweeps=limit)
        except T.TTMError as e:
            assert e.code == T.TTM_ENOCONV
    raise AssertionError("no limit up to 40")


def _check(A, B, chi, tol, what, **opts):
    import paper_2410_19747_amd as T

    limit, (C0, st0) = _least_limit(T, A, B, chi, tol)
    print("%s: block method within %d sweeps" % (what, limit), flush=True)
    C, st = T.multiply(A, B, chi, tol, svd_max_sweeps=limit, **opts)
    assert st["jacobi_max_sweeps"] <= limit and st["ranks"] == st0["ranks"]
    return O.rel_frob(_host(C), _host(C0))


@pytest.mark.parametrize("phys,ca,cb,chi", [([4] * 6, 16, 16, 16), ([8] * 5, 12, 12, 12),
                                            ([3, 5, 2, 7, 4, 6, 3], 23, 19, 21)])
def test_one_workgroup_svds(phys, ca, cb, chi):
    A, B = I.random_tt(len(phys), phys, ca, 3), I.random_tt(len(phys), phys, cb, 4)
    assert _check(A, B, chi, 1e-14, "sides up to %d" % (max(phys) * chi)) <= 1e-12


@pytest.mark.parametrize("grid,chi", [(64, 32), (64, 64), (128, 40)])
def test_capped_svds(grid, chi):
    """Swap matrices of side 8 chi, of which chi triplets are kept."""
    A, B = I.turbulence_qtt(grid, 101, chi), I.turbulence_qtt(grid, 102, chi)
    assert _check(A, B, chi, 1e-14, "%d^3 at bond %d" % (grid, chi)) <= 1e-12


@pytest.mark.parametrize("m,n,cap", [(160, 200, 30), (300, 280, 60)])
def test_capped_svd_leaves_the_limit_to_the_full_one(m, n, cap):
    """One sweep is too few for the projection's columns (below and above 64 of
    them): refused, so that the full SVD runs, and no error."""
    import torch

    import paper_2410_19747_amd as T

    L = T.lib()
    rng = np.random.default_rng(m)
    k = min(m, n)
    a, _ = np.linalg.qr(rng.standard_normal((m, k)))
    b, _ = np.linalg.qr(rng.standard_normal((n, k)))
    M = (a * (1.0 + np.arange(k)) ** -1.5) @ b.T
    d = torch.from_numpy(np.ascontiguousarray(M.T)).cuda()
    pt = torch.zeros(cap * n, dtype=torch.float64, device="cuda")
    xt = torch.zeros(m * cap, dtype=torch.float64, device="cuda")
    ws = torch.zeros(int(L.ttm_test_capped_svd_ws_bytes(m, n, cap)) // 8 + 1, dtype=torch.float64, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    for sweeps, want in ((1, 1), (60, 0)):
        rank, refused, w = ctypes.c_int(0), ctypes.c_int(-1), (ctypes.c_double * 3)()
        rc = L.ttm_test_capped_svd_sweeps(p(d), m, n, cap, 1e-14, sweeps, p(pt), p(xt), ctypes.byref(rank),
                                          ctypes.byref(refused), w, p(ws), ws.numel() * 8, None)
        assert (rc, refused.value) == (0, want)
