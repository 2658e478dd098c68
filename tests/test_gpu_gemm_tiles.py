"""The FP64 and FP32 products at the edges of their kernels: few output tiles
(32 x 32 tiles without LDS, K over one wave up to 256 and over four above) and
many (64 x 64 tiles), remainders in every direction, and operands whose
strides and bases allow or forbid 16-byte loads.

Tolerance, entry by entry: 2 K u |A| |B| in FP64 (the bound of a K-term dot
product, on either side); 32 * 2^-24 |A| |B| in FP32 (two operand roundings
and sums of 16 terms).
"""
import ctypes

import numpy as np
import pytest

import paper_2410_19747_amd as T

pytestmark = pytest.mark.gpu

GUARD = 7.25


def _operand(torch, X, k_first, pad, shift):
    """X on the device with its first (k_first) or second index contiguous
    after it: the tensor, the address of X(0, 0) and the strides of X."""
    rows, cols = X.shape
    ld = (rows if k_first else cols) + pad
    buf = np.full(shift + ld * (cols if k_first else rows), np.nan)
    view = buf[shift:].reshape(-1, ld)
    if k_first:
        view[:, :rows] = X.T
    else:
        view[:, :cols] = X
    t = torch.from_numpy(buf).cuda()
    return t, ctypes.c_void_p(t.data_ptr() + 8 * shift), (1, ld) if k_first else (ld, 1)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (31, 33, 3), (33, 32, 16), (64, 65, 17), (65, 1, 255), (32, 31, 256),
                                   (33, 65, 257), (1, 33, 271), (96, 40, 320), (40, 200, 1001), (1030, 1025, 37)])
def test_product_at_the_edges(M, N, K, prec):
    import torch

    L = T.lib()
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A, B = rng.standard_normal((M, K)), rng.standard_normal((K, N))
    ref = A @ B
    tol = (2 * K * 2.0 ** -53 if prec == 0 else 32 * 2.0 ** -24) * (np.abs(A) @ np.abs(B)) + 1e-300
    for a_first, b_first in ((False, False), (False, True), (True, False), (True, True)):
        for pad, shift in ((0, 0), (1, 0), (2, 0), (2, 1)):
            print("product %dx%dx%d prec %d: %d %d pad %d shift %d" % (M, N, K, prec, a_first, b_first, pad, shift),
                  flush=True)
            ta, pa, (ars, acs) = _operand(torch, A, a_first, pad, shift)
            tb, pb, (brs, bcs) = _operand(torch, B, b_first, pad, shift)
            ldc = N + 3
            C = torch.full(((M + 1) * ldc,), GUARD, dtype=torch.float64, device="cuda")
            rc = L.ttm_test_gemm_prec(prec, M, N, K, pa, ars, acs, pb, brs, bcs, ctypes.c_void_p(C.data_ptr()), ldc,
                                      None)
            assert rc == 0, rc
            out = C.cpu().numpy().reshape(M + 1, ldc)
            assert (np.abs(out[:M, :N] - ref) <= tol).all()
            assert (out[M] == GUARD).all() and (out[:, N:] == GUARD).all()
            del ta, tb
