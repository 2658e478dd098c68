"""The products with K split over workgroups: the direct kernel's slices (of
multiples of 64 terms, over which its four waves share K as well), the tiled
kernel's, their last and ragged slices, with alpha, beta and a batch, in scratch
that allows two slices, three, or all that a split takes.

Tolerance, entry by entry: 2 K u |A| |B| in FP64 (a K-term dot product in any
order, on either side), 32 * 2^-24 |A| |B| with FP32 operands (two roundings and
sums of 16 terms), both times |alpha|; and 4 u |beta C|.
"""
import ctypes

import numpy as np
import pytest

import paper_2410_19747_amd as T

pytestmark = pytest.mark.gpu

U = 2.0 ** -53
GUARD = 7.25


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("M,N,K,batch", [(33, 31, 257, 1), (1, 1, 513, 1), (32, 64, 513, 3), (65, 40, 1001, 1),
                                         (17, 128, 4097, 1), (96, 100, 770, 2), (128, 96, 4097, 1), (40, 24, 8190, 1),
                                         (160, 130, 300, 1), (256, 512, 4100, 1), (300, 257, 7001, 1)])
def test_split_product(M, N, K, batch, prec):
    import torch

    L = T.lib()
    rng = np.random.default_rng(M + 3 * N + 7 * K)
    A, B = rng.standard_normal((batch, M, K)), rng.standard_normal((batch, K, N))
    C0 = rng.standard_normal((batch, M, N))
    ref = A @ B
    tol = (2 * K * U if prec == 0 else 32 * 2.0 ** -24) * (np.abs(A) @ np.abs(B))
    outs = M * N * batch
    p = lambda t, o=0: ctypes.c_void_p(t.data_ptr() + 8 * o)  # noqa: E731
    for k_a, k_b in ((False, False), (True, True), (True, False)):  # which operand has unit stride along K
        a = torch.from_numpy(np.ascontiguousarray(A if k_a else A.transpose(0, 2, 1))).cuda()
        b = torch.from_numpy(np.ascontiguousarray(B.transpose(0, 2, 1) if k_b else B)).cuda()
        ars, acs = (K, 1) if k_a else (1, M)
        brs, bcs = (1, K) if k_b else (N, 1)
        for slices in (2, 3, 600):
            for alpha, beta in ((1.0, 0.0), (-0.5, 0.25)):
                print("split product %dx%dx%d batch %d prec %d: %d %d, room for %d, beta %g"
                      % (M, N, K, batch, prec, k_a, k_b, slices, beta), flush=True)
                ldc, room = N + 3, slices * outs + 5
                cbuf = np.full((batch, M + 1, ldc), GUARD)
                cbuf[:, :M, :N] = C0
                c = torch.from_numpy(cbuf).cuda()
                part = torch.full((64 + room + 64,), float("nan"), dtype=torch.float64, device="cuda")
                rc = L.ttm_test_gemm_split(prec, M, N, K, batch, p(a), ars, acs, M * K, p(b), brs, bcs, K * N, p(c),
                                           ldc, (M + 1) * ldc, alpha, beta, p(part, 64), room, None)
                assert rc == 0, rc
                out = c.cpu().numpy()
                err = np.abs(out[:, :M, :N] - (alpha * ref + beta * C0))
                assert (err <= abs(alpha) * tol + 4 * U * np.abs(beta * C0) + 1e-300).all()
                assert (out[:, M] == GUARD).all() and (out[:, :, N:] == GUARD).all()
                assert torch.isnan(part[:64]).all() and torch.isnan(part[64 + room:]).all()
                if K >= 513 and M * N < 20000:  # few tiles and a long sum: split
                    assert not torch.isnan(part[64:64 + 2 * outs]).any()
