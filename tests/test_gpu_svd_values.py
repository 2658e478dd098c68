"""Singular values of the one-workgroup SVD, whose columns carry every rotation
to the end: their norms must not drift.

Tolerance: a column takes part in at most about ten sweeps of k rotations, each
of which changes its norm by up to u, either way alike: 2 sqrt(10 k) u of the
largest value.
"""
import numpy as np
import pytest

from test_gpu_svd_small import _svd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["power", "exponential", "flat"])
@pytest.mark.parametrize("m,n", [(16, 16), (32, 32), (64, 64), (300, 64), (64, 200), (96, 96), (128, 128), (128, 500)])
def test_values_do_not_drift(m, n, kind):
    rng = np.random.default_rng(m + n)
    k = min(m, n)
    a, _ = np.linalg.qr(rng.standard_normal((m, k)))
    b, _ = np.linalg.qr(rng.standard_normal((n, k)))
    s = {"power": (1.0 + np.arange(k)) ** -2.0, "exponential": 10.0 ** (-6.0 * np.arange(k) / k),
         "flat": np.linspace(1.1, 0.1, k)}[kind]
    M = (a * s) @ b.T
    got = _svd(M)[2]
    err = np.abs(got - np.linalg.svd(M, compute_uv=False)).max() / s[0] / 2.0 ** -53
    print("%dx%d %s: %.1f u" % (m, n, kind, err), flush=True)
    assert err <= 2 * np.sqrt(10 * k)
