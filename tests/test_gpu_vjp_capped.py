"""Reverse mode through capped swaps, whose kept triplets alone are computed
(swap matrices of more than 128 rows and columns, the cap at most a quarter of
them): against the oracle's reverse mode, within the sweep limit of the product
itself, and where a tie at the cut ends no series.
"""
import numpy as np
import pytest

import oracle as O
import ttm_inputs as I
from test_gpu_vjp import _bound, _cbar, _host, _rel, _vjp_conditioning

pytestmark = pytest.mark.gpu


def _decaying(phys, chi, seed):
    """A random train whose bonds carry the weights 1 / k."""
    cores = I.random_tt(len(phys), phys, chi, seed)
    return [c / (1.0 + np.arange(c.shape[2])) if i + 1 < len(cores) else c for i, c in enumerate(cores)]


def _check(A, B, W, chi, tol, monkeypatch, **opts):
    import paper_2410_19747_amd as T

    res = O.ttm(A, B, chi, tol)
    (_, oA, oB), kappa = _vjp_conditioning(monkeypatch, A, B, chi, tol, _cbar(W, res.cores))
    C0, _ = T.multiply(A, B, chi, tol, **opts)
    C, dA, dB, st = T.multiply_vjp(A, B, chi, tol, _cbar(W, _host(C0)), **opts)
    assert st["ranks"] == res.ranks
    # the product that multiply gave, signs of its singular vectors included
    assert all(np.array_equal(x, y) for x, y in zip(_host(C), _host(C0)))
    ea, eb = _rel(_host(dA), oA), _rel(_host(dB), oB)
    print("  rel err dA %.3e dB %.3e, conditioning %.3e" % (ea, eb, kappa), flush=True)
    assert max(ea, eb) <= _bound(kappa)


@pytest.mark.parametrize("phys,chi_a,chi_b,chi", [([8] * 4, 24, 20, 20), ([8] * 5, 17, 40, 33),
                                                  ([6, 4, 9, 12, 3, 7], 36, 30, 31), ([5, 40, 6, 40, 5], 24, 24, 23)])
def test_vjp_of_capped_swaps(phys, chi_a, chi_b, chi, monkeypatch):
    """Square, tall and wide swap matrices."""
    print("vjp %s chi_a=%d chi_b=%d chi=%d" % (phys, chi_a, chi_b, chi), flush=True)
    A, B, W = _decaying(phys, chi_a, 1), _decaying(phys, chi_b, 2), I.random_tt(len(phys), phys, 5, 3)
    _check(A, B, W, chi, 1e-14, monkeypatch)


def test_vjp_within_the_products_sweep_limit():
    """The least svd_max_sweeps that multiply accepts, multiply_vjp accepts."""
    import paper_2410_19747_amd as T

    chi = 40
    A, B = I.turbulence_qtt(64, 101, chi), I.turbulence_qtt(64, 102, chi)
    for limit in range(1, 41):
        try:
            C, _ = T.multiply(A, B, chi, 1e-14, svd_max_sweeps=limit)
            break
        except T.TTMError as e:
            assert e.code == T.TTM_ENOCONV
    print("multiply within %d sweeps" % limit, flush=True)
    C2, dA, dB, st = T.multiply_vjp(A, B, chi, 1e-14, C, svd_max_sweeps=limit)
    assert all(np.array_equal(x, y) for x, y in zip(_host(C), _host(C2)))


def test_vjp_at_a_tie():
    """Every singular value twice, an odd cap: the two values at the cut differ
    by rounding alone.  No derivative exists there; what comes back is finite."""
    import paper_2410_19747_amd as T

    half = _decaying([8] * 5, 30, 5)
    tied = []
    for i, c in enumerate(half):
        l, d, r = c.shape
        if i == 0:
            t = np.zeros((1, 2 * d, 2 * r))
            t[:, :d, :r], t[:, d:, r:] = c, c
        elif i == len(half) - 1:
            t = np.zeros((2 * l, 2 * d, 1))
            t[:l, :d], t[l:, d:] = c, c
        else:
            t = np.zeros((2 * l, d, 2 * r))
            t[:l, :, :r], t[l:, :, r:] = c, c
        tied.append(t)
    ones = [np.ones((1, c.shape[1], 1)) for c in tied]
    C, _ = T.multiply(ones, tied, 33, 1e-14)
    _, dA, dB, _ = T.multiply_vjp(ones, tied, 33, 1e-14, C)
    for g in _host(dA) + _host(dB):
        assert np.isfinite(g).all()
