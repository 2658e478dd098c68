"""ttm_multiply_block and ttm_multiply_block_vjp, every SVD by the block method:
against the oracle at the bounds of the default entries' tests, and next to the
default entry at sizes that it takes by one workgroup and as capped SVDs."""
import ctypes

import numpy as np
import pytest

import oracle as O
import ttm_inputs as I
from test_gpu_vjp import _bound, _cbar, _host, _rel, _vjp_conditioning

pytestmark = pytest.mark.gpu


def _trains(n, d, chi, seed):
    cores = I.random_tt(n, d, chi, seed)
    return [c / (1.0 + np.arange(c.shape[2])) if i + 1 < n else c for i, c in enumerate(cores)]


@pytest.mark.parametrize("n,d,chi_a,chi_b,chi", [(4, 2, 3, 2, 3), (6, 4, 16, 8, 12), (5, 8, 24, 20, 20)])
def test_block_entries_vs_oracle(n, d, chi_a, chi_b, chi, monkeypatch):
    import paper_2410_19747_amd as T

    print("block entries n=%d d=%d chi=%d" % (n, d, chi), flush=True)
    A, B, W = _trains(n, d, chi_a, 1), _trains(n, d, chi_b, 2), I.random_tt(n, d, 4, 3)
    res = O.ttm(A, B, chi, 1e-14)
    (_, oA, oB), kappa = _vjp_conditioning(monkeypatch, A, B, chi, 1e-14, _cbar(W, res.cores))
    C0, st0 = T._run("block", A, B, chi, 1e-14)
    assert st0["ranks"] == res.ranks and O.rel_frob(_host(C0), res.cores) <= 1e-12
    Cd, _ = T.multiply(A, B, chi, 1e-14)
    assert O.rel_frob(_host(C0), _host(Cd)) <= 1e-12
    C, dA, dB, st = T._vjp(T.lib().ttm_multiply_block_vjp, A, B, chi, 1e-14, _cbar(W, _host(C0)), None, None, {})
    assert all(np.array_equal(x, y) for x, y in zip(_host(C), _host(C0)))
    assert st["ranks"] == res.ranks
    assert max(_rel(_host(dA), oA), _rel(_host(dB), oB)) <= _bound(kappa)


def test_block_entries_refuse_what_the_default_ones_refuse():
    import paper_2410_19747_amd as T

    A, B = I.random_tt(4, 2, 3, 1), I.random_tt(4, 2, 3, 2)
    with pytest.raises(T.TTMError) as e:
        T._run("block", A, B, 0, 1e-14)
    assert e.value.code == T.TTM_EINVAL
    C, _ = T._run("block", A, B, 3, 1e-14)
    with pytest.raises(T.TTMError) as e:
        T._vjp(T.lib().ttm_multiply_block_vjp, A, B, 3, 1e-14, C, None, None, {"svd_mode": "randomized"})
    assert e.value.code == T.TTM_EUNSUPPORTED
    rc = T.lib().ttm_multiply_block(None, None, 3, ctypes.c_double(1e-14), None, None, 0, None, None, None)
    assert rc == T.TTM_EINVAL
