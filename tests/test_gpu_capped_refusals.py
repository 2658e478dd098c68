"""What a swap pays whose capped SVD cannot succeed: where the kept rank lies
below the cap and below the noise level, the start of the iteration shows it and
the full SVD runs, without a second, shifted iteration before it.
"""
import numpy as np
import pytest

import oracle as O
import ttm_inputs as I

pytestmark = pytest.mark.gpu


def _padded(n, d, chi, rank, seed):
    """A random train of the given rank with bonds up to chi."""
    rng = np.random.default_rng(seed)
    cores, inv = [], np.eye(1)
    for i, c in enumerate(I.random_tt(n, d, rank, seed)):
        r = c.shape[2]
        g = np.eye(1) if i == n - 1 else rng.standard_normal((r, min(chi, d ** (i + 1), d ** (n - i - 1))))
        cores.append(np.einsum("ab,bsc,cd->asd", inv, c, g))
        inv = np.linalg.pinv(g)
    return cores


def _host(packed):
    return [c.detach().cpu().numpy() for c in packed.cores()]


@pytest.mark.parametrize("rank,chi,cap", [(3, 32, 40), (4, 64, 100), (2, 30, 33)])
def test_low_rank_costs_one_start(rank, chi, cap):
    """Products and factorisations (timed regions) where every swap's rank lies
    below the cap: at most those of the block method and of one start a swap
    (five products, three orthonormalisations)."""
    import paper_2410_19747_amd as T

    A, B = _padded(6, 8, chi, rank, 7), _padded(6, 8, chi, rank, 8)
    C, st = T.multiply(A, B, cap, 0.0, profile=True)
    _, full = T._run("block", A, B, cap, 0.0, profile=True)
    count = lambda s: s["kernel_launches"]["gemm"] + s["kernel_launches"]["qr"]  # noqa: E731
    print("rank %d cap %d: %d regions, block method %d, %d swaps" % (rank ** 2, cap, count(st), count(full),
                                                                    st["n_swap"]), flush=True)
    assert count(st) <= count(full) + 8 * st["n_swap"]
    assert max(C.bonds) == rank ** 2
    assert O.rel_frob(_host(C), O.ttm(A, B, cap, 0.0).cores) <= 1e-12


@pytest.mark.parametrize("scale", [1e-70, 1e-45, 1e45, 1e70])
def test_scale_does_not_refuse(scale):
    """The capped SVD of the matrix times a power of two: the same vectors to
    the bit, where the squares of its squares stay in range."""
    import test_gpu_svd_capped as S

    scale = 2.0 ** round(np.log2(scale))
    m, n, cap = 200, 260, 32
    M = S._with_values(m, n, (1.0 + np.arange(200)) ** -1.2, 9)[0]
    a, b = S._capped(M, cap, 1e-14), S._capped(M * scale, cap, 1e-14)
    assert a is not None and b is not None
    assert a[2] == b[2] == cap
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1] * scale, b[1])
