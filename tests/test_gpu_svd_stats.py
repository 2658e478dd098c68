"""The statistics of a product's SVDs describe the work that ran: pair solves
where the block method was launched and nowhere else, and the flops of the
method whose result was taken.
"""
import math

import numpy as np
import pytest

import oracle as O
import ttm_inputs as I

pytestmark = pytest.mark.gpu


def _pair_flops(rows):
    """Arithmetic of one 32-column pair solve over the partial Grams of at least
    64 rows each: their sum, 31 rotation steps (6 flops an entry), two products."""
    return math.ceil(rows / 64) * 32 ** 2 + 6 * 32 ** 2 * 31 + 4 * 32 ** 3


def _launches(st):
    return st["kernel_launches"]["jacobi_solve"]


@pytest.mark.parametrize("svd_mode", ["jacobi", "randomized"])
def test_no_pair_solves_in_one_workgroup_svds(svd_mode):
    import paper_2410_19747_amd as T

    A, B = I.random_tt(6, 4, 16, 1), I.random_tt(6, 4, 16, 2)  # swap matrices up to 64 x 64
    _, st = T.multiply(A, B, 16, 1e-14, profile=True, svd_mode=svd_mode)
    assert st["sweeps"] > 0 and _launches(st) == 0 and st["jacobi_solve_flops"] == 0.0


@pytest.mark.parametrize("svd_mode", ["jacobi", "randomized"])
@pytest.mark.parametrize("chi", [40, 64])
def test_pair_solves_of_capped_svds(chi, svd_mode):
    """Every launch solves between one and half the pairs of 8 chi columns."""
    import paper_2410_19747_amd as T

    A, B = I.turbulence_qtt(64, 101, chi), I.turbulence_qtt(64, 102, chi)
    _, st = T.multiply(A, B, chi, 1e-14, profile=True, svd_mode=svd_mode)
    n, rows = _launches(st), 8 * chi
    print("bond %d, %s: %d launches, %.3g flops" % (chi, svd_mode, n, st["jacobi_solve_flops"]), flush=True)
    assert n > 0
    assert n * _pair_flops(64) <= st["jacobi_solve_flops"] <= n * math.ceil(rows / 32) * _pair_flops(rows)


def test_pair_solves_of_the_block_method():
    """One swap matrix, 48 x 48 (two sites of 48 at bond 1 x 1, chi 48): two
    blocks of 16 and one of padding to four, three rounds of two pairs a sweep."""
    import paper_2410_19747_amd as T

    rng = np.random.default_rng(0)
    A = [rng.standard_normal((1, 48, 40)), rng.standard_normal((40, 48, 1))]
    B = [rng.standard_normal((1, 48, 1)), rng.standard_normal((1, 48, 1))]
    _, st = T._run("block", A, B, 48, 1e-14, profile=True, final_round=False)
    assert st["n_svd"] == 1
    assert _launches(st) == 3 * st["sweeps"]
    assert st["jacobi_solve_flops"] == 2 * _launches(st) * _pair_flops(48)


def test_flops_of_the_method_that_ran():
    """Outside the SVDs every method does the oracle's schedule; the capped and
    the randomized SVDs count their own steps, not the full ones' model."""
    import paper_2410_19747_amd as T

    chi = 64
    A, B = I.turbulence_qtt(256, 101, chi), I.turbulence_qtt(256, 102, chi)
    stats = {k: f[1] for k, f in (("block", T._run("block", A, B, chi, 1e-14)), ("jacobi", T.multiply(A, B, chi, 1e-14)),
                                  ("randomized", T.multiply(A, B, chi, 1e-14, svd_mode="randomized")))}
    rest = {k: st["model_flops"] - st["svd_model_flops"] for k, st in stats.items()}
    print({k: "%.4g" % st["svd_model_flops"] for k, st in stats.items()}, flush=True)
    assert np.isclose(stats["block"]["model_flops"], O.ttm(A, B, chi, 1e-14).flops, rtol=1e-12)
    for k in ("jacobi", "randomized"):
        assert np.isclose(rest[k], rest["block"], rtol=1e-9)
        assert 0.0 < stats[k]["svd_model_flops"] != stats["block"]["svd_model_flops"]
