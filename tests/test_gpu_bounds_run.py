"""The bounds estimate's Lanczos run at the edges of its blocks of 256 rows,
of its block count, and of spaces smaller than its number of steps; and many
matrices in one run (a batch) against each by itself.

The estimate encloses the spectrum (Ritz value, residual bound and a margin,
clamped to Gershgorin).  In a batch a matrix's partial sums are split over
other blocks: the same numbers up to rounding, which three-term Lanczos
carries forward without growth until a Ritz pair converges, so the bounds
agree to 1e-8 of the spectrum's width.
"""
import numpy as np
import pytest

from oracle import flp_oracle as O
from paper_2409_15053_amd import flp
from paper_2409_15053_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible MI355X"
    flp.load()
    return t


@pytest.mark.parametrize("n", [1, 2, 3, 39, 40, 41, 64, 65, 255, 256, 257, 1023, 1025])
def test_enclosure_edges(torch, n):
    A = I.random_sym(n, min(1.0, 8.0 / n), seed=n)
    w = np.linalg.eigvalsh(A.to_dense())
    lmin, lmax = flp.flp_estimate_bounds(flp.DeviceCsr.from_host(A), 40, 3)
    slack = 1e-12 * max(abs(w[0]), abs(w[-1]))
    assert lmin <= w[0] + slack and lmax >= w[-1] - slack
    if n > 1:  # (an interval of one point is widened by 1e-8 of it)
        glo, ghi = O.gershgorin(A)
        assert glo - slack <= lmin and lmax <= ghi + slack


@pytest.mark.parametrize("n", [256 * 1024 - 1, 256 * 1024, 256 * 1024 + 1, 700001])
def test_enclosure_many_blocks(torch, n):
    d = 2.0 + (np.arange(n) % 7) / 3.0
    d[n - 1] = 9.0
    A = I.diagonal_csr(d)
    lmin, lmax = flp.flp_estimate_bounds(flp.DeviceCsr.from_host(A), 40, 3)
    assert 2.0 - 0.01 * 7.0 <= lmin <= 2.0
    assert d[:-1].max() <= lmax <= 9.0 * (1 + 1e-12)


@pytest.mark.parametrize("prec", [flp.FLP_PREC_FP64, flp.FLP_PREC_FP32_FILTER], ids=["fp64", "fp32"])
def test_batch_matches_each(torch, prec):
    mats = [I.laplacian_3d(g) for g in (7, 9, 12, 16)] + [I.laplacian_2d(23), I.laplacian_3d_13pt(11)]
    dAs = [flp.DeviceCsr.from_host(A, with_fp32=True) for A in mats]
    g = [O.gershgorin(A) for A in mats]
    al = [lo + 0.05 * (hi - lo) for lo, hi in g]
    be = [lo + 0.12 * (hi - lo) for lo, hi in g]
    res, _ = flp.flp_solve_batch(dAs, al, be, block=4, prec=prec)
    for i, (r, dA, a, b) in enumerate(zip(res, dAs, al, be)):
        one = flp.flp_solve(dA, a, b, block=4, prec=prec, seed=i)  # a batch's default seeds
        width = one["lmax"] - one["lmin"]
        assert abs(r["lmin"] - one["lmin"]) <= 1e-8 * width
        assert abs(r["lmax"] - one["lmax"]) <= 1e-8 * width
        assert r["count"] == one["count"]
