"""Filter steps over block widths that no launch shape covers exactly: lanes
of 2, 4 or 8 columns whose last ones overlap, on blocks with odd leading
dimensions (rows aligned to their elements only).

Every shape computes an element with the same operations in the same order,
so each result has the bits of the one-column shape, which is within the
parity bound of the oracle's forward recurrence (k products and a three-term
update rounded in each of the m steps, amplified by at most m):
2 m^2 (k + 4) u sum |b_i| max|V| in FP64, 2 m (k + 4) u_32 sum |b_i| max|V| in FP32.
"""
import numpy as np
import pytest

from oracle import flp_oracle as O
from paper_2409_15053_amd import flp
from paper_2409_15053_amd import inputs as I

pytestmark = pytest.mark.gpu

U = {flp.FLP_PREC_FP64: 2.0 ** -53, flp.FLP_PREC_FP32_FILTER: 2.0 ** -24}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible MI355X"
    flp.load()
    return t


@pytest.mark.parametrize("prec", [flp.FLP_PREC_FP64, flp.FLP_PREC_FP32_FILTER], ids=["fp64", "fp32"])
@pytest.mark.parametrize("r", [1, 2, 3, 5, 6, 7, 9, 11, 13, 15, 17, 23, 31, 32])
def test_overlapping_lanes(torch, r, prec):
    m = 9
    A = I.laplacian_3d_13pt(17)
    g = max(abs(x) for x in O.gershgorin(A))
    f = flp.flp_build_filter(0.1 * g, 0.3 * g, m, -g, g)
    b = f.coeffs()
    V = I.random_block(A.n, r, seed=r)
    dA = flp.DeviceCsr.from_host(A, with_fp32=True)
    Vd = torch.full((A.n, r + 1), 5.0, dtype=torch.float64, device="cuda:0")
    Vd[:, 1:] = torch.from_numpy(V).to("cuda:0")

    def run(lpr, vec, nt, fmt):
        W = torch.full((A.n, r + 2), -3.0, dtype=torch.float64, device="cuda:0")
        try:
            flp.flp_set_filter_shape(lpr, vec, r, nt, tile_chunk=4)
            flp.flp_filter_apply(f, dA, Vd[:, 1:], W[:, 1:r + 1], prec=prec, format=fmt)
        finally:
            flp.flp_set_filter_shape(0, 0, 0)
        return W

    ref = run(0, 0, False, flp.FLP_FORMAT_CSR)
    for fmt in (flp.FLP_FORMAT_CSR, flp.FLP_FORMAT_SELL):
        for lpr in (1, 2, 4, 8, 16):
            for vec in (0, 2, 4, 8):
                for nt in (False, True):
                    assert torch.equal(ref, run(lpr, vec, nt, fmt)), (lpr, vec, nt, fmt)
    got = ref.cpu().numpy()
    assert (got[:, 0] == -3.0).all() and (got[:, r + 1] == -3.0).all()
    gain = m * m if prec == flp.FLP_PREC_FP64 else m
    tol = 2 * gain * (13 + 4) * U[prec] * np.sum(np.abs(b)) * np.max(np.abs(V))
    err = np.max(np.abs(got[:, 1:r + 1] - O.filter_apply(A, -g, g, b, V)))
    assert err <= tol, (err, tol)
    flp.flp_release_workspace()


@pytest.mark.parametrize("n", [1, 2, 63, 64, 257, 4913])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 8, 13, 16, 17, 24, 31, 32])
def test_product(torch, n, r):
    """Y = A X for every kind of width on odd leading dimensions: each element
    rounds at most k products and k sums."""
    g = np.random.Generator(np.random.PCG64(n * r))
    A = I.laplacian_3d_13pt(17) if n == 4913 else I.random_sym(n, min(1.0, 6.0 / n), seed=n)
    X = torch.full((n, r + 3), 7.0, dtype=torch.float64, device="cuda:0")
    Xh = g.normal(size=(n, r))
    X[:, 2:r + 2] = torch.from_numpy(Xh).to("cuda:0")
    Y = torch.full((n, r + 2), -3.0, dtype=torch.float64, device="cuda:0")
    flp.flp_spmm(flp.DeviceCsr.from_host(A), X[:, 2:r + 2], Y[:, 1:r + 1])
    got = Y.cpu().numpy()
    assert (got[:, 0] == -3.0).all() and (got[:, r + 1] == -3.0).all()
    k = int(np.max(np.diff(A.rowptr)))
    Aabs = I.Csr(A.n, A.rowptr, A.colind, np.abs(A.val))
    bound = 2 * (k + 1) * 2.0 ** -53 * O.spmm(Aabs, np.abs(Xh))
    assert (np.abs(got[:, 1:r + 1] - O.spmm(A, Xh)) <= bound).all()
