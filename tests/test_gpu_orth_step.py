"""The block step's reorthogonalisation and normalisation kernels at the
edges of their tiles.

* flp_block_qr over block widths that fill, under-fill and just miss the
  16-column operand, and row counts around its 16- and 64-row pieces: the
  unique QR with a positive diagonal, W = Q S to 1e-12 and Q^T Q = I to 1e-13
  (Cholesky QR twice is backward stable).
* flp_block_orth for bases around the widths where its kernels change (one
  wavefront of columns, the FMA projection from 256 columns at 8 columns of
  W): two passes of classical Gram-Schmidt, 1e-12 relative.
* Whole solves whose basis ends up spanning the matrix's whole space: late
  block steps then take most of each new vector away, which flags them for
  another pass or for repair; count and eigenvalues against dense eigh
  (1e-10 relative), residuals at the solver's tolerance (1e-9).
"""
import numpy as np
import pytest

from paper_2409_15053_amd import flp
from paper_2409_15053_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible MI355X"
    flp.load()
    return t


@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 7, 8, 11, 12, 15, 16])
@pytest.mark.parametrize("n", [16, 17, 63, 65, 129, 1000, 70001])
def test_block_qr_edges(torch, n, r):
    g = np.random.Generator(np.random.PCG64(100 * n + r))
    W = g.standard_normal((n, r)) @ np.triu(g.standard_normal((r, r)) + 3 * np.eye(r))
    Wd = torch.from_numpy(W).to("cuda:0")
    S = flp.flp_block_qr(Wd)
    Q = Wd.cpu().numpy()
    assert np.allclose(np.tril(S, -1), 0) and np.all(np.diag(S) > 0)
    assert np.max(np.abs(Q.T @ Q - np.eye(r))) < 1e-13
    assert np.max(np.abs(Q @ S - W)) < 1e-12 * np.max(np.abs(W))


@pytest.mark.parametrize("n,k,r", [(64, 16, 1), (65, 17, 8), (2001, 64, 8), (2001, 65, 5), (5003, 255, 8),
                                   (5003, 256, 8), (5003, 257, 8), (5003, 319, 8), (4097, 320, 7), (4097, 511, 16),
                                   (9001, 700, 16), (9001, 641, 8)])
def test_block_orth_edges(torch, n, k, r):
    g = np.random.Generator(np.random.PCG64(n + k + r))
    Q, _ = np.linalg.qr(g.standard_normal((n, k)))
    W = g.standard_normal((n, r))
    Wd = torch.from_numpy(W).to("cuda:0")
    H = flp.flp_block_orth(torch.from_numpy(np.ascontiguousarray(Q)).to("cuda:0"), k, Wd)
    H1 = Q.T @ W
    W1 = W - Q @ H1
    H2 = Q.T @ W1
    W2 = W1 - Q @ H2
    assert np.max(np.abs(H - (H1 + H2))) < 1e-12 * np.max(np.abs(W)) * np.sqrt(n)
    got = Wd.cpu().numpy()
    assert np.max(np.abs(got - W2)) < 1e-12 * np.max(np.abs(W))
    assert np.max(np.abs(Q.T @ got)) < 1e-13 * np.sqrt(n) * np.max(np.abs(W))


@pytest.mark.parametrize("block", [1, 3, 4, 8])
@pytest.mark.parametrize("n", [40, 97])
def test_basis_of_the_whole_space(torch, n, block):
    A = I.random_sym(n, 0.2, seed=n)
    lam = np.linalg.eigvalsh(A.to_dense())
    i0, cnt = n // 4, n // 2
    alpha, beta = 0.5 * (lam[i0 - 1] + lam[i0]), 0.5 * (lam[i0 + cnt - 1] + lam[i0 + cnt])
    dA = flp.DeviceCsr.from_host(A)
    run = lambda: flp.flp_solve(dA, alpha, beta, block=block, unfiltered=True, seed=3, check_every=1000)
    if n % block:
        # the step after the last whole block has fewer than `block`
        # directions left: no replacement completes it
        with pytest.raises(flp.FlpError, match="rank-deficient"):
            run()
        return
    res = run()
    assert res["count"] == cnt
    assert np.max(np.abs(np.sort(res["evals"]) - lam[i0:i0 + cnt])) <= 1e-10 * np.max(np.abs(lam))
    assert np.max(res["resid"]) <= 1e-9
    X = res["evecs"].cpu().numpy()
    assert np.max(np.abs(X.T @ X - np.eye(cnt))) <= 1e-9
