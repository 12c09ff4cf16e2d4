"""The repair of blocks with numerically dependent columns: the numbers it
leaves, on both sides of the block count up to which the Cholesky blocks add
the partial Gram matrices themselves (at most 8192 numbers), with scratch
memory that holds another block's coefficients from an earlier call.

* flp_block_qr reports the deficiency and leaves the repaired block:
  Q^T Q = I and W = Q S with S = Q^T W upper triangular, its diagonal positive
  for the good columns and zero for the dependent ones (whose random
  replacements the columns after them are orthogonalised against).  Cholesky QR twice is backward stable (1e-13 on
  Q^T Q, 1e-12 of max|W| on the products), and a dependent column is taken for
  one up to 1e-7 ||W||_F; these are dependent to rounding.
* flp_solve from a start block with dependent columns, and from one that holds
  eigenvectors of A (their filtered columns lie in the basis, so the first
  block step has dependent columns and goes on with replaced ones): every
  eigenvalue of the interval, checked after every block step, so a coupling
  block S_j that is wrong would end the run early or not at all.
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


def fill_scratch(torch, r):
    """The coefficients 3 I, a well-conditioned 'Gram matrix', in the calling
    thread's scratch."""
    Q = torch.eye(64, r, dtype=torch.float64, device="cuda:0")
    H = flp.flp_block_orth(Q, r, (3.0 * Q).contiguous())
    assert np.allclose(H, 3.0 * np.eye(r))


@pytest.mark.parametrize("n,r,dep", [(500, 1, (0,)), (500, 2, (1,)), (500, 4, (0, 3)), (500, 5, (2,)), (500, 8, (7,)),
                                     (500, 16, (1, 8, 15)), (4096, 16, (3,)), (4097, 16, (3,)), (16384, 8, (2, 5)),
                                     (16385, 8, (2, 5)), (70001, 8, (0,)), (70001, 16, (4, 9))])
def test_block_qr_leaves_the_repaired_block(torch, n, r, dep):
    g = np.random.Generator(np.random.PCG64(n + r))
    W = g.standard_normal((n, r)) @ np.triu(g.standard_normal((r, r)) + 3 * np.eye(r))
    for j in dep:  # combinations of the columns before (none before the first: zero)
        W[:, j] = W[:, :j] @ g.standard_normal(j)
    Wd = torch.from_numpy(W).to("cuda:0")
    fill_scratch(torch, r)
    with pytest.raises(flp.FlpError, match="rank deficient"):
        flp.flp_block_qr(Wd)
    Q = Wd.cpu().numpy()
    good = [j for j in range(r) if j not in dep]
    S = Q.T @ W
    scale = np.max(np.abs(W)) if good else 1.0
    assert np.max(np.abs(Q.T @ Q - np.eye(r))) < 1e-13
    assert np.max(np.abs(Q @ S - W)) < 1e-12 * scale
    root = np.sqrt(n) * scale
    assert np.max(np.abs(np.tril(S, -1))) < 1e-12 * root
    assert np.max(np.abs(np.diag(S)[list(dep)])) < 1e-12 * root
    assert np.all(np.diag(S)[good] > 0)


def spectrum(n):
    """Distinct eigenvalues, 24 of them inside (1, 1.3)."""
    return np.concatenate([np.linspace(-3.0, 0.9, n // 2), np.linspace(1.01, 1.29, 24),
                           np.linspace(1.4, 4.0, n - n // 2 - 24)])


def solve_all(torch, n, block, start):
    d = spectrum(n)
    d = d[np.random.Generator(np.random.PCG64(n)).permutation(n)]
    fill_scratch(torch, block)
    res = flp.flp_solve(flp.DeviceCsr.from_host(I.diagonal_csr(d)), 1.0, 1.3, block=block, seed=2, start=start(d),
                        check_every=1)
    want = np.sort(d[(d > 1.0) & (d < 1.3)])
    assert res["count"] == want.size
    assert np.max(np.abs(np.sort(res["evals"]) - want)) <= 1e-12 * 4.0
    assert np.max(res["resid"]) <= 1e-9


@pytest.mark.parametrize("n,block", [(400, 2), (400, 8), (5001, 16), (20001, 8)])
def test_dependent_start_block(torch, n, block):
    def start(d):
        V = I.random_block(n, block, seed=block)
        V[:, -1] = V[:, 0]
        return V
    solve_all(torch, n, block, start)


@pytest.mark.parametrize("n,block,eig", [(400, 2, (0,)), (400, 4, (1, 2)), (400, 8, (7,)), (5001, 16, (3, 4)),
                                         (20001, 8, (0, 5))])
def test_start_block_with_eigenvectors(torch, n, block, eig):
    def start(d):
        V = I.random_block(n, block, seed=block)
        rows = np.argsort(np.abs(d - 1.1))[:len(eig)]  # inside the interval
        V[rows] = 0.0
        for j, i in zip(eig, rows):
            V[:, j] = 0.0
            V[i, j] = 1.0
        return V
    solve_all(torch, n, block, start)
