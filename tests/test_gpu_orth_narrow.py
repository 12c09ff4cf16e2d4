"""flp_block_orth against narrow bases on many rows, around the sizes where its
first update and second projection are one kernel or two (2^17 rows; 32 basis
columns for up to 8 columns of W, 20 beyond).

Two passes of classical Gram-Schmidt in FP64 NumPy: entries of H and W are
sums of n or k products of entries of at most max|W| and 1 / sqrt(n) here, so
they agree to 1e-12 relative.  The last test holds the time of a narrow basis
against that of a wider one: 0.55 with two kernels, 0.75 with one.
"""
import time

import numpy as np
import pytest

from paper_2409_15053_amd import flp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible MI355X"
    flp.load()
    return t


def basis(n, k):
    """k orthonormal columns."""
    Q, _ = np.linalg.qr(np.random.Generator(np.random.PCG64(n + k)).standard_normal((n, k)))
    return np.ascontiguousarray(Q)


@pytest.mark.parametrize("n,k,r", [(131071, 8, 8), (131072, 32, 8), (131073, 1, 1), (131073, 32, 8), (131073, 33, 8),
                                   (131073, 20, 16), (131073, 21, 9), (140001, 16, 3), (140001, 31, 5),
                                   (140001, 20, 11), (262144, 32, 4)])
def test_both_forms(torch, n, k, r):
    Q = basis(n, k)
    W = np.random.Generator(np.random.PCG64(r)).standard_normal((n, r))
    Wd = torch.from_numpy(W).to("cuda:0")
    H = flp.flp_block_orth(torch.from_numpy(Q).to("cuda:0"), k, Wd)
    H1 = Q.T @ W
    W1 = W - Q @ H1
    H2 = Q.T @ W1
    top = np.max(np.abs(W))
    assert np.max(np.abs(H - (H1 + H2))) < 1e-12 * top * np.sqrt(n)
    assert np.max(np.abs(Wd.cpu().numpy() - (W1 - Q @ H2))) < 1e-12 * top


def test_narrow_basis_takes_the_shorter_form(torch):
    n = 1000000

    def best(k):
        Q = torch.randn(n, k, dtype=torch.float64, device="cuda:0") / n ** 0.5
        W = torch.randn(n, 1, dtype=torch.float64, device="cuda:0")
        t = []
        for _ in range(9):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(5):
                flp.flp_block_orth(Q, k, W)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    narrow, wide = best(8), best(40)
    assert narrow <= 0.66 * wide, (narrow, wide)
