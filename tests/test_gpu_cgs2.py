"""flp_block_orth's fused update and projection at the edges of its tiles of
16 columns (per wave and per block), of 16 rows and of a block's rows, on
bases with odd leading dimensions, and past its widest basis.

Two passes of W -= Q (Q^T W), each sum of n or K products rounding at most
once per term: elementwise 2 (n + K + 4) u times the same recurrence on
absolute values.  Q and W are not orthogonal, so both passes do work.
"""
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


@pytest.mark.parametrize("r", [1, 5, 8, 16])
@pytest.mark.parametrize("n,ks", [(1, (1, 3)), (16, (4, 17)), (17, (15, 16, 64)), (70, (5, 33, 65, 129)),
                                  (1000, (1, 64, 128, 192, 193, 256, 257, 320, 321)),
                                  (16401, (7, 127, 130, 319, 384, 385, 512)), (3000, (513, 639, 640, 641))])
def test_fused_passes(torch, n, ks, r):
    g = np.random.Generator(np.random.PCG64(n + r))
    for k in ks:
        for pad in (0, 3):
            Q = g.standard_normal((n, k)) / np.sqrt(n + k)
            W = g.standard_normal((n, r))
            Qd = torch.full((n, k + pad), float("nan"), dtype=torch.float64, device="cuda:0")
            Qd[:, :k] = torch.from_numpy(Q).to("cuda:0")
            Wd = torch.from_numpy(W).to("cuda:0")
            H = flp.flp_block_orth(Qd, k, Wd)
            H1 = Q.T @ W
            W1 = W - Q @ H1
            H2 = Q.T @ W1
            A = np.abs(Q)
            b1 = A.T @ np.abs(W)
            w1 = np.abs(W) + A @ b1
            b2 = A.T @ w1
            w2 = w1 + A @ b2
            u = 2 * (n + k + 4) * 2.0 ** -53
            assert (np.abs(H - (H1 + H2)) <= u * (b1 + b2)).all(), (k, pad)
            assert (np.abs(Wd.cpu().numpy() - (W1 - Q @ H2)) <= u * w2).all(), (k, pad)
