"""The banded host eigensolver at the edges of its reflectors' vector lengths
(multiples of four, each doubling of the vector count, the widest band it
takes) and of its double sweeps (blocks of up to 8 rows take one), against
numpy's dense solver.

N columns are cleared, each by reflectors whose errors act once on an entry,
and N eigenvalues deflate after a few sweeps each: both add at most about a
unit roundoff per column to an entry of the factors, of the matrix and of the
vectors, so the bound is 10 N u, times the matrix's norm where it scales.
"""
import numpy as np
import pytest

from paper_2409_15053_amd import flp

U = 2.0 ** -53


@pytest.mark.parametrize("bw", [0, 1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129])
@pytest.mark.parametrize("kind", ["random", "sparse", "duplicates", "tiny", "huge"])
def test_band(bw, kind):
    g = np.random.Generator(np.random.PCG64(bw))
    for N in (1, 2, 3, 4, 7, 8, 9, 10, 12, 31, 33, 130, 8 * bw + 9 if bw > 23 else 8 * bw + 3):
        M = np.triu(np.tril(g.normal(size=(N, N)), bw), -bw)
        M = M + M.T
        if kind == "sparse":
            M = np.triu(np.where(g.random((N, N)) < 0.5, 0.0, M))
            M = M + np.triu(M, 1).T
        elif kind == "duplicates":
            M = np.diag(g.integers(0, 3, N).astype(float)) + 1e-9 * M
        elif kind == "tiny":
            M = M * 1e-180
        elif kind == "huge":
            M = M * 1e150
        ev, V = flp.flp_host_sym_eig(M, bw)
        norm = max(np.abs(M).sum(axis=1).max(), 1e-300)
        tol = 10 * N * U
        assert np.abs(ev / norm - np.linalg.eigvalsh(M / norm)).max() <= tol
        assert np.abs(M / norm @ V - V * (ev / norm)).max() <= tol
        assert np.abs(V.T @ V - np.eye(N)).max() <= tol
