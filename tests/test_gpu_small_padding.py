"""The one-launch filter where the sliced ELL copy is larger than the matrix:
average row lengths at which the copy's padded rows, but not the matrix's own,
exceed 8 entries, over the row counts up to which each number of register
slots has a kernel (2048, 3072 and 4096 rows).

Bits and tolerance as in test_gpu_small_filter (the same check): all three
storages give the bits of the launch-per-step form.  Whole solves in the
default storage against dense eigenvalues (1e-10 relative; residuals at the
solver's tolerance 1e-9).
"""
import numpy as np
import pytest

from paper_2409_15053_amd import flp
from paper_2409_15053_amd import inputs as I

from .test_gpu_small_filter import U, band, check, torch  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu

FMTS = (flp.FLP_FORMAT_CSR, flp.FLP_FORMAT_AUTO, flp.FLP_FORMAT_SELL)


def from_edges(n, a, b, seed):
    """Symmetric matrix with these off-diagonal entries (each pair once) and
    a full diagonal, random, its absolute row sums at most 1."""
    key = np.unique(np.minimum(a, b).astype(np.int64) * n + np.maximum(a, b))
    a, b = key // n, key % n
    a, b = a[a != b], b[a != b]
    g = np.random.Generator(np.random.PCG64(seed))
    w = g.uniform(-1.0, 1.0, a.size)
    r = np.concatenate([a, b, np.arange(n)])
    c = np.concatenate([b, a, np.arange(n)])
    v = np.concatenate([w, w, g.uniform(-1.0, 1.0, n)])
    v /= np.max(np.bincount(r, np.abs(v)))
    o = np.lexsort((c, r))
    ptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))])
    return I.Csr(n, ptr.astype(np.int32), c[o].astype(np.int32), v[o])


def ring(n):
    """Eight entries in every row: i, i +- 1, i +- 2, i +- 3 and i + n / 2."""
    i = np.arange(n)
    return from_edges(n, np.tile(i, 4), np.concatenate([(i + d) % n for d in (1, 2, 3)] + [(i + n // 2) % n]), n)


def mesh(s):
    """A triangulated s x s grid, a tenth of its points with an edge more."""
    i = np.arange(s * s).reshape(s, s)
    x = np.random.Generator(np.random.PCG64(s)).permutation(s * s)[:s * s // 10]
    a = [i[:-1].ravel(), i[:, :-1].ravel(), i[:-1, :-1].ravel(), x]
    b = [i[1:].ravel(), i[:, 1:].ravel(), i[1:, 1:].ravel(), (x + 2 * s) % (s * s)]
    return from_edges(s * s, np.concatenate(a), np.concatenate(b), s)


MATRICES = {
    "ring1030": lambda: ring(1030), "ring2046": lambda: ring(2046), "ring2050": lambda: ring(2050),
    "ring3000": lambda: ring(3000), "ring3074": lambda: ring(3074), "ring4094": lambda: ring(4094),
    "mesh45": lambda: mesh(45), "mesh54": lambda: mesh(54), "mesh63": lambda: mesh(63),
    "band2600": lambda: band(2600, 3, 60), "band3500": lambda: band(3500, 3, 60),
    "band4096": lambda: band(4096, 3, 100), "band2600wide": lambda: band(2600, 6, 60),
}


@pytest.mark.parametrize("prec", list(U))
@pytest.mark.parametrize("name", list(MATRICES))
@pytest.mark.parametrize("m", [5, 9])
def test_padded_copies(torch, name, prec, m):
    check(torch, MATRICES[name](), m, 3, prec, fmts=FMTS)


@pytest.mark.parametrize("prec", list(U))
@pytest.mark.parametrize("name", ["ring2050", "mesh54", "ring3074"])
def test_solve_in_the_default_storage(torch, name, prec):
    A = MATRICES[name]()
    lam = np.linalg.eigvalsh(A.to_dense())
    alpha, beta = lam[0] - 0.1, 0.5 * (lam[19] + lam[20])
    res = flp.flp_solve(flp.DeviceCsr.from_host(A, with_fp32=True), alpha, beta, block=4, degree=40, seed=1, prec=prec)
    assert res["count"] == 20
    assert np.max(np.abs(np.sort(res["evals"]) - lam[:20])) <= 1e-10 * np.max(np.abs(lam))
    assert np.max(res["resid"]) <= 1e-9
