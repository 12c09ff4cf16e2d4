"""Performance cases of the library: the calls that users make, over the sizes they make them at.

A case is a plain dict.  Its "kind" names the public call:

* filter: ``flp_filter_apply``, the Chebyshev filter of a block of vectors
  (the call that carries nearly all of a solve's time), from a 40 x 40 grid
  with one vector (launch-bound) to the 120^3 Hamiltonian with sixteen;
* orth: ``flp_block_orth``, one block step's full reorthogonalisation
  against the Lanczos basis;
* qr: ``flp_block_qr``, one block step's normalisation;
* solve: ``flp_solve``, every eigenpair in an interval;
* batch: ``flp_solve_batch``, many independent problems together.

The matrices are the repository's synthetic Hamiltonians (5-, 7- and
13-point stencils plus a potential).  Solves use separable potentials, so
the whole spectrum and its eigenvectors are known from small dense problems
along each axis; the interval then holds a fixed number of eigenvalues.
"""
import math
import random

import numpy as np
import torch

from paper_2409_15053_amd import flp
from paper_2409_15053_amd import inputs as I

DEV = "cuda:0"
PREC = {"fp64": flp.FLP_PREC_FP64, "fp32": flp.FLP_PREC_FP32_FILTER}


def listed():
    return [
        # the smallest use: a 2D model problem, one vector at a time (degree-50 filter of the 40 x 40 Laplacian)
        dict(name="filter 2d 40 r1 fp64", kind="filter", stencil=5, g=40, r=1, degree=50, prec="fp64"),
        # one of the many small problems of a batched or served workload, FP32 filter
        dict(name="filter 3d7 24 r8 fp32", kind="filter", stencil=7, g=24, r=8, degree=60, prec="fp32"),
        # an odd block width on a ragged grid: no vector-aligned shape fits
        dict(name="filter 3d13 37 r5 fp64", kind="filter", stencil=13, g=37, r=5, degree=30, prec="fp64"),
        # the benchmark's filter: 100^3, block 8, FP64
        dict(name="filter 3d7 100 r8 fp64", kind="filter", stencil=7, g=100, r=8, degree=110, prec="fp64"),
        # the large Hamiltonian: 120^3, 13-point, block 16, FP32
        dict(name="filter 3d13 120 r16 fp32", kind="filter", stencil=13, g=120, r=16, degree=65, prec="fp32"),
        # reorthogonalisation late in the benchmark's Lanczos run
        dict(name="orth 1e6 k320 r8", kind="orth", n=1000000, k=320, r=8),
        # the same in a mid-size solve with the block width 5 and a ragged basis
        dict(name="orth 59319 k135 r5", kind="orth", n=59319, k=135, r=5),
        # normalisation of a 16-column block of the large Hamiltonian
        dict(name="qr 1728000 r16", kind="qr", n=1728000, r=16),
        # a whole small solve, one vector at a time, interior interval (2D model problem)
        dict(name="solve 2d 40 r1 fp64", kind="solve", stencil=5, g=40, r=1, degree=50, prec="fp64", target=60,
             offset=40, check_every=0),
        # the benchmark's solve: 100^3, about 100 eigenpairs at the low end
        dict(name="solve 3d7 100 r8 fp64", kind="solve", stencil=7, g=100, r=8, degree=110, prec="fp64", target=104,
             offset=0, check_every=10),
        # a mid-size Hamiltonian window with the FP32 filter and its polish
        dict(name="solve 3d13 60 r16 fp32", kind="solve", stencil=13, g=60, r=16, degree=65, prec="fp32", target=120,
             offset=20, check_every=0),
        # a batch of small problems, FP32 filter, the library's degrees
        dict(name="batch 16 r8 fp32", kind="batch", count=16, gmin=20, gmax=40, r=8, prec="fp32", family=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["filter", "filter", "filter", "orth", "qr", "solve", "batch"])
    prec = rng.choice(["fp64", "fp32"])
    if kind == "filter":
        stencil = rng.choice([5, 7, 13])
        r = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 8, 10, 12, 15, 16, 16, 24, 32])
        degree = _log_int(rng, 20, 150)
        lo, hi = (20, 1000) if stencil == 5 else (8, 120)
        g = _log_int(rng, lo, hi)
        dim = 2 if stencil == 5 else 3
        while float(g) ** dim * r * degree > 1.8e9:
            degree, g = max(20, degree * 3 // 4), max(lo, g * 9 // 10)
        return dict(kind=kind, stencil=stencil, g=g, r=r, degree=degree, prec=prec)
    if kind == "orth":
        r = rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 11, 16, 16])
        n = _log_int(rng, 2000, 1728000)
        k = max(r, _log_int(rng, 8, min(720, n // 4, 3.2e8 / n)))
        return dict(kind=kind, n=n, k=k, r=r)
    if kind == "qr":
        return dict(kind=kind, n=_log_int(rng, 2000, 1728000), r=rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 16]))
    if kind == "solve":
        stencil = rng.choice([5, 7, 7, 13])
        g = _log_int(rng, 30, 200) if stencil == 5 else _log_int(rng, 12, 64)
        n = g ** (2 if stencil == 5 else 3)
        target = min(n // 40, _log_int(rng, 10, 120))
        return dict(kind=kind, stencil=stencil, g=g, r=rng.choice([2, 3, 4, 5, 8, 8, 16]),
                    degree=rng.choice([0, 40, 65, 90, 110]), prec=prec, target=target,
                    offset=rng.choice([0, 0, target // 3]), check_every=0)
    return dict(kind=kind, count=rng.randint(4, 16), gmin=12, gmax=_log_int(rng, 20, 40), r=rng.choice([4, 8, 8, 16]),
                prec=prec, family=rng.randint(0, 10 ** 6))


# ---------------------------------------------------------------- matrices

_AXIS = {5: {0: 2.0, 1: -1.0}, 7: {0: 2.0, 1: -1.0}, 13: I.FOURTH_ORDER_1D}


def _matrix(stencil, g, potential):
    """Device CSR of the stencil on a g^2 or g^3 grid plus the potential (a
    device tensor), columns sorted within a row."""
    dim = 2 if stencil == 5 else 3
    n = g ** dim
    axis = _AXIS[stencil]
    strides = [g ** (dim - 1 - d) for d in range(dim)]
    pts = [(0, 0, None)]
    for d in range(dim):
        for dist in range(1, max(axis) + 1):
            for sgn in (-1, 1):
                pts.append((sgn * dist * strides[d], d, sgn * dist))
    pts.sort()
    row = torch.arange(n, device=DEV, dtype=torch.int64)
    cols = torch.empty((n, len(pts)), dtype=torch.int32, device=DEV)
    vals = torch.empty((n, len(pts)), dtype=torch.float64, device=DEV)
    ok = torch.ones((n, len(pts)), dtype=torch.bool, device=DEV)
    for j, (off, d, step) in enumerate(pts):
        cols[:, j] = (row + off).to(torch.int32)
        if step is None:
            vals[:, j] = dim * axis[0] + potential
        else:
            vals[:, j] = axis[abs(step)]
            q = (row // strides[d]) % g + step
            ok[:, j] = (q >= 0) & (q < g)
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rowptr[1:] = torch.cumsum(ok.sum(1), 0).to(torch.int32)
    return n, rowptr, cols[ok], vals[ok]


def _device_csr(stencil, g, potential, prec):
    n, rowptr, colind, val = _matrix(stencil, g, potential)
    return flp.DeviceCsr(n, rowptr, colind, val, val.float() if prec == "fp32" else None)


def _gershgorin(stencil, potential):
    """An enclosure of the spectrum: the potential's range plus the row sums of an interior point."""
    dim = 2 if stencil == 5 else 3
    mid = dim * _AXIS[stencil][0]
    rad = 2 * dim * sum(abs(c) for d, c in _AXIS[stencil].items() if d)
    return mid - rad + float(potential.min()), mid + rad + float(potential.max())


def _axis_potentials(stencil, g, seed):
    """Random 1D potentials, one per axis: U[0, 1) per point, or for the
    13-point Hamiltonian a well of random centre, depth and width on a weak
    random background."""
    rng = I.rng(seed)
    out = []
    for _ in range(2 if stencil == 5 else 3):
        if stencil == 13:
            c, d, s = rng.uniform(0.3, 0.7) * (g - 1), rng.uniform(1.0, 2.0), rng.uniform(0.1, 0.2) * g
            out.append(0.1 * rng.random(g) - d * np.exp(-(np.arange(g) - c) ** 2 / (2 * s * s)))
        else:
            out.append(rng.random(g) / (2 if stencil == 5 else 3))
    return out


def _axis_eigs(stencil, v):
    g = len(v)
    M = np.diag(v)
    for dist, cf in _AXIS[stencil].items():
        M += cf * (np.eye(g) if dist == 0 else np.eye(g, k=dist) + np.eye(g, k=-dist))
    return np.linalg.eigh(M)


def _separable(case, seed):
    """Axis potentials and eigen-decompositions, and the level indices of the
    eigenvalues offset .. offset + target with the gap-midpoint interval."""
    st, t, off = case["stencil"], case["target"], case["offset"]
    vs = _axis_potentials(st, case["g"], seed)
    eig = [_axis_eigs(st, v) for v in vs]
    lam = eig[0][0]
    for w, _ in eig[1:]:
        lam = (lam[:, None] + w[None, :]).reshape(-1)
    take = min(off + t + 2, lam.size)
    idx = np.argpartition(lam, take - 1)[:take]
    idx = idx[np.argsort(lam[idx])]
    s = lam[idx]
    alpha = s[0] - 0.5 if off == 0 else 0.5 * (s[off - 1] + s[off])
    beta = 0.5 * (s[off + t - 1] + s[off + t])
    return vs, eig, idx[off:off + t], s[off:off + t], float(alpha), float(beta)


def _field(vs):
    f = torch.from_numpy(vs[0]).to(DEV)
    for v in vs[1:]:
        f = (f[:, None] + torch.from_numpy(v).to(DEV)[None, :]).reshape(-1)
    return f


def _batch_members(case):
    rng = random.Random(case["family"])
    out = []
    for _ in range(case["count"]):
        g = _log_int(rng, case["gmin"], case["gmax"])
        out.append(dict(stencil=7, g=g, target=min(g ** 3 // 40, rng.randint(10, 60)), offset=0))
    return out


# ---------------------------------------------------------------- prepare and run

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(n, c, gen):
    return torch.randn((n, c), dtype=torch.float64, device=DEV, generator=gen)


def _filter_inputs(case, seed):
    gen = _gen(seed)
    g = case["g"]
    if case["stencil"] == 13:
        pot = torch.from_numpy(I.gaussian_wells(g, seed % (1 << 30))).to(DEV)
    else:
        pot = torch.rand(g ** (2 if case["stencil"] == 5 else 3), dtype=torch.float64, device=DEV, generator=gen)
    A = _device_csr(case["stencil"], g, pot, case["prec"])
    lmin, lmax = _gershgorin(case["stencil"], pot)
    # a window of the lower spectrum, as the solves filter
    alpha, beta = lmin + 0.05 * (lmax - lmin), lmin + 0.12 * (lmax - lmin)
    f = flp.flp_build_filter(alpha, beta, case["degree"], lmin, lmax)
    return A, f, _randn(A.n, case["r"], gen)


def _orth_inputs(case, seed):
    gen = _gen(seed)
    n, k, r = case["n"], case["k"], case["r"]
    Q = _randn(n, k, gen)
    for _ in range(2):  # orthonormal columns (Cholesky QR twice)
        R = torch.linalg.cholesky((Q.t() @ Q).cpu(), upper=True)
        Q = Q @ torch.linalg.inv(R).to(DEV)
    # a filtered block: mostly in the span of the basis, plus new directions
    W = Q @ _randn(k, r, gen) + _randn(n, r, gen) * (0.3 / math.sqrt(n))
    return Q.contiguous(), W.contiguous()


def _qr_input(case, seed):
    gen = _gen(seed)
    r = case["r"]
    T = torch.triu(_randn(r, r, gen)) + 3.0 * torch.eye(r, dtype=torch.float64, device=DEV)
    return (_randn(case["n"], r, gen) @ T).contiguous()


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind == "filter":
        A, f, V = _filter_inputs(case, seed)
        st.update(A=A, f=f, V=V, W=torch.empty_like(V))
    elif kind == "orth":
        Q, W = _orth_inputs(case, seed)
        st.update(Q=Q, W0=W, W=torch.empty_like(W))
    elif kind == "qr":
        W = _qr_input(case, seed)
        st.update(W0=W, W=torch.empty_like(W))
    elif kind == "solve":
        vs, _, _, _, alpha, beta = _separable(case, seed)
        A = _device_csr(case["stencil"], case["g"], _field(vs), case["prec"])
        st.update(A=A, alpha=alpha, beta=beta, probe=_probe(A.n))
    else:
        As, al, be = [], [], []
        for i, m in enumerate(_batch_members(case)):
            vs, _, _, _, alpha, beta = _separable(m, seed * 64 + i)
            As.append(_device_csr(7, m["g"], _field(vs), case["prec"]))
            al.append(alpha)
            be.append(beta)
        st.update(As=As, al=al, be=be, probes=[_probe(A.n) for A in As])
    return st


def _probe(n):
    return _randn(n, 1, _gen(99))[:, 0].contiguous()


def _result(res, prec, probe):
    """A solve's outputs: eigenvalues and eigenvectors with the sign of their
    product with a fixed vector.  The FP32 filter's eigenvectors hold what
    its residual tolerance leaves open, so its eigenvalues stand alone."""
    if prec == "fp32":
        return dict(evals=res["evals"])
    X = res["evecs"]
    return dict(evals=res["evals"], evecs=X * torch.sign(probe @ X))


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "filter":
        flp.flp_filter_apply(st["f"], st["A"], st["V"], st["W"], prec=PREC[case["prec"]])
        return st["W"]
    if kind == "orth":
        st["W"].copy_(st["W0"])
        H = flp.flp_block_orth(st["Q"], case["k"], st["W"])
        return dict(H=H, W=st["W"])
    if kind == "qr":
        st["W"].copy_(st["W0"])
        S = flp.flp_block_qr(st["W"])
        return dict(S=S, Q=st["W"])
    if kind == "solve":
        res = flp.flp_solve(st["A"], st["alpha"], st["beta"], block=case["r"], degree=case["degree"], seed=1,
                            prec=PREC[case["prec"]], check_every=case["check_every"])
        return _result(res, case["prec"], st["probe"])
    out, _ = flp.flp_solve_batch(st["As"], st["al"], st["be"], block=case["r"], prec=PREC[case["prec"]])
    return [_result(res, case["prec"], p) for res, p in zip(out, st["probes"])]


# ---------------------------------------------------------------- work and exact results

def _shape(case):
    st, g = case["stencil"], case["g"]
    dim, reach = (2, 1) if st == 5 else (3, 1 if st == 7 else 2)
    n = g ** dim
    nnz = n + sum(2 * (g - d) * g ** (dim - 1) for d in range(1, reach + 1)) * dim
    return n, nnz


def _solve_work(case, prec, degree):
    n, nnz = _shape(case)
    t, wv = case["target"], 4 if prec == "fp32" else 8
    # at least one filtered and orthogonalised vector per eigenpair
    return 12.0 * nnz + 8.0 * n * t, 2.0 * nnz * degree * t + 2.0 * n * t * t


def work(case):
    kind = case["kind"]
    if kind == "filter":
        n, nnz = _shape(case)
        r, wv = case["r"], 4 if case["prec"] == "fp32" else 8
        return dict(bytes=nnz * (wv + 4.0) + 4.0 * (n + 1) + 16.0 * n * r,
                    flops=case["degree"] * (2.0 * nnz + 6.0 * n) * r)
    if kind == "orth":
        n, k, r = case["n"], case["k"], case["r"]
        return dict(bytes=8.0 * n * k + 16.0 * n * r + 8.0 * k * r, flops=8.0 * n * k * r)
    if kind == "qr":
        n, r = case["n"], case["r"]
        return dict(bytes=16.0 * n * r, flops=6.0 * n * r * r)
    if kind == "solve":
        b, f = _solve_work(case, case["prec"], case["degree"] or 30)
        return dict(bytes=b, flops=f)
    bs, fs = zip(*(_solve_work(m, case["prec"], 30) for m in _batch_members(case)))
    return dict(bytes=sum(bs), flops=sum(fs))


def _exact_solve(m, prec, seed):
    vs, eig, idx, lam, _, _ = _separable(m, seed)
    if prec == "fp32":
        return dict(evals=lam)
    g, dim = m["g"], len(vs)
    X = None
    for d, (_, U) in enumerate(eig):
        lev = (idx // g ** (dim - 1 - d)) % g
        u = torch.from_numpy(np.ascontiguousarray(U[:, lev])).to(DEV)
        X = u if X is None else (X[:, None, :] * u[None, :, :]).reshape(-1, u.shape[1])
    return dict(evals=lam, evecs=X * torch.sign(_probe(X.shape[0]) @ X))


def exact(case, seed):
    kind = case["kind"]
    if kind == "filter":
        A, f, V = _filter_inputs(case, seed)
        b, inf = f.coeffs(), f.info()
        rows = torch.repeat_interleave(torch.arange(A.n, device=DEV), (A.rowptr[1:] - A.rowptr[:-1]).long())
        width = int((A.rowptr[1:] - A.rowptr[:-1]).max())
        slot = torch.arange(A.nnz, device=DEV) - A.rowptr[:-1].long()[rows]
        col = torch.zeros((A.n, width), dtype=torch.int64, device=DEV)
        val = torch.zeros((A.n, width), dtype=torch.float64, device=DEV)
        col[rows, slot] = A.colind.long()
        val[rows, slot] = A.val

        def mapped(X):  # (A X - c X) / e
            Y = -inf["c"] * X
            for j in range(width):
                Y.addcmul_(val[:, j:j + 1], X[col[:, j]])
            return Y.div_(inf["e"])

        T0, T1 = V, mapped(V)
        W = b[0] * T0 + b[1] * T1
        for i in range(2, len(b)):
            T0, T1 = T1, 2.0 * mapped(T1) - T0
            W += b[i] * T1
        return W
    if kind == "orth":
        Q, W = _orth_inputs(case, seed)
        H1 = Q.t() @ W
        W = W - Q @ H1
        H2 = Q.t() @ W
        return dict(H=(H1 + H2).cpu().numpy(), W=W - Q @ H2)
    if kind == "qr":
        W = _qr_input(case, seed)
        Q, S = W, torch.eye(case["r"], dtype=torch.float64)
        for _ in range(2):
            R = torch.linalg.cholesky((Q.t() @ Q).cpu(), upper=True)
            Q, S = Q @ torch.linalg.inv(R).to(DEV), R @ S
        return dict(S=S.numpy(), Q=Q)
    if kind == "solve":
        return _exact_solve(case, case["prec"], seed)
    return [_exact_solve(m, case["prec"], seed * 64 + i) for i, m in enumerate(_batch_members(case))]
