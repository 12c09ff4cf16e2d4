"""The one-launch filter of small matrices (one workgroup per column) at the
edges of its range: rows around each multiple of the workgroup's 1024
threads, rows longer than its register slots, empty rows, degrees around
its limits, both storages and precisions, strided blocks.

Every result has the bits of the launch-per-step form (forced through
flp_set_filter_shape, which the one-launch form steps aside for), and is
within the parity bound of the oracle's forward recurrence (each of the m
steps rounds a sum of at most k products and a three-term update, and the
recurrence amplifies an error by at most m): 2 m^2 (k + 4) u sum |b_i| max|V|
in FP64, 2 m (k + 4) u_32 sum |b_i| max|V| in FP32.
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


def band(n, reach, long_row=0, empty=()):
    """Symmetric band of half-width `reach`, random entries, scaled so the
    spectrum lies in [-1, 1]; optionally one row of `long_row` entries and
    empty rows (not symmetric then: the filter does not need it)."""
    g = np.random.Generator(np.random.PCG64(n + reach))
    w = g.uniform(-1.0, 1.0, (reach + 1, n)) / (2 * reach + 1)
    cols, vals, ptr = [], [], [0]
    for i in range(n):
        js = [j for j in range(max(0, i - reach), min(n, i + reach + 1))]
        if i == n // 3 and long_row:
            js = sorted(g.choice(n, size=min(long_row, n), replace=False).tolist())
        if i in empty:
            js = []
        cols += js
        if i == n // 3 and long_row:
            vals += list(g.uniform(-1.0, 1.0, len(js)) / len(js))
        else:
            vals += [w[abs(i - j), min(i, j)] for j in js]
        ptr.append(len(cols))
    return I.Csr(n, np.array(ptr, np.int32), np.array(cols, np.int32), np.array(vals))


def check(torch, A, m, r, prec, fmts=(flp.FLP_FORMAT_CSR, flp.FLP_FORMAT_SELL), pad=0):
    f = flp.flp_build_filter(-0.4, 0.1, m, -1.0, 1.0)
    b = f.coeffs()
    V = I.random_block(A.n, r, seed=m + r)
    dA = flp.DeviceCsr.from_host(A, with_fp32=True)
    Vd = torch.full((A.n, r + pad), 5.0, dtype=torch.float64, device="cuda:0")
    Vd[:, pad:] = torch.from_numpy(V).to("cuda:0")
    outs = []
    for fmt in fmts:
        for forced in (False, True):
            try:
                if forced:
                    flp.flp_set_filter_shape(0, 0, r)
                W = torch.full((A.n, r + pad), -3.0, dtype=torch.float64, device="cuda:0")
                flp.flp_filter_apply(f, dA, Vd[:, pad:], W[:, :r], prec=prec, format=fmt)
                outs.append(W)
            finally:
                flp.flp_set_filter_shape(0, 0, 0)
    W = torch.full((A.n, r + pad), -3.0, dtype=torch.float64, device="cuda:0")
    flp.flp_filter_apply_noalloc(f, dA, Vd[:, pad:], W[:, :r], prec=prec)
    outs.append(W)
    torch.cuda.synchronize()
    flp.flp_release_workspace()
    for W in outs[1:]:
        assert torch.equal(outs[0], W)
    got = outs[0].cpu().numpy()
    assert np.all(got[:, r:] == -3.0)
    k = int(np.max(np.diff(A.rowptr)))
    gain = m * m if prec == flp.FLP_PREC_FP64 else m
    tol = 2 * gain * (k + 4) * U[prec] * np.sum(np.abs(b)) * np.max(np.abs(V))
    err = np.max(np.abs(got[:, :r] - O.filter_apply(A, -1.0, 1.0, b, V)))
    assert err <= tol, (err, tol)


@pytest.mark.parametrize("prec", list(U))
@pytest.mark.parametrize("n,reach", [(1, 0), (7, 1), (1023, 3), (1024, 3), (1025, 6), (2048, 7), (2049, 3),
                                     (3071, 6), (3073, 3), (4096, 2), (4097, 2)])
def test_row_counts(torch, prec, n, reach):
    check(torch, band(n, reach), 9, 3, prec)


@pytest.mark.parametrize("prec", list(U))
@pytest.mark.parametrize("n,reach,long_row", [(700, 2, 60), (1500, 2, 300), (1500, 5, 200), (2600, 3, 40)])
def test_long_and_empty_rows(torch, prec, n, reach, long_row):
    A = band(n, reach, long_row, empty=(0, 5, n // 2, n - 1))
    check(torch, A, 12, 2, prec)


@pytest.mark.parametrize("prec", list(U))
@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 384, 385])
def test_degrees(torch, prec, m):
    check(torch, band(300, 2), m, 1, prec)


@pytest.mark.parametrize("r,pad", [(1, 3), (5, 2), (32, 1)])
def test_strided_blocks(torch, r, pad):
    check(torch, band(1100, 3), 17, r, flp.FLP_PREC_FP64, pad=pad)


def test_capture_replays(torch):
    """Recorded into a graph (no allocation, no synchronisation on the path)
    and replayed on changed inputs, with eager work between the replays."""
    A = band(1200, 3)
    f = flp.flp_build_filter(-0.4, 0.1, 20, -1.0, 1.0)
    dA = flp.DeviceCsr.from_host(A)
    V = torch.empty((A.n, 4), dtype=torch.float64, device="cuda:0")
    W = torch.empty_like(V)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        flp.flp_filter_apply(f, dA, V, W, stream=s)
    for seed in range(4):
        V.copy_(torch.from_numpy(I.random_block(A.n, 4, seed=seed)))
        g.replay()
        torch.cuda.synchronize()
        want = torch.empty_like(V)
        flp.flp_filter_apply(f, dA, V, want)
        torch.cuda.synchronize()
        assert torch.equal(W, want)
