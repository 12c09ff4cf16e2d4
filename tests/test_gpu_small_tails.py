"""The one-launch filter's rows of more entries than its register slots: the
lengths at which their classes end, few and many of them (64 rows are summed
at a time), in one and in all of a thread's rows, alone and together with rows
of thousands of entries.

Bits and tolerance as in test_gpu_small_filter (the same check).  The last
test times one launch against a launch per step where eight rows hold half of
the entries: walked by one thread each, an entry at a time, they took 3.8
times as long; half of that is the line here (0.34 measured).
"""
import time

import numpy as np
import pytest

from paper_2409_15053_amd import flp
from paper_2409_15053_amd import inputs as I

from .test_gpu_small_filter import U, check, torch  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


def rows_of(lengths, seed):
    """Rows of these lengths at random columns (sorted, distinct), absolute
    row sums of 1."""
    g = np.random.Generator(np.random.PCG64(seed))
    n = len(lengths)
    cols = [np.sort(g.choice(n, size=k, replace=False)) for k in lengths]
    vals = [g.uniform(-1.0, 1.0, k) / max(k, 1) for k in lengths]
    ptr = np.concatenate([[0], np.cumsum(lengths)])
    return I.Csr(n, ptr.astype(np.int32), np.concatenate(cols).astype(np.int32), np.concatenate(vals))


def lengths(n, fill, long, where):
    """`fill` entries per row, the lengths in `long` in rows spread by
    `where`: over all of them, or next to each other."""
    k = np.full(n, fill)
    at = np.linspace(0, n - 1, len(long)).astype(int) if where == "spread" else np.arange(len(long)) + n // 3
    k[at] = long
    return k


EDGES = {
    "slots8": (3, [8, 9, 12, 13, 16, 17, 24, 25, 40, 41, 72, 73, 74]),
    "slots16": (12, [16, 17, 20, 21, 24, 25, 32, 33, 48, 49, 80, 81, 82]),
}


@pytest.mark.parametrize("prec", list(U))
@pytest.mark.parametrize("where", ["spread", "together"])
@pytest.mark.parametrize("n,name", [(600, "slots8"), (1600, "slots8"), (2500, "slots8"), (4096, "slots8"),
                                    (1000, "slots16"), (2048, "slots16"), (3000, "slots16")])
def test_class_edges(torch, n, name, where, prec):
    fill, long = EDGES[name]
    check(torch, rows_of(lengths(n, fill, long, where), n), 9, 2, prec)


@pytest.mark.parametrize("prec", list(U))
@pytest.mark.parametrize("n,fill,count,length", [
    (300, 2, 1, 300), (4096, 2, 1, 4096), (4096, 2, 3, 4000), (2049, 2, 63, 90), (2049, 2, 64, 90), (2049, 2, 65, 90),
    (4096, 2, 129, 100), (4096, 1, 250, 100), (1024, 3, 300, 18), (4096, 3, 1300, 18), (4000, 1, 2000, 13),
    (4096, 7, 4000, 8), (4096, 2, 3500, 9), (1900, 3, 700, 40)])
def test_many_and_long(torch, n, fill, count, length, prec):
    check(torch, rows_of(lengths(n, fill, [length] * count, "spread"), n + count), 6, 2, prec)


@pytest.mark.parametrize("prec", list(U))
def test_mixed(torch, prec):
    long = [2000, 900, 500] + [70] * 30 + [30] * 100 + [12] * 300 + [9] * 500
    check(torch, rows_of(lengths(4000, 2, np.random.Generator(np.random.PCG64(1)).permutation(long), "spread"), 5),
          12, 3, prec)


def test_no_slower_than_a_launch_per_step(torch):
    A = rows_of(lengths(4000, 4, [500] * 8, "spread"), 7)
    f = flp.flp_build_filter(-0.4, 0.1, 30, -1.0, 1.0)
    dA = flp.DeviceCsr.from_host(A)
    V = torch.from_numpy(I.random_block(A.n, 1, seed=1)).to("cuda:0")
    W = torch.empty_like(V)

    def best():
        t = []
        for _ in range(7):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                flp.flp_filter_apply(f, dA, V, W)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        return min(t)

    one = best()
    try:
        flp.flp_set_filter_shape(0, 0, 1)
        steps = best()
    finally:
        flp.flp_set_filter_shape(0, 0, 0)
    assert one <= 1.9 * steps, (one, steps)
