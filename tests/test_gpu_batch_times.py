"""Phase times of a batch's solves: the bounds estimate is one run for all of
them, so their shares of it add up to no more than the batch's set-up, in
which it lies, and follow the matrices' sizes."""
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


def test_bounds_time_is_shared(torch):
    sizes = [8] * 48 + [16] * 16
    dAs = [flp.DeviceCsr.from_host(I.laplacian_3d(g)) for g in sizes]
    res, st = flp.flp_solve_batch(dAs, [0.0] * 64, [0.3 if g == 16 else 0.9 for g in sizes], block=4)
    t = [r["stats"]["t_pre"] for r in res]
    assert min(t) > 0.0
    assert sum(t) <= st["t_setup"] * (1 + 1e-12)
    w = [dA.nnz + dA.n for dA in dAs]
    assert all(abs(x - sum(t) * y / sum(w)) <= 1e-9 * sum(t) for x, y in zip(t, w))
