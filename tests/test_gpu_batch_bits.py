"""A batched solve's bits do not depend on the solves that run beside it: the
same matrix alone in a batch and with other matrices, smaller and larger, that
leave it earlier and later.  Row counts on both sides of the sizes at which a
solve's passes take one row block and many, and its partial Gram matrices are
few or many (8192 numbers)."""
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


def problem(g, count):
    """g^3 Laplacian with a separable potential, so that its lowest `count`
    eigenvalues' interval is known."""
    field, *axes = I.separable_potential(g, 100 + g)
    lap = 2 * np.eye(g) - np.eye(g, k=1) - np.eye(g, k=-1)
    a, b, c = (np.linalg.eigvalsh(lap + np.diag(v)) for v in axes)
    lam = np.sort((a[:, None, None] + b[None, :, None] + c[None, None, :]).reshape(-1))[:count + 1]
    return I.laplacian_3d(g, field), lam[0] - 0.5, 0.5 * (lam[count - 1] + lam[count])


@pytest.mark.parametrize("g,block,prec", [(16, 8, flp.FLP_PREC_FP64), (30, 8, flp.FLP_PREC_FP64),
                                          (30, 8, flp.FLP_PREC_FP32_FILTER), (40, 4, flp.FLP_PREC_FP64),
                                          (26, 16, flp.FLP_PREC_FP64)])
def test_bits_in_any_company(torch, g, block, prec):
    def run(others):
        probs = [problem(g, 24)] + [problem(h, c) for h, c in others]
        dAs = [flp.DeviceCsr.from_host(A, with_fp32=True) for A, _, _ in probs]
        res, _ = flp.flp_solve_batch(dAs, [p[1] for p in probs], [p[2] for p in probs], block=block, degree=40,
                                     prec=prec, check_every=8, seeds=[11 + i for i in range(len(probs))])
        return res[0]

    alone = run([])
    assert alone["count"] == 24
    for others in ([(12, 6)], [(20, 30), (34, 20), (9, 4)], [(45, 30)]):
        res = run(others)
        assert res["stats"]["basis_cols"] == alone["stats"]["basis_cols"]
        assert np.array_equal(res["evals"], alone["evals"])
        assert np.array_equal(res["resid"], alone["resid"])
        assert torch.equal(res["evecs"], alone["evecs"])
