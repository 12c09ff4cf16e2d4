"""The filter launch configuration that a solve reports: a step's shape where
steps are launched, none where a small matrix is filtered in one launch."""
import pytest

from paper_2409_15053_amd import flp
from paper_2409_15053_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPE = ("filter_lanes_per_row", "filter_cols_per_lane", "filter_streaming_loads", "filter_tile_chunk",
         "filter_lds_window", "filter_window_halo")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible MI355X"
    flp.load()
    return t


@pytest.mark.parametrize("prec", [flp.FLP_PREC_FP64, flp.FLP_PREC_FP32_FILTER], ids=["fp64", "fp32"])
def test_reported_shape(torch, prec):
    def stats(A):
        return flp.flp_solve(flp.DeviceCsr.from_host(A, with_fp32=True), 0.0, 0.3, block=4, degree=30,
                             prec=prec)["stats"]

    small = stats(I.laplacian_3d(15))
    assert [small[k] for k in SHAPE] == [0] * len(SHAPE) and small["filter_group_width"] == 4
    large = stats(I.laplacian_3d(18))
    assert large["filter_lanes_per_row"] * large["filter_cols_per_lane"] >= large["filter_group_width"] > 0
    try:
        flp.flp_set_filter_shape(0, 0, 4)
        forced = stats(I.laplacian_3d(15))
    finally:
        flp.flp_set_filter_shape(0, 0, 0)
    assert forced["filter_lanes_per_row"] * forced["filter_cols_per_lane"] >= 4
