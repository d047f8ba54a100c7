"""The projection products of the module on every tile shape (256 x 256, 256 x 128, 128 x 128,
64 x 128), split and unsplit contractions, row and column counts at the edges of the tiles and
token counts (the contraction of the weight gradients) that end inside a slice of k.  Stage by
stage against the oracle on sampled rows and columns.  Each case says which shapes the products
with the tokens as rows and the weight gradients take, and checks that they do."""
import numpy as np
import pytest

from paper_2512_06989_amd import mhffn
from tests.helpers import launch_plan, small_workload
from tests.test_gpu_module import _stages

CASES = [
    (1023, 8, 128, "64x128 splits=1", "128x128 splits=4"),
    (2049, 15, 128, "128x128 splits=1", "128x128 splits=1"),     # 1920 columns
    (4097, 16, 128, "256x256 splits=1", "128x128 splits=1"),
    (8200, 8, 256, "256x128 splits=1", "256x256 splits=4"),
    (705, 5, 64, "few rows", "128x128 splits=1"),
    (2501, 5, 64, "64x128 splits=1", "128x128 splits=10"),       # 320 columns: the last column tile is half empty
    (3001, 21, 64, "256x128 splits=1", "128x128 splits=2"),      # 1344 columns: the same
    (16380, 8, 128, "256x256 splits=1", "256x128 splits=8")]


@pytest.mark.parametrize("N,H,dh,rows,weights", CASES)
def test_the_cases_take_the_shapes_they_name(N, H, dh, rows, weights):
    plan = launch_plan(mhffn.OP_MODULE_BACKWARD, N, H, 2, 32, dh=dh)
    assert plan.startswith("rows %s; weights %s; " % (rows, weights)), plan


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,dh", [c[:3] for c in CASES])
def test_every_tile_shape(N, H, dh):
    rng = np.random.default_rng(N)
    rows = np.unique(np.concatenate([[0, 63, 64, 127, 128, 255, 256, N - 1], rng.choice(N, size=120, replace=False)]))
    cols = np.unique(np.concatenate([[0, 127, 128, H * dh - 1], rng.choice(H * dh, size=60, replace=False)]))
    _stages(small_workload("gemm_tiles", N, H, 2, 32, "bf16", dh=dh, backward=True), seed=N, heads=(0,),
            rows=rows, cols=cols)
