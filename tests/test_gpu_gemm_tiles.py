"""The projection products of the module on every tile shape (256 x 256, 256 x 128, 128 x 128,
64 x 128), split and unsplit contractions, row and column counts at the edges of the tiles and
token counts (the contraction of the weight gradients) that end inside a slice of k.  Stage by
stage against the oracle on sampled rows and columns."""
import numpy as np
import pytest

from tests.helpers import small_workload
from tests.test_gpu_module import _stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,dh", [
    (1023, 8, 128),     # 64 x 128 tiles forward, 128 x 128 split weight gradients, ragged slice
    (2049, 15, 128),    # 1920 columns: tiles of 128 x 128, edges on both sides
    (4097, 16, 128),    # 256 x 128
    (8200, 8, 256),     # 256 x 256
    (705, 5, 64)])      # 320 columns: the last column tile is half empty
def test_every_tile_shape(N, H, dh):
    rng = np.random.default_rng(N)
    rows = np.unique(np.concatenate([[0, 63, 64, 127, 128, 255, 256, N - 1], rng.choice(N, size=120, replace=False)]))
    cols = np.unique(np.concatenate([[0, 127, 128, H * dh - 1], rng.choice(H * dh, size=60, replace=False)]))
    _stages(small_workload("gemm_tiles", N, H, 2, 32, "bf16", dh=dh, backward=True), seed=N, heads=(0,),
            rows=rows, cols=cols)
