"""The module at decode-sized batches: its projections run on the few-rows product kernel (blocks
of 32 rows), in the forward and in the backward form, on row counts at the edges of those
blocks, contractions that leave some of its waves without a slice or give them several, and on
both sides of the rule that picks it.  Stage by stage against the oracle, like the other module tests."""
import pytest

from tests.helpers import small_workload
from tests.test_gpu_module import _stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,dh", [(1, 3, 64), (31, 16, 128), (32, 1, 64), (33, 2, 128), (64, 9, 128),
                                    (65, 1, 256), (127, 10, 128), (128, 3, 64), (129, 2, 128),
                                    (384, 16, 128), (385, 16, 128), (50, 18, 256)])
def test_projections_of_few_rows(N, H, dh):
    _stages(small_workload("module_decode", N, H, 2, 64, "bf16", dh=dh, backward=True), seed=N)
