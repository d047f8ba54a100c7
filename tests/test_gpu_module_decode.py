"""The module at decode-sized batches: its projections run on the few-rows product kernel (blocks
of 32 rows), in the forward and in the backward form, on row counts at the edges of those
blocks, contractions that leave some of its waves without a slice, give them several, or take its
loop around a second time (more than 32 slices of 64), and on both sides of the rule that picks
it.  Stage by stage against the oracle, like the other module tests."""
import pytest

from paper_2512_06989_amd import mhffn
from tests.helpers import launch_plan, small_workload
from tests.test_gpu_module import _stages

FEW = [(1, 3, 64), (31, 16, 128), (32, 1, 64), (33, 2, 128), (64, 9, 128), (65, 1, 256), (127, 10, 128),
       (128, 3, 64), (129, 2, 128), (64, 20, 128), (96, 20, 128), (128, 16, 128), (512, 8, 128)]
TILED = [(384, 16, 128), (385, 16, 128), (50, 18, 256), (97, 20, 128), (129, 16, 128), (513, 8, 128)]


@pytest.mark.parametrize("N,H,dh", FEW + TILED)
def test_the_cases_take_the_kernel_they_name(N, H, dh):
    plan = launch_plan(mhffn.OP_MODULE_BACKWARD, N, H, 2, 64, dh=dh)
    assert plan.startswith("rows few rows;") == ((N, H, dh) in FEW), plan


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,dh", FEW + TILED)
def test_projections_of_few_rows(N, H, dh):
    _stages(small_workload("module_decode", N, H, 2, 64, "bf16", dh=dh, backward=True), seed=N)
