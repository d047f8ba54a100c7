"""The module's projections of up to 16 rows (8 where the weights lie in row form): row counts at
both limits and one beyond, contractions of one slice of 64 (15 of 16 waves have none), of an odd
number of slices, and of two slices for every wave.  Stage by stage against the oracle; strided X
and O give the bits of dense ones."""
import pytest

from paper_2512_06989_amd import mhffn
from tests.helpers import launch_plan, small_workload
from tests.test_gpu_module import _stages

CASES = [(1, 1, 64), (7, 3, 64), (8, 1, 128), (9, 9, 64), (15, 16, 128), (16, 2, 64), (16, 16, 128), (17, 16, 128)]


@pytest.mark.parametrize("N,H,dh", CASES)
def test_plan(N, H, dh):
    assert launch_plan(mhffn.OP_MODULE_BACKWARD, N, H, 2, 32, dh=dh).startswith("rows few rows;")
    for op, rows in ((mhffn.OP_MODULE_FORWARD, 16), (mhffn.OP_MODULE_BACKWARD, 8)):
        assert launch_plan(op, N, H, 2, 32, dh=dh).endswith("; few rows columns=%d" % (16 if N <= rows else 32))


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,dh", CASES)
def test_projections(N, H, dh):
    _stages(small_workload("module_few", N, H, 2, 32, "bf16", dh=dh, backward=True), seed=N + H)


@pytest.mark.gpu
def test_strided_rows():
    import torch
    dm, wide = 512, 512 + 24
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    n = lambda *s: (torch.randn(*s, generator=g, device="cuda") * 0.05).to(torch.bfloat16)  # noqa: E731
    X, Wi, Wo, Wr = n(11, dm), n(dm, dm), n(dm, dm), n(4, 128, 3)
    W = [n(4, 3, 32, 128) for _ in range(3)]
    want = mhffn.module_forward(X, Wi, *W, Wr, Wo, 1e-6)
    Xs = torch.full((11, wide), float("nan"), dtype=torch.bfloat16, device="cuda")
    Xs[:, :dm] = X
    Os = torch.full((11, wide + 8), 7.0, dtype=torch.bfloat16, device="cuda")
    got = mhffn.module_forward(Xs[:, :dm], Wi, *W, Wr, Wo, 1e-6, out={"O": Os[:, :dm]})
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    assert torch.equal(Os[:, :dm], want[0]) and torch.all(Os[:, dm:] == 7.0)
