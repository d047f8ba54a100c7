"""Scratch that the binding allocates for a call on a given stream belongs to that stream: freed
when the call returns, it must not go to the next tensor of the current stream while the kernels
still use it."""
import pytest

from paper_2512_06989_amd import inputs, mhffn
from tests.helpers import device_inputs, small_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("call", ["forward", "backward", "module_forward", "module_backward"])
def test_scratch_lives_on_the_stream_of_the_call(dtype, call):
    import torch
    N, H, E, de, dh = 500, 2, 4, 64, 128
    w = small_workload("stream", N, H, E, de, dtype, dh=dh, backward=True)
    g = device_inputs(inputs.make_inputs(w, seed=2, with_dy=True), dtype)
    W, Wr, X, dY = [g[k] for k in ("W_gate", "W_up", "W_down")], g["W_r"], g["X"], g["dY"]
    P = [torch.eye(H * dh, device="cuda", dtype=X.dtype) for _ in range(2)]
    op, args = {"forward": (mhffn.OP_FORWARD, (X, *W, Wr)),
                "backward": (mhffn.OP_BACKWARD, (X, *W, Wr, dY)),
                "module_forward": (mhffn.OP_MODULE_FORWARD, (X, P[0], *W, Wr, P[1])),
                "module_backward": (mhffn.OP_MODULE_BACKWARD, (X, P[0], *W, Wr, P[1], X, X, dY))}[call]
    fn = getattr(mhffn, call)
    need = mhffn.workspace_bytes(mhffn.make_desc(X, W[0], mhffn.ROUTE_PARAMS, 1e-6), op)
    assert need > 0
    flat = lambda r: list(r.values()) if isinstance(r, dict) else list(r) if isinstance(r, tuple) else [r]  # noqa: E731
    want = flat(fn(*args))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()

    def held():
        return sum(s["total_size"] for s in torch.cuda.memory_snapshot() if s["stream"] == side.cuda_stream)

    assert held() == 0
    got = flat(fn(*args, stream=side))
    assert held() >= need
    assert torch.cuda.current_stream() != side
    side.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
