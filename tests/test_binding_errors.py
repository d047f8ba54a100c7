"""Errors raised while the binding allocates outputs and scratch keep their type: a training loop
catches torch.OutOfMemoryError to go on with a smaller batch."""
import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2512_06989_amd import mhffn


class Allocations(TorchDispatchMode):
    """Every new tensor fails with `error`."""

    def __init__(self, error):
        super().__init__()
        self.error = error

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        if "empty" in str(func):
            raise self.error
        return func(*args, **(kwargs or {}))


def _calls(N, H, E, DE, DH, device, dtype=torch.bfloat16):
    dm = H * DH
    X = torch.zeros(N, dm, dtype=dtype, device=device)
    W = [torch.zeros(H, E, DE, DH, dtype=dtype, device=device) for _ in range(3)]
    Wr = torch.zeros(H, DH, E, dtype=dtype, device=device)
    P = [torch.zeros(dm, dm, dtype=dtype, device=device) for _ in range(2)]
    return {"forward": lambda: mhffn.forward(X, *W, Wr),
            "backward": lambda: mhffn.backward(X, *W, Wr, X),
            "module_forward": lambda: mhffn.module_forward(X, P[0], *W, Wr, P[1]),
            "module_backward": lambda: mhffn.module_backward(X, P[0], *W, Wr, P[1], X, X, X)}


CALLS = ("forward", "backward", "module_forward", "module_backward")


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("error", [torch.OutOfMemoryError("no room"), KeyError("k"), MemoryError("host")])
def test_a_failed_allocation_keeps_its_type(call, error):
    fn = _calls(64, 2, 3, 64, 128, "cpu")[call]
    with pytest.raises(type(error)) as e, Allocations(error):
        fn()
    assert e.value is error


def test_an_aten_error_reads_as_torch_raises_it():
    X = torch.eye(256, dtype=torch.bfloat16).to_sparse_csr()
    W = [torch.zeros(2, 3, 64, 128, dtype=torch.bfloat16) for _ in range(3)]
    with pytest.raises(RuntimeError) as want:
        X.stride(1)
    with pytest.raises(RuntimeError) as got:
        mhffn.forward(X, *W, torch.zeros(2, 128, 3, dtype=torch.bfloat16))
    assert str(got.value) == str(want.value)   # (no C++ backtrace)


@pytest.mark.gpu
@pytest.mark.parametrize("call", CALLS)
def test_out_of_memory_on_the_gpu(call):
    fn = _calls(1 << 19, 2, 2, 32, 128, "cuda")[call]     # every output of N rows: 256 MiB
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError) as e:
            fn()
        assert "Exception raised from" not in str(e.value)   # no C++ backtrace in the message
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
