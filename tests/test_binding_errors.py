"""Errors raised inside the native binding are Python exceptions of the type torch gives them: a
training loop catches torch.OutOfMemoryError to go on with a smaller batch, and tensors without
memory of their own (those of torch.func) are refused with torch's own message."""
import gc
import subprocess
import sys

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


WRAPPED = """
import types
import torch
from paper_2512_06989_amd import mhffn
X = torch.zeros(8, 256, dtype=torch.bfloat16)
W = [torch.zeros(2, 3, 64, 128, dtype=torch.bfloat16) for _ in range(3)]
Wr, P = torch.zeros(2, 128, 3, dtype=torch.bfloat16), torch.zeros(256, 256, dtype=torch.bfloat16)
stream = types.SimpleNamespace(cuda_stream=0)
ws = torch.zeros(8)
calls = {"forward": lambda x: mhffn.forward(x, *W, Wr, stream=stream, workspace=ws),
         "forward_out": lambda x: mhffn.forward(X, *W, Wr, out=x, stream=stream, workspace=ws),
         "forward_static": lambda x: mhffn.forward_static(x, *W, Wr, X, stream=stream),
         "backward": lambda x: mhffn.backward(x, *W, Wr, X, stream=stream, workspace=ws),
         "module_forward": lambda x: mhffn.module_forward(x, P, *W, Wr, P, stream=stream, workspace=ws)[0],
         "module_backward": lambda x: mhffn.module_backward(x, P, *W, Wr, P, X, X, X, stream=stream, workspace=ws)}
for name, call in calls.items():
    for transform in (lambda f: torch.vmap(f)(torch.stack([X, X])), lambda f: torch.func.grad(lambda x: f(x).sum())(X)):
        try:
            transform(call)
            print(name, "passed")
        except RuntimeError as e:
            print(name, "storage" in str(e))
"""


def test_tensors_without_memory_are_refused():
    """(a process of its own: an exception that leaves the binding without the interpreter lock ends it)"""
    r = subprocess.run([sys.executable, "-W", "ignore", "-c", WRAPPED], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-400:]
    lines = r.stdout.split("\n")[:-1]
    assert len(lines) == 12 and all(line.endswith(" True") for line in lines), r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("call", CALLS)
def test_out_of_memory_on_the_gpu(call):
    fn = _calls(1 << 19, 2, 2, 32, 128, "cuda")[call]     # every output of N rows: 256 MiB
    torch.cuda.synchronize()
    gc.collect()   # (an exception kept by pytest.raises is a cycle: the case before would free its tensors at any time)
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError) as e:
            fn()
        assert "Exception raised from" not in str(e.value)   # no C++ backtrace in the message
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
