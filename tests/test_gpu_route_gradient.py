"""bf16 dW_r: token blocks shared out over workgroups by the number of heads, one partial per
workgroup: several blocks per wave and one, a ragged last block, token counts whose rows of dp do
and do not start on 16 bytes, one to three blocks of 32 sub-networks, against the fp64 oracle at
the bf16 bar with the per-column bound."""
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import inputs, mhffn
from tests.helpers import TOL, check_parity, device_inputs, small_workload, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,dh,E,de", [
    (2500, 32, 64, 3, 32), (2501, 32, 64, 3, 32), (4130, 16, 64, 70, 32), (33, 2, 64, 96, 32),
    (2302, 16, 128, 40, 32), (1028, 24, 128, 2, 32), (131, 1, 128, 66, 32), (3, 3, 128, 5, 32),
    (1100, 8, 256, 33, 32), (129, 2, 256, 4, 32)])
def test_route_gradient(N, H, dh, E, de):
    import torch
    w = small_workload("route", N, H, E, de, "bf16", dh=dh, backward=True)
    d = inputs.make_inputs(w, seed=N + E, with_dy=True)
    g = device_inputs(d, "bf16")
    a = [g[k] for k in ("X", "W_gate", "W_up", "W_down", "W_r")]
    got = mhffn.backward(*a, g["dY"], w.eps, want=("d_route",))["d_route"]
    again = mhffn.backward(*a, g["dY"], w.eps, want=("d_route",))["d_route"]
    assert torch.equal(got, again)
    want = orc.backward(*[d[k] for k in ("X", "W_gate", "W_up", "W_down", "W_r")], d["dY"], w.eps)
    check_parity({"d_route": to_host(got)}, {"d_route": want["d_route"]}, TOL["bf16"], dh, "route")
