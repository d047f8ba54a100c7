"""bf16 token-major backward with few tokens: the sub-networks of a token block are shared out
over workgroups and bwd_finish.hip adds the partial dX up and takes the routing derivative.
Oracle parity at the bf16 bar with the per-row bound, run-to-run bit identity, and every
gradient-request subset that changes what the last step does."""
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import inputs, mhffn
from tests.helpers import TOL, check_parity, device_inputs, launch_plan, small_workload, to_host

CASES = [
    (1, 1, 128, 2, 32, False), (255, 2, 128, 7, 64, False), (257, 3, 128, 44, 32, True),
    (300, 2, 128, 90, 32, False),                 # register-staged tiles (E > 88)
    (129, 2, 64, 5, 96, False), (128, 1, 64, 33, 32, True),
    (127, 2, 256, 3, 64, False), (130, 1, 256, 40, 32, True),    # (E > 32: register-staged)
    (1, 1, 128, 8, 64, False), (127, 2, 256, 6, 96, False), (1, 2, 256, 12, 64, True),
    (128, 4, 256, 7, 32, True), (128, 4, 256, 13, 32, True)]
ONE_SHARE = [CASES[0], CASES[6], CASES[11]]       # too little work to share out


@pytest.mark.parametrize("N,H,dh,E,de,route_weights", CASES)
def test_the_cases_are_shared_out(N, H, dh, E, de, route_weights):
    plan = launch_plan(mhffn.OP_BACKWARD, N, H, E, de, dh=dh, route_weights=route_weights)
    assert (" shares=1;" in plan) == ((N, H, dh, E, de, route_weights) in ONE_SHARE), plan


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,dh,E,de,route_weights", CASES)
def test_shared_sub_networks(N, H, dh, E, de, route_weights):
    import torch
    w = small_workload("shares", N, H, E, de, "bf16", dh=dh, backward=True)
    d = inputs.make_inputs(w, seed=N + E, with_dy=True, route_weights=route_weights)
    g = device_inputs(d, "bf16")
    key, mode = ("R", mhffn.ROUTE_WEIGHTS) if route_weights else ("W_r", mhffn.ROUTE_PARAMS)
    names = ("X", "W_gate", "W_up", "W_down", key)
    a = [g[k] for k in names]
    got = mhffn.backward(*a, g["dY"], w.eps, mode)
    again = mhffn.backward(*a, g["dY"], w.eps, mode)
    want = orc.backward(*[d[k] for k in names], d["dY"], w.eps, mode)
    for k in got:
        assert torch.equal(got[k], again[k]), k
    # E = 2 on one token: the two columns of dW_r cancel to their common rounding
    skip = ("d_route",) if N == 1 else ()
    check_parity({k: to_host(v) for k, v in got.items()}, want, TOL["bf16"], dh, "shares", route_weights, skip)
    for sub in (("dX",), ("d_route",), ("dW_up", "d_route")):
        part = mhffn.backward(*a, g["dY"], w.eps, mode, want=sub)
        for k in sub:
            assert torch.equal(part[k], got[k]), (sub, k)
    wide = torch.full((N, H * dh + 64), 7.0, dtype=torch.bfloat16, device="cuda")
    Xw = torch.zeros_like(wide)
    Xw[:, :H * dh] = g["X"]
    mhffn.backward(Xw[:, :H * dh], *a[1:], g["dY"], w.eps, mode, want=("dX",), out={"dX": wide[:, :H * dh]})
    assert torch.equal(wide[:, :H * dh], got["dX"]) and torch.all(wide[:, H * dh:] == 7.0)
