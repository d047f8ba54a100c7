"""The work list of the bf16 token-major backward: whole token blocks beside blocks whose
sub-networks are shared out, in equal shares and with a shorter last one.  The heads at both ends
(whole blocks lie in the first, shared ones in the last) against the oracle, run-to-run bit
identity, and the same dX when it is the only gradient asked for."""
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import inputs, mhffn
from tests.helpers import TOL, check_parity, device_inputs, launch_plan, small_workload, to_host

# N, H, d_h, E, d_e, R given, shares
CASES = [
    (4200, 17, 128, 4, 128, False, "4 of 33"),      # 256 whole blocks and 33
    (332, 33, 128, 13, 256, False, "3+1 of 66"),
    (2100, 32, 64, 8, 64, True, "8 of 32"),         # 512 whole blocks and 32
    (552, 36, 64, 9, 224, False, "2+1 of 180"),
    (4200, 9, 256, 5, 96, False, "3 of 41"),
    (304, 30, 256, 9, 224, True, "2+1 of 90")]


@pytest.mark.parametrize("N,H,dh,E,de,route_weights,shares", CASES)
def test_plan(N, H, dh, E, de, route_weights, shares):
    plan = launch_plan(mhffn.OP_BACKWARD, N, H, E, de, dh=dh, route_weights=route_weights)
    assert " shares=%s;" % shares in plan, plan


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,dh,E,de,route_weights,shares", CASES)
def test_backward(N, H, dh, E, de, route_weights, shares):
    import torch
    w = small_workload("lists", N, H, E, de, "bf16", dh=dh, backward=True)
    d = inputs.make_inputs(w, seed=N + E, with_dy=True, route_weights=route_weights)
    g = device_inputs(d, "bf16")
    key, mode = ("R", mhffn.ROUTE_WEIGHTS) if route_weights else ("W_r", mhffn.ROUTE_PARAMS)
    a = [g[k] for k in ("X", "W_gate", "W_up", "W_down", key)]
    got = mhffn.backward(*a, g["dY"], w.eps, mode)
    again = mhffn.backward(*a, g["dY"], w.eps, mode)
    for k in got:
        assert torch.equal(got[k], again[k]), k
    assert torch.equal(mhffn.backward(*a, g["dY"], w.eps, mode, want=("dX",))["dX"], got["dX"])
    dm = H * dh
    Xs, dXs = (torch.full((N, dm + 24), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    dYs = torch.full((N, dm + 56), 7.0, dtype=torch.bfloat16, device="cuda")
    Xs[:, :dm], dYs[:, :dm] = g["X"], g["dY"]
    mhffn.backward(Xs[:, :dm], *a[1:], dYs[:, :dm], w.eps, mode, want=("dX",), out={"dX": dXs[:, :dm]})
    assert torch.equal(dXs[:, :dm], got["dX"]) and torch.all(dXs[:, dm:] == 7.0)
    for h in (0, H - 1):                              # heads are independent
        c, hs = slice(h * dh, (h + 1) * dh), slice(h, h + 1)
        one = [d[k][hs] for k in ("W_gate", "W_up", "W_down")] + [d["R"][:, hs] if route_weights else d["W_r"][hs]]
        want = orc.backward(d["X"][:, c], *one, d["dY"][:, c], w.eps, mode)
        part = {k: to_host(v) for k, v in got.items()}
        part = {k: v[:, c] if k == "dX" else v[:, hs] if k == "d_route" and route_weights else v[hs] for k, v in part.items()}
        check_parity(part, want, TOL["bf16"], dh, "lists, head %d" % h, route_weights)
