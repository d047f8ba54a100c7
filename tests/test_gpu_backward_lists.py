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


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,dh,E,de,route_weights,shares", [c for c in CASES if not c[5]])
def test_infinite_gating_weight(N, H, dh, E, de, route_weights, shares):
    """An infinite element of W_r: its column of dX is dp (which the workspace holds) times infinity, of the
    same kind in whole blocks, where dp is an operand of two products, and in shared ones."""
    import torch
    w = small_workload("lists_inf", N, H, E, de, "bf16", dh=dh, backward=True)
    g = device_inputs(inputs.make_inputs(w, seed=N, with_dy=True), "bf16")
    col, sub = 5, E - 1
    g["W_r"][:, col, sub] = float("inf")
    a = [g[k] for k in ("X", "W_gate", "W_up", "W_down", "W_r")]
    need = mhffn.workspace_bytes(mhffn.make_desc(a[0], a[1], mhffn.ROUTE_PARAMS, w.eps), mhffn.OP_BACKWARD)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    dX = mhffn.backward(*a, g["dY"], w.eps, want=("dX",), workspace=ws)["dX"].float().view(N, H, dh)
    at = (4 * H * E * N + 255) // 256 * 256          # R, then dp, both [H][E][N] fp32
    dp = ws[at:at + 4 * H * E * N].view(torch.float32).view(H, E, N)
    want = (dp[:, sub] * float("inf")).t()           # [N][H]: no sign and no NaN comes from elsewhere
    got = dX[:, :, col]
    assert int(torch.isinf(want).sum()) > want.numel() // 20
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got[~torch.isnan(got)], want[~torch.isnan(want)])
    rest = torch.cat([dX[:, :, :col], dX[:, :, col + 1:]], 2)
    assert torch.equal(torch.isfinite(rest).all(dim=2), torch.isfinite(dp).all(dim=1).t())
