"""The work list of the pipelined bf16 forward (d_h = 128, up to 64 sub-networks, more than 128
tokens): whole blocks of 256 tokens, blocks cut in halves of 128 (with an empty or ragged second half)
alone and behind whole rounds; up to 128 blocks, tiles in equal shares and, of halves, with one
shorter share.  Oracle parity at
the bf16 bar with the per-row bound on the heads at both ends, and run-to-run bit identity."""
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import inputs, mhffn
from tests.helpers import TOL, check_parity, device_inputs, launch_plan, small_workload, to_host
from tests.test_gpu_forward import run_forward

# N, H, E, d_e, R given, plan
CASES = [
    (129, 3, 1, 32, False, "whole=0 units=6x128 tiles=1x1+0 shares=1"),
    (130, 2, 64, 64, True, "whole=0 units=4x128 tiles=32x4+0 shares=32"),
    (300, 16, 8, 128, False, "whole=0 units=48x128 tiles=4x8+0 shares=4"),
    (700, 5, 64, 32, False, "whole=0 units=30x128 tiles=6x11+0 shares=6"),
    (1000, 16, 22, 32, True, "whole=0 units=128x128 tiles=1x22+0 shares=1"),
    (2049, 8, 20, 256, False, "whole=0 units=72x256 tiles=3x54+0 shares=3"),
    (1800, 12, 20, 384, False, "whole=0 units=96x256 tiles=2x120+0 shares=2"),
    (193, 26, 14, 352, False, "whole=0 units=52x128 tiles=4x37+6 shares=5"),      # a second half of 65 tokens
    (141, 15, 31, 192, True, "whole=0 units=30x128 tiles=8x23+2 shares=9"),       # and one of 13
    (2200, 17, 33, 32, False, "whole=153 units=0x256 tiles=1x33+0 shares=1"),
    (4097, 17, 2, 64, False, "whole=256 units=66x128 tiles=1x4+0 shares=1"),
    (4480, 16, 40, 64, True, "whole=256 units=64x128 tiles=1x80+0 shares=1"),
    (66000, 1, 64, 64, False, "whole=256 units=4x128 tiles=1x128+0 shares=1"),
]


@pytest.mark.parametrize("N,H,E,de,route_weights,plan", CASES)
def test_plan(N, H, E, de, route_weights, plan):
    assert launch_plan(mhffn.OP_FORWARD, N, H, E, de) == "flow " + plan
    d = mhffn.Desc(N, H, 128, E, de, 0, 0, mhffn.BF16, mhffn.ROUTE_PARAMS, 1e-6)
    units, shares = plan.split("units=")[1].split()[0].split("x"), int(plan.split("shares=")[1])
    want = int(units[0]) * int(units[1]) * 128 * 4 * shares if shares > 1 else 0
    assert mhffn.workspace_bytes(d, mhffn.OP_FORWARD) == want


def test_scratch_never_exceeds_what_the_interface_states():
    """32 MiB, whatever the token count: callers hold workspaces of that size."""
    import random
    rng = random.Random(1)
    for _ in range(20000):
        d = mhffn.Desc(int(2 ** rng.uniform(0, 21)), rng.randint(1, 300), 128, rng.randint(1, 64), 32 * rng.randint(1, 32),
                       0, 0, mhffn.BF16, mhffn.ROUTE_PARAMS, 1e-6)
        assert mhffn.workspace_bytes(d, mhffn.OP_FORWARD) <= 32 << 20


def test_plan_of_many_long_rounds():
    """8256 blocks of 2^19 tiles: their product has 33 bits.  The plan is that of half the tiles."""
    a, b = (launch_plan(mhffn.OP_FORWARD, 256 * 8256, 1, 64, de) for de in (1 << 17, 1 << 18))
    assert a.split(" tiles=")[0] == b.split(" tiles=")[0] == "flow whole=8256 units=0x256", (a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,E,de,route_weights,plan", CASES)
def test_flow_forward(N, H, E, de, route_weights, plan):
    import torch
    w = small_workload("flow", N, H, E, de, "bf16")
    d, Y = run_forward(w, seed=N + E, route_weights=route_weights)
    for h in sorted({0, H - 1}):                      # heads are independent
        c = slice(h * 128, (h + 1) * 128)
        rows = slice(0, N) if N <= 5000 else slice(N - 600, N)   # and tokens
        one = [d[k][h:h + 1] for k in ("W_gate", "W_up", "W_down")]
        one.append(d["R"][rows, h:h + 1] if route_weights else d["W_r"][h:h + 1])
        want = orc.forward(d["X"][rows, c], *one, w.eps, orc.ROUTE_WEIGHTS if route_weights else orc.ROUTE_PARAMS)
        check_parity({"Y": Y[rows, c]}, {"Y": want}, TOL["bf16"], 128, "flow, head %d" % h)
    g = device_inputs(d, "bf16")
    key, mode = ("R", mhffn.ROUTE_WEIGHTS) if route_weights else ("W_r", mhffn.ROUTE_PARAMS)
    again = [mhffn.forward(g["X"], g["W_gate"], g["W_up"], g["W_down"], g[key], w.eps, mode) for _ in range(2)]
    assert torch.equal(again[0], again[1])
    assert (to_host(again[0]) == Y).all()


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,E,de,route_weights,plan", [c for c in CASES if c[0] in (141, 1000, 2200, 4097)])
def test_strided_rows(N, H, E, de, route_weights, plan):
    """Rows of X and Y wider than d_model and than each other: whole blocks, halves beside whole
    rounds, halves alone (all store Y themselves) and the sum over shares."""
    import torch
    w = small_workload("flow_strided", N, H, E, de, "bf16")
    g = device_inputs(inputs.make_inputs(w, seed=N, with_dy=False, route_weights=route_weights), "bf16")
    key, mode = ("R", mhffn.ROUTE_WEIGHTS) if route_weights else ("W_r", mhffn.ROUTE_PARAMS)
    a, dm = [g[k] for k in ("W_gate", "W_up", "W_down", key)], w.d_model
    want = mhffn.forward(g["X"], *a, w.eps, mode)
    Xs = torch.full((N, dm + 40), float("nan"), dtype=torch.bfloat16, device="cuda")
    Xs[:, :dm] = g["X"]
    Ys = torch.full((N, dm + 72), 7.0, dtype=torch.bfloat16, device="cuda")
    mhffn.forward(Xs[:, :dm], *a, w.eps, mode, out=Ys[:, :dm])
    assert torch.equal(Ys[:, :dm], want) and torch.all(Ys[:, dm:] == 7.0)
