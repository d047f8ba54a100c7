"""bf16 forward at d_h = 64: shares per token block by how many workgroups the fullest CU gets (one,
two, three, four and more), down to whole blocks, with a last share of one tile.  Oracle parity on
the heads at both ends, and run-to-run bit identity."""
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import mhffn
from tests.helpers import TOL, check_parity, device_inputs, launch_plan, small_workload, to_host
from tests.test_gpu_forward import run_forward

CASES = [(129, 1, 3, 32, 1), (500, 8, 14, 96, 14), (1000, 16, 14, 96, 4),
         (3000, 8, 21, 64, 5), (4000, 20, 9, 64, 1), (6000, 8, 40, 128, 2),
         (5000, 16, 14, 192, 2), (2000, 31, 13, 32, 1), (6200, 15, 8, 64, 1),
         (139, 21, 26, 96, 12)]                       # 78 tiles: eleven shares of 7 and one


@pytest.mark.parametrize("N,H,E,de,shares", CASES)
def test_plan(N, H, E, de, shares):
    assert launch_plan(mhffn.OP_FORWARD, N, H, E, de, dh=64) == "tiles256 shares=%d" % shares


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,E,de,shares", CASES)
def test_forward(N, H, E, de, shares):
    import torch
    w = small_workload("shares64", N, H, E, de, "bf16", dh=64)
    d, Y = run_forward(w, seed=N + E)
    for h in sorted({0, H - 1}):                      # heads are independent
        c = slice(h * 64, (h + 1) * 64)
        want = orc.forward(d["X"][:, c], *[d[k][h:h + 1] for k in ("W_gate", "W_up", "W_down", "W_r")], w.eps)
        check_parity({"Y": Y[:, c]}, {"Y": want}, TOL["bf16"], 64, "d_h = 64, head %d" % h)
    g = device_inputs(d, "bf16")
    again = mhffn.forward(*[g[k] for k in ("X", "W_gate", "W_up", "W_down", "W_r")], w.eps)
    assert (to_host(again) == Y).all()
