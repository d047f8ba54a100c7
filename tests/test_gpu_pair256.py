"""bf16 forward at d_h = 256 with up to 16 sub-networks: two waves share 32 tokens and a
workgroup takes 128 (the tiles of a share: one, two, three and more; one share and several;
ragged token blocks; 16 sub-networks, the most it takes, and 17).  Oracle parity at the bf16 bar
with the per-row bound, and run-to-run bit identity."""
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import mhffn
from tests.helpers import TOL, check_parity, device_inputs, launch_plan, small_workload, to_host
from tests.test_gpu_forward import oracle_forward, run_forward


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,E,de,route_weights", [
    (1, 1, 1, 32, False), (15, 2, 1, 64, False), (16, 1, 3, 32, False), (33, 3, 2, 96, True),
    (127, 2, 16, 32, False), (129, 1, 16, 64, True), (128, 8, 17, 32, False), (200, 2, 4, 704, False),
    # a share of two, three and four tiles over whole heads (more than 128 token blocks)
    (2060, 8, 1, 64, False), (2060, 8, 1, 96, False), (2060, 8, 2, 64, True)])
def test_pair_forward(N, H, E, de, route_weights):
    import torch
    w = small_workload("pair", N, H, E, de, "bf16", dh=256)
    d, Y = run_forward(w, seed=N + E, route_weights=route_weights)
    want = oracle_forward(d, w, route_weights=route_weights)
    check_parity({"Y": Y}, {"Y": want}, TOL["bf16"], 256, "pair")
    g = device_inputs(d, "bf16")
    key, mode = ("R", mhffn.ROUTE_WEIGHTS) if route_weights else ("W_r", mhffn.ROUTE_PARAMS)
    again = [mhffn.forward(g["X"], g["W_gate"], g["W_up"], g["W_down"], g[key], w.eps, mode) for _ in range(2)]
    assert torch.equal(again[0], again[1])
    assert (to_host(again[0]) == Y).all()


# 129 .. 383 token blocks: one or two whole rounds of workgroups, or more of less depth where a head
# has enough tiles (the pair kernel and the one for more sub-networks)
UNEVEN = [(800, 20, 4, 96, 1), (800, 20, 5, 416, 3), (1000, 20, 17, 96, 3), (1000, 25, 17, 96, 1), (1000, 25, 5, 416, 1),
          (1300, 24, 4, 64, 1), (1300, 24, 16, 96, 2), (1281, 24, 4, 416, 2), (1900, 24, 17, 32, 1), (1281, 24, 17, 96, 2),
          (1280, 24, 48, 64, 1), (2049, 24, 48, 64, 1)]


@pytest.mark.parametrize("N,H,E,de,shares", UNEVEN)
def test_uneven_rounds_are_shared_out(N, H, E, de, shares):
    assert launch_plan(mhffn.OP_FORWARD, N, H, E, de, dh=256).endswith(" shares=%d" % shares), launch_plan(mhffn.OP_FORWARD, N, H, E, de, dh=256)


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,E,de", [c[:4] for c in UNEVEN if c[4] == 2])
def test_uneven_rounds(N, H, E, de):
    w = small_workload("uneven", N, H, E, de, "bf16", dh=256)
    d, Y = run_forward(w, seed=N + E)
    for h in (0, H - 1):                              # heads are independent
        c = slice(h * 256, (h + 1) * 256)
        one = [d[k][h:h + 1] for k in ("W_gate", "W_up", "W_down", "W_r")]
        want = orc.forward(d["X"][:, c], *one, w.eps)
        check_parity({"Y": Y[:, c]}, {"Y": want}, TOL["bf16"], 256, "uneven rounds, head %d" % h)
