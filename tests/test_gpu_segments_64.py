"""Weight-major backward at d_h = 64: token segments per neuron group by what the fullest CU gets, from
one to eight, with a shorter last segment and a ragged last block, for one group and for several
heads with several groups (also with an idle pair of waves in a head's last one).  Weight gradients
of the heads at both ends against the oracle, and run-to-run bit identity."""
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import inputs, mhffn
from tests.helpers import TOL, check_parity, device_inputs, launch_plan, small_workload, to_host

WANT = ("dW_gate", "dW_up", "dW_down")
CASES = [(363, 1, 1, 32, 1), (1013, 1, 1, 32, 2), (1840, 1, 1, 32, 3), (2139, 1, 1, 32, 4),
         (2807, 1, 1, 32, 5), (3075, 1, 1, 32, 6), (3610, 1, 1, 32, 7), (4723, 1, 1, 32, 8),
         (2000, 4, 8, 128, 3), (4000, 8, 8, 128, 4), (4000, 3, 5, 96, 7)]


@pytest.mark.parametrize("N,H,E,de,segs", CASES)
def test_plan(N, H, E, de, segs):
    assert "; wgt segs=%d;" % segs in launch_plan(mhffn.OP_BACKWARD, N, H, E, de, dh=64)


@pytest.mark.parametrize("N,H,E,de,segs", [
    (31102, 25, 49, 448, 1), (32212, 23, 54, 480, 1),   # two segments: 804 and 874 MiB for nothing
    (28119, 12, 33, 288, 1), (26753, 21, 33, 160, 1),   # 167 and 162 MiB for less than the model's error
    (5000, 16, 14, 192, 1), (16384, 16, 14, 192, 3), (6940, 17, 16, 256, 2)])
def test_scratch_is_taken_for_a_gain_only(N, H, E, de, segs):
    test_plan(N, H, E, de, segs)


@pytest.mark.parametrize("N,H,E,de,dense,wide", [(8000, 10, 8, 128, 3, 3), (5000, 16, 14, 192, 1, 3),
                                                 (2013, 9, 12, 224, 2, 1), (20460, 6, 11, 160, 3, 3)])
def test_generic_kernel_is_planned_with_its_own_occupancy(N, H, E, de, dense, wide):
    """Row strides from 2^24 on take the kernel of which a CU holds two workgroups."""
    test_plan(N, H, E, de, dense)
    for ld in ((1 << 24, 0), (0, 1 << 24)):
        assert "; wgt segs=%d;" % wide in launch_plan(mhffn.OP_BACKWARD, N, H, E, de, dh=64, ld=ld)


@pytest.mark.gpu
@pytest.mark.parametrize("N,H,E,de,segs", CASES)
def test_weight_gradients(N, H, E, de, segs):
    import torch
    w = small_workload("segments64", N, H, E, de, "bf16", dh=64, backward=True)
    d = inputs.make_inputs(w, seed=N + E, with_dy=True)
    g = device_inputs(d, "bf16")
    a = [g[k] for k in ("X", "W_gate", "W_up", "W_down", "W_r", "dY")]
    got = mhffn.backward(*a, w.eps, want=WANT)
    again = mhffn.backward(*a, w.eps, want=WANT)
    for k in WANT:
        assert torch.equal(got[k], again[k]), k
    for h in sorted({0, H - 1}):                      # heads are independent
        c, hs = slice(h * 64, (h + 1) * 64), slice(h, h + 1)
        one = [d[k][hs] for k in ("W_gate", "W_up", "W_down", "W_r")]
        want = orc.backward(d["X"][:, c], *one, d["dY"][:, c], w.eps)
        check_parity({k: to_host(got[k])[hs] for k in WANT}, want, TOL["bf16"], 64, "segments, head %d" % h)
