"""The fp32 kernels at the edges of their tiles (16 tokens, 16 neurons, head widths rounded up
to 64, 96, 128, 192, 256), shares and block sizes, against the fp64 oracle at the fp32 parity
bar (1e-5; measured 3e-7 .. 6e-7: fp32 sums of up to a few thousand terms)."""
import numpy as np
import pytest

from oracle import mhffn_oracle as orc
from paper_2512_06989_amd import inputs, mhffn
from tests.helpers import TOL, device_inputs, relerr, to_host

pytestmark = pytest.mark.gpu
ARGS = ("X", "W_gate", "W_up", "W_down")


@pytest.mark.parametrize("N,H,dh,E,de,route_weights", [
    (1, 1, 4, 2, 1, False),          # the smallest problem: one token, one neuron per sub-network
    (15, 2, 64, 3, 16, False), (16, 1, 68, 2, 17, True), (17, 3, 96, 5, 15, False),
    (64, 2, 100, 4, 33, False), (65, 1, 192, 3, 20, True), (63, 2, 196, 2, 40, False),
    (700, 2, 128, 6, 48, True),      # shares of the sub-networks, token segments, weights given
    (513, 5, 128, 7, 100, False), (300, 1, 256, 17, 24, False),
    (20, 1, 4, 614, 1, False),       # nor those of 32: 16-token blocks, the most sub-networks the backward takes
    (40, 1, 64, 400, 2, False),      # gating rows of 64 tokens do not fit: 32-token blocks (backward)
    (30, 1, 64, 700, 1, None),       # the same for the forward alone
    (20, 2, 4, 1229, 1, None), (33, 1, 16, 1181, 2, None)])   # nor those of 32: the most the forward takes
def test_f32_tile_edges(N, H, dh, E, de, route_weights):
    import torch
    w = inputs.Workload("f32_edges", N, H, dh, E, de, "f32", w_std=0.1, route_scale=2.0, backward=True)
    d = inputs.make_inputs(w, seed=N + dh, with_dy=True, route_weights=bool(route_weights))
    g = device_inputs(d, "f32")
    key, mode = ("R", mhffn.ROUTE_WEIGHTS) if route_weights else ("W_r", mhffn.ROUTE_PARAMS)
    a, o = [g[k] for k in ARGS + (key,)], [d[k] for k in ARGS + (key,)]
    ref = orc.forward(*o, w.eps, mode)
    Y = mhffn.forward(*a, w.eps, mode)
    assert relerr(to_host(Y), ref) <= TOL["f32"]
    # the scratch is optional for fp32: without it, and through the library's own buffer
    Y0 = mhffn.forward(*a, w.eps, mode, workspace=torch.empty(0, device="cuda"))
    Ys = mhffn.forward_static(*a, torch.empty_like(Y), w.eps, mode)
    assert relerr(to_host(Y0), ref) <= TOL["f32"] and torch.equal(Ys, Y)
    if route_weights is None:
        return
    got = mhffn.backward(*a, g["dY"], w.eps, mode)
    again = mhffn.backward(*a, g["dY"], w.eps, mode)
    want = orc.backward(*o, d["dY"], w.eps, mode)
    for k in got:
        assert torch.equal(got[k], again[k]), k
        assert relerr(to_host(got[k]), want[k]) <= TOL["f32"], (k, relerr(to_host(got[k]), want[k]))
    only = mhffn.backward(*a, g["dY"], w.eps, mode, want=("d_route",))
    assert np.array_equal(to_host(only["d_route"]), to_host(got["d_route"]))
