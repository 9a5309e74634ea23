"""Full CROWN on convolutional layers by receptive-field windows.

A pass that bounds every neuron of a convolutional layer keeps its rows' coefficients on
windows of the layers below.  Checked against the FP64 oracle and against the whole-layer
passes (BOUND_OPT_GEMM_ONLY, which takes the general path) on networks whose windows meet
the layers' borders, exceed them, use every column count of the tiles (below 16, 16, 32,
64 and more), strides, paddings and kernel sizes, and on one that the windows do not cover.
Tolerance: 1e-4 relative, the parity tolerance of every FP32 bound against FP64.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import crown as O

pytestmark = pytest.mark.gpu

#         input      (channels, kernel, stride, padding) ...               FC widths
NETS = {
    "c8": ((3, 12, 12), [(8, 3, 1, 1), (8, 4, 2, 1)], (16, 4)),
    "c12_ragged": ((3, 13, 13), [(12, 3, 1, 1), (20, 4, 2, 1), (12, 3, 1, 1)], (10,)),
    "c64": ((3, 10, 10), [(64, 3, 1, 1), (32, 4, 2, 1), (96, 3, 1, 0)], (10,)),
    "pad0": ((3, 14, 14), [(16, 3, 1, 0), (16, 5, 1, 2), (32, 4, 2, 0)], (10,)),
    "wide_in": ((8, 12, 12), [(16, 3, 1, 1), (16, 3, 1, 1)], (10,)),
    "one_channel_stride2": ((1, 16, 16), [(16, 4, 2, 1), (16, 3, 1, 1)], (10,)),
    "k3_stride2": ((3, 12, 12), [(16, 3, 1, 1), (16, 3, 2, 1), (16, 3, 1, 1)], (10,)),
}


def _net(name):
    shape, convs, fc = NETS[name]
    rng = np.random.default_rng(11)
    layers = []
    for co, k, s, p in convs:
        layers.append(W._conv(rng, shape, co, k, s, p))
        shape = layers[-1]["out_shape"]
    d = int(np.prod(shape))
    for w in fc:
        layers.append(W._linear(rng, d, w))
        d = w
    return layers


@pytest.mark.parametrize("name,slack", [(n, True) for n in NETS] + [("c8", False)])
def test_window_bounds_match_oracle_and_whole_layers(name, slack):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    net = _net(name)
    n = 3
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, W.in_dim(net), 12), 0.02)
    # a workspace that no conv layer's rows fill evenly: the passes run in several chunks
    bn = N.BoundNet(net, n, 1000)
    lo, hi = (t.double().cpu().numpy() for t in bn.crown_bounds(x_lo, x_hi, slack=slack))
    B.bound_set_options(bn.handle, B.BOUND_OPT_GEMM_ONLY)
    dlo, dhi = (t.double().cpu().numpy() for t in bn.crown_bounds(x_lo, x_hi, slack=slack))
    for a, b in ((lo, dlo), (hi, dhi)):
        assert np.all(np.abs(a - b) <= 1e-4 * np.maximum(np.abs(b), 1.0)), "whole layers"
    for i in range(1):
        ob = O.crown_bounds(net, x_lo[i], x_hi[i], use_slack=slack)
        for got, side in ((lo[i], 0), (hi[i], 1)):
            want = np.concatenate([b[side] for b in ob])
            assert np.all(np.abs(got - want) <= 1e-4 * np.maximum(np.abs(want), 1.0)), f"oracle, input {i}"


def test_window_pass_keeps_the_best_bounds_and_one_side():
    """best / best_upper of a window pass, the row stride, and a pass for lower bounds only."""
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    net = _net("c8")
    n = 2
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, W.in_dim(net), 13), 0.02)
    bn = N.BoundNet(net, n, 4096)
    xl, xh = torch.as_tensor(x_lo, device="cuda"), torch.as_tensor(x_hi, device="cuda")
    lo, hi = bn.crown_bounds(xl, xh)
    for k in (1, 2):
        off, d = bn.relu_off[k - 1], bn.d[k]
        ref_lo, ref_hi = lo[:, off:off + d], hi[:, off:off + d]
        best, bup = ref_lo + 0.5, ref_hi + 0.5
        low = torch.empty(n, d + 3, device="cuda")
        up = torch.empty_like(low)
        bl, bu = torch.full_like(low, -1e9), torch.full_like(low, 1e9)
        bl[:, :d], bu[:, :d] = best, bup
        kw = dict(lo=lo, hi=hi, n_bounds=n, x_lo=xl, x_hi=xh, ld=d + 3)
        B.bound_backward(bn.handle, n, d, k, flags=B.BOUND_BOTH_SIDES, lower=low, upper=up, best=bl,
                         best_upper=bu, **kw)
        one = torch.empty_like(low)
        B.bound_backward(bn.handle, n, d, k, lower=one, **kw)
        # the same pass again: only the order of its atomic row sums differs
        tol = 1e-5 * ref_lo.abs().clamp_min(1.0)
        assert bool(((low[:, :d] - ref_lo).abs() <= tol).all()) and bool(((one[:, :d] - ref_lo).abs() <= tol).all())
        assert torch.equal(bl[:, :d], torch.maximum(best, low[:, :d]))
        assert torch.equal(bu[:, :d], torch.minimum(bup, up[:, :d]))
