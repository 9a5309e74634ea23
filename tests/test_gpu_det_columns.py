"""Deterministic row sums on column counts that leave a wave of the last tile without columns
(65 .. 96 of 128 with 64-column tiles and so on): such a wave has no slot, and may not store
its zeros in those of the next pixel or image.  Linear layers on every implicit-GEMM tile, and
a 96-channel convolution on its automatic one, with as many rows as the workspace holds;
against the same passes with atomic sums.  Tolerance: 1e-5 relative, as for any two orders
of one FP32 sum here.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _run(net, n, R, cfgs):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, W.in_dim(net), 212), 0.05)
    C = np.random.default_rng(213).normal(0, 1, (n, R, net[-1]["out_shape"][0])).astype(np.float32)
    bn = N.BoundNet(net, n, n * 2 * R)
    lo, hi = bn.crown_bounds(x_lo, x_hi)
    for cfg in cfgs:
        if cfg is not None:
            for k in range(1, len(net) + 1):
                for p in "RC":
                    B.bound_set_plan(bn.handle, p, k, 2, cfg, 0)
        out = []
        for options in (0, B.BOUND_OPT_DETERMINISTIC):
            B.bound_set_options(bn.handle, options)
            out.append([t.double().cpu().numpy() for t in bn.spec_bounds(C, lo, hi, x_lo, x_hi)])
        for a, b in zip(*out):
            assert np.all(np.abs(a - b) <= 1e-5 * np.maximum(np.abs(a), 1.0)), f"plan {cfg}"


@pytest.mark.parametrize("n,R", [(1, 3), (50, 4)])
@pytest.mark.parametrize("dims", [(8, 80, 300, 5), (784, 150, 65, 7), (96, 33, 7)])
def test_linear_layers(dims, n, R):
    _run(W.mlp(list(dims), seed=211), n, R, [None] + list(range(11)))


def test_convolution_of_96_channels():
    rng = np.random.default_rng(214)
    net = [W._conv(rng, (4, 6, 6), 96, 3, 1, 1), W._conv(rng, (96, 6, 6), 12, 3, 2, 1), W._linear(rng, 108, 5)]
    _run(net, 7, 3, [None, -1, 0, 1])
