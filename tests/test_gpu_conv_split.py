"""Relaxing convolutions on the bf16 matrix cores (full CROWN's passes save nothing).

Window passes and whole layers at sizes where the kernel's tiles can go wrong: windows of
4, 8 and 16 pixels a side and phase, pairs of phases with 8, 12 and 16 channels, 20 to 96
columns, one to six channel chunks, last groups of images that are not full, several
groups a block, and bands of a large layer.  Against the FP64 oracle and against the
general kernels (BOUND_OPT_GEMM_ONLY).  Tolerance: 1e-4 relative, the parity tolerance of
every FP32 bound against FP64; the error against FP64 must also stay within twice that of
the general kernels' bounds (both add as many FP32 terms) plus 1e-6 of the largest bound.
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import crown as O

pytestmark = pytest.mark.gpu

#          input       (channels, kernel, stride, padding) ...                        FC widths
NETS = {
    "pair16": ((3, 16, 16), [(16, 3, 1, 1), (32, 4, 2, 1), (32, 3, 1, 1), (48, 4, 2, 1)], (12, 4)),
    "pair12": ((3, 12, 12), [(12, 3, 1, 1), (16, 4, 2, 1), (20, 3, 1, 1), (32, 4, 2, 1)], (4,)),
    "pair8_pad0": ((3, 18, 18), [(8, 3, 1, 1), (32, 4, 2, 0), (64, 3, 1, 1)], (4,)),
    "wide": ((3, 8, 8), [(96, 3, 1, 1), (96, 3, 1, 1), (32, 3, 1, 1)], (4,)),
    "k2_stride2": ((3, 16, 16), [(16, 3, 1, 1), (16, 2, 2, 0), (32, 3, 1, 1)], (4,)),
}


def _net(name):
    shape, convs, fc = NETS[name]
    rng = np.random.default_rng(181)
    layers = []
    for co, k, s, p in convs:
        layers.append(W._conv(rng, shape, co, k, s, p))
        shape = layers[-1]["out_shape"]
    d = int(np.prod(shape))
    for w in fc:
        layers.append(W._linear(rng, d, w))
        d = w
    return layers


@pytest.mark.parametrize("name,n,rows", [("pair16", 3, 5003), ("pair16", 1, 20000), ("pair12", 3, 4999),
                                         ("pair8_pad0", 3, 5000), ("wide", 2, 6001), ("k2_stride2", 3, 4097)])
def test_split_convolutions(name, n, rows):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    net = _net(name)
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, W.in_dim(net), 182), 0.02)
    bn = N.BoundNet(net, n, rows)
    got = [t.double().cpu().numpy() for t in bn.crown_bounds(x_lo, x_hi)]
    B.bound_set_options(bn.handle, B.BOUND_OPT_GEMM_ONLY)
    gen = [t.double().cpu().numpy() for t in bn.crown_bounds(x_lo, x_hi)]
    for a, b in zip(got, gen):
        assert np.all(np.abs(a - b) <= 1e-4 * np.maximum(np.abs(b), 1.0)), "general kernels"
    ob = O.crown_bounds(net, x_lo[0], x_hi[0], use_slack=True)
    for k in range(2):
        ref = np.concatenate([b[k] for b in ob])
        assert np.all(np.abs(got[k][0] - ref) <= 1e-4 * np.maximum(np.abs(ref), 1.0)), "oracle"
        e_got, e_gen = (np.sqrt(np.mean((x[k][0] - ref) ** 2)) for x in (got, gen))
        assert e_got <= 2 * e_gen + 1e-6 * np.max(np.abs(ref)), (e_got, e_gen)
