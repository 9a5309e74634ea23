"""Window passes in the configurations that only large ones reach: blocks that take several
groups of images in turn (from 8192 tiles on), with a last block and a last group that are
not full, pairs of phases and whole fragments, and windows of 16 pixels a side; every
neuron of every input against the whole-layer kernels (BOUND_OPT_GEMM_ONLY) at the same
bounds of the layers below.  Tolerance: 5e-6 of max(|bound|, 1): both add some thousand
terms in FP32 (root mean square error about 2e-7).  test_host_rules.py looks at the
launches of these very passes.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

#         input        (channels, kernel, stride, padding) ...                  inputs  rows   targets
NETS = {
    "pairs": ((3, 32, 32), [(16, 3, 1, 1), (32, 4, 2, 1), (32, 3, 1, 1), (64, 4, 2, 1)], 5, 81901, (3, 4)),
    "wide_windows": ((3, 20, 20), [(32, 3, 1, 1)] * 5, 1, 25600, (5,)),
}


@pytest.mark.parametrize("name", NETS)
def test_large_window_passes(name):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    shape, convs, n, rows, targets = NETS[name]
    rng = np.random.default_rng(281)
    net = []
    for co, k, s, p in convs:
        net.append(W._conv(rng, shape, co, k, s, p))
        shape = net[-1]["out_shape"]
    net.append(W._linear(rng, int(np.prod(shape)), 2))
    x_lo, x_hi = (torch.as_tensor(a, device="cuda") for a in W.linf_box(W.uniform_inputs(n, W.in_dim(net), 282), 0.01))
    bn = N.BoundNet(net, n, rows)
    z = torch.as_tensor(rng.normal(0, 1, (n, bn.n_relu)).astype(np.float32), device="cuda")
    w = torch.as_tensor(rng.uniform(0, 1, (n, bn.n_relu)).astype(np.float32), device="cuda")
    lo, hi = z - w, z + w
    for k in targets:
        d = bn.d[k]
        out = []
        for options in (0, B.BOUND_OPT_GEMM_ONLY):
            B.bound_set_options(bn.handle, options)
            low, up = torch.empty(n, d, device="cuda"), torch.empty(n, d, device="cuda")
            B.bound_backward(bn.handle, n, d, k, lo=lo, hi=hi, n_bounds=n, x_lo=x_lo, x_hi=x_hi,
                             flags=B.BOUND_BOTH_SIDES, lower=low, upper=up)
            out.append((low, up))
        for a, b in zip(*out):
            assert bool(((a - b).abs() <= 5e-6 * b.abs().clamp_min(1.0)).all()), f"target {k}"


def test_debug_check_names_the_window_product():
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    rng = np.random.default_rng(283)
    net = [W._conv(rng, (3, 16, 16), 16, 3, 1, 1), W._conv(rng, (16, 16, 16), 16, 3, 1, 1), W._linear(rng, 4096, 2)]
    x_lo, x_hi = W.linf_box(W.uniform_inputs(1, 768, 284), 0.01)
    bn = N.BoundNet(net, 1, 8192)
    B.bound_set_options(bn.handle, B.BOUND_OPT_CHECK)
    bn.crown_bounds(x_lo, x_hi)
    x_lo[0, 5] = np.nan
    with pytest.raises(B.BoundError) as e:
        bn.crown_bounds(x_lo, x_hi)
    assert e.value.status == B.BOUND_E_NUMERIC and "L2" in str(e.value)   # z_1's NaN bounds reach its records
