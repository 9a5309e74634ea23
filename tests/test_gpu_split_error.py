"""The dense tile on the bf16 matrix cores gives coefficients at least as near to FP64 as the
FP32 kernels: root mean square error of the coefficient form (no box, so no row sums take
part) over all rows, against the same pass on the general GEMM.  The bound is the FP32
kernels' own error.  16384 rows, so that every product takes the bf16 tile; K of full and of
ragged chunks, 256 and 300 columns.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _exact(net, C, lo, hi):
    """Coefficients on the input in float64, default slopes."""
    Ws = [torch.as_tensor(l["W"], device="cuda").double() for l in net]
    g = C.double().reshape(-1, C.shape[2])
    off = np.concatenate([[0], np.cumsum([w.shape[0] for w in Ws[:-1]])]).astype(int)
    for m in range(len(net) - 1, 0, -1):
        g = g @ Ws[m]
        s = slice(off[m - 1], off[m])
        l, u = (t[:, s].double().repeat_interleave(C.shape[1], 0) for t in (lo, hi))
        un = (l < 0) & (u > 0)
        low = torch.where(un, (u >= -l).double(), (l >= 0).double())
        up = torch.where(un, u / (u - l).clamp(min=1e-300), (l >= 0).double())
        g = torch.where(g >= 0, g * low, g * up)
    return g @ Ws[0]


@pytest.mark.parametrize("width", [256, 260])
def test_coefficients_are_as_near_to_fp64_as_the_fp32_kernels(width):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    net = W.mlp([300, width, width, width, width, 10], seed=221)
    n, R = 256, 64
    rng = np.random.default_rng(222)
    t = lambda a: torch.as_tensor(a.astype(np.float32), device="cuda")
    C = t(rng.normal(0, 1, (n, R, 10)))
    z = rng.normal(0, 1, (n, 4 * width))
    w = rng.uniform(0, 1, z.shape)
    lo, hi = t(z - w), t(z + w)
    want = _exact(net, C, lo, hi)
    err = []
    for options in (0, B.BOUND_OPT_GEMM_ONLY):
        bn = N.BoundNet(net, n, n * R)
        B.bound_set_options(bn.handle, options)
        co = torch.empty(n * R, 300, device="cuda")
        off, mag = torch.empty(n * R, device="cuda"), torch.empty(n * R, device="cuda")
        B.bound_backward(bn.handle, n, R, len(net), spec=C, lo=lo, hi=hi, n_bounds=n, coeff=co, offset=off,
                         offset_mag=mag)
        err.append(((co.double() - want).pow(2).mean() / want.pow(2).mean()).sqrt().item())
    print(err)
    assert err[0] <= err[1]
