"""Full CROWN's first pass on more values than one launch takes threads for: instances on both
sides of the parts it runs in, against float64.  Tolerance: 1e-5 of the summed magnitudes'
scale (a few roundings of sums of 4 and 9 terms)."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["linear", "conv"])
def test_first_pass_in_several_launches(kind):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    rng = np.random.default_rng(241)
    if kind == "linear":          # 64 threads for 8 neurons: 32768 instances a launch
        net, n = [W._linear(rng, 4, 8192)], 65537
    else:                         # a thread a neuron: 131072 instances a launch
        net, n = [W._conv(rng, (1, 32, 32), 16, 3, 1, 1)], 131075
    d0, d = W.in_dim(net), int(np.prod(net[0]["out_shape"]))
    g = torch.Generator("cuda").manual_seed(242)
    x = torch.rand(n, d0, device="cuda", generator=g)
    lo, hi = torch.full((n, d), 7.0, device="cuda"), torch.full((n, d), 7.0, device="cuda")
    bn = N.BoundNet(net, n, 1024)
    B.bound_backward(bn.handle, n, d, 1, x_lo=x - 0.25, x_hi=x + 0.25, flags=B.BOUND_BOTH_SIDES | B.BOUND_NO_SLACK,
                     lower=lo, upper=hi)
    pick = torch.tensor([0, 1, 32767, 32768, 32769, 65535, 65536, n - 4, n - 3, n - 2, n - 1], device="cuda")
    xs = x[pick].double()
    w, b = torch.as_tensor(net[0]["W"], device="cuda").double(), torch.as_tensor(net[0]["b"], device="cuda").double()
    if kind == "linear":
        mid, rad = xs @ w.T + b, 0.25 * w.abs().sum(1)
    else:
        im, one = xs.reshape(-1, 1, 32, 32), torch.ones(1, 1, 32, 32, device="cuda", dtype=torch.float64)
        f = lambda v, k: torch.nn.functional.conv2d(v, k, padding=1).flatten(1)
        mid, rad = f(im, w) + b.repeat_interleave(1024), 0.25 * f(one, w.abs())
    assert bool(((lo[pick].double() - (mid - rad)).abs() <= 1e-5 * (1 + rad)).all())
    assert bool(((hi[pick].double() - (mid + rad)).abs() <= 1e-5 * (1 + rad)).all())
    assert int((lo == 7.0).sum()) < 10 and int((hi == 7.0).sum()) < 10     # all of them are written
