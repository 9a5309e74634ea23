"""Automatic staging of the direct convolutions: LDS DMA from as many blocks on as there are
compute units, registers below and where the tile does not fit.  Both add a row's terms in
the same order, so a saving pass and its gradient are bitwise those of plans that ask for
register staging (deterministic row sums: no order of atomics), at batches on both sides of
the rule and with a ragged last group of images.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin", [3, 4])
@pytest.mark.parametrize("n", [1, 67, 301])
def test_automatic_staging_keeps_the_bits(cin, n):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    net = W.cnn(seed=171, in_shape=(cin, 16, 16), spec=[(16, 3, 1), (32, 4, 2), (32, 3, 1), (64, 4, 2)], fc=(16, 5))
    x0 = W.uniform_inputs(1, W.in_dim(net), 172)
    x_lo, x_hi = (np.repeat(a, n, 0) for a in W.linf_box(x0, 0.03))
    C = np.repeat(W.margin_spec(W.clean_logits(net, x0)), n, 0)
    ref = N.BoundNet(net, 1, 4096)
    lo, hi = (t.repeat(n, 1).contiguous() for t in ref.crown_bounds(x_lo[:1], x_hi[:1]))
    alpha = torch.as_tensor(W.random_alpha(n, lo.shape[1], 173), dtype=torch.float32, device="cuda")
    out = []
    for explicit in (False, True):
        bn = N.BoundNet(net, n, n * C.shape[1], n * C.shape[1])
        B.bound_set_options(bn.handle, B.BOUND_OPT_DETERMINISTIC)
        for prod, layer in [("C", 1), ("A", 1)] + [(p, k) for p in "RA" for k in (2, 3, 4)] if explicit else []:
            if (prod, layer) != ("A", 2):        # 16 channels of 4 x 4 taps: the automatic plan is a GEMM
                B.bound_set_plan(bn.handle, prod, layer, 1, -1, 0)
        low, _ = bn.spec_bounds(C, lo, hi, x_lo, x_hi, alpha=alpha, both=False, save=True)
        ga, _ = bn.grad(torch.ones(n, C.shape[1], device="cuda"), 0)
        out.append((low.clone(), ga.clone()))
    assert torch.equal(out[0][0], out[1][0]), "bounds"
    assert torch.equal(out[0][1], out[1][1]), "gradient"
