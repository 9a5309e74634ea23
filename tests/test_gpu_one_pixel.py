"""Convolutions whose products have one source pixel and one tap on it: 1x1 layers on a 1x1
map (padded too) and stride-2 layers onto one pixel, whose input pixels are phases of their
own.  Full CROWN, spec bounds, coefficients, gradients and forward samples against the FP64
oracle, on automatic and implicit-GEMM plans.  Tolerance: 1e-4 relative, the parity tolerance
of every FP32 bound against FP64 (of the largest gradient for gradients).
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import crown as O

pytestmark = pytest.mark.gpu

#         input     (channels, kernel, stride, padding) ...                              FC widths
NETS = {
    "k2s2": ((3, 2, 2), [(5, 2, 2, 0)], (6, 4)),
    "k2s2_deep": ((3, 4, 4), [(8, 3, 1, 1), (12, 2, 2, 0), (20, 2, 2, 0), (17, 1, 1, 0)], (9, 4)),
    "k1s2": ((4, 2, 2), [(8, 3, 1, 1), (16, 1, 2, 0)], (8, 4)),
    "k3s2_pad": ((3, 2, 2), [(8, 3, 1, 1), (16, 3, 2, 1)], (8, 4)),
    "k1_pad": ((6, 1, 1), [(8, 1, 1, 0), (5, 1, 1, 1), (7, 3, 1, 1)], (8, 4)),
}


def _net(name):
    shape, convs, fc = NETS[name]
    rng = np.random.default_rng(191)
    layers = []
    for co, k, s, p in convs:
        layers.append(W._conv(rng, shape, co, k, s, p))
        shape = layers[-1]["out_shape"]
    d = int(np.prod(shape))
    for w in fc:
        layers.append(W._linear(rng, d, w))
        d = w
    return layers


def _close(a, b, what, scale=None):
    scale = np.maximum(np.abs(b), 1.0) if scale is None else scale
    assert np.all(np.abs(a - b) <= 1e-4 * scale), what


@pytest.mark.parametrize("path", ["auto", "gemm"])
@pytest.mark.parametrize("name", NETS)
def test_one_pixel_convolutions(name, path):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    net, n, R = _net(name), 5, 3
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, W.in_dim(net), 192), 0.2)
    C = np.random.default_rng(193).normal(0, 1, (n, R, 4)).astype(np.float32)
    bn = N.BoundNet(net, n, 64, n * R)
    if path == "gemm":
        B.bound_set_options(bn.handle, B.BOUND_OPT_GEMM_ONLY)
    lo, hi = bn.crown_bounds(x_lo, x_hi)
    alpha = W.random_alpha(n, bn.n_relu, 194)
    both = bn.spec_bounds(C, lo, hi, x_lo, x_hi)
    low, _ = bn.spec_bounds(C, lo, hi, x_lo, x_hi, alpha=torch.as_tensor(alpha, device="cuda"), both=False,
                            slack=False, save=True)
    ga, _ = bn.grad(torch.ones(n, R, device="cuda"))
    x = torch.as_tensor((x_lo + x_hi) / 2, device="cuda")
    out = torch.empty(n, 4, device="cuda")
    slo, shi = torch.empty(n, bn.n_relu, device="cuda"), torch.empty(n, bn.n_relu, device="cuda")
    B.bound_sample_bounds(bn.handle, n, 1, x, slo, shi, out)
    lo, hi, low, ga, out, slo = (t.double().cpu().numpy() for t in (lo, hi, low, ga, out, slo))
    L = len(net)
    for i in range(n):
        ob = O.crown_bounds(net, x_lo[i], x_hi[i])
        for got, side in ((lo, 0), (hi, 1)):
            _close(got[i], np.concatenate([b[side] for b in ob]), f"side {side}")
        want = O.spec_lower(net, L, C[i], ob, x_lo[i], x_hi[i])
        _close(both[0][i].double().cpu().numpy(), want, "spec lower")
        # the gradient's branches at the GPU's own intermediate bounds
        b = list(zip(O.per_layer(net, lo[i]), O.per_layer(net, hi[i])))
        al = O.per_layer(net, alpha[i])
        want, oga, _ = O.spec_lower_grad(net, L, C[i], b, x_lo[i], x_hi[i], al)
        _close(low[i], want, "raw lower")
        oga = np.concatenate(oga)
        _close(ga[i], oga, "gradient", max(np.abs(oga).max(), 1e-30))
        z = O.forward(net, x[i:i + 1].double().cpu().numpy())
        _close(slo[i], np.concatenate([v.reshape(-1) for v in z[:-1]]), "samples")
        _close(out[i], z[-1].reshape(-1), "outputs")


def test_dense_convolution_without_bf16_weights():
    """A 1x1 layer on one pixel from 256 tiles of 128 x 128 on, where Linear layers take the
    bf16 tile: automatic, pinned (the plan falls back) and tuned."""
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    rng = np.random.default_rng(195)
    net = [W._conv(rng, (24, 1, 1), 300, 1, 1, 0), W._conv(rng, (300, 1, 1), 300, 1, 1, 0),
           W._conv(rng, (300, 1, 1), 20, 1, 1, 0), W._linear(rng, 20, 4)]
    n, R = 3000, 4
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, 24, 196), 0.05)
    C = np.random.default_rng(197).normal(0, 1, (n, R, 4)).astype(np.float32)
    bn = N.BoundNet(net, n, n * 2 * R)          # 24000 rows x 300 columns: 564 tiles
    small = [N.BoundNet(net, 1, 2 * 300).crown_bounds(x_lo[i:i + 1], x_hi[i:i + 1]) for i in range(n)]
    lo, hi = (torch.cat([b[k] for b in small]) for k in (0, 1))
    del small
    rows = (0, 1, n - 1)
    want = {}
    for i in rows:
        b = list(zip(O.per_layer(net, lo[i].double().cpu().numpy()), O.per_layer(net, hi[i].double().cpu().numpy())))
        want[i] = O.spec_lower(net, 4, C[i], b, x_lo[i], x_hi[i])
    for plan in ("auto", "pinned", "tuned"):
        if plan == "pinned":
            for k in (1, 2, 3):
                for p in "RC":
                    B.bound_set_plan(bn.handle, p, k, 2, 16, 0)
        if plan == "tuned":
            low, up = torch.empty(n, R, device="cuda"), torch.empty(n, R, device="cuda")
            t = lambda a: torch.as_tensor(a, device="cuda")
            B.bound_autotune(bn.handle, n, R, 4, spec=t(C), lo=lo, hi=hi, n_bounds=n, x_lo=t(x_lo), x_hi=t(x_hi),
                             lower=low, upper=up, flags=B.BOUND_BOTH_SIDES)
        low, _ = bn.spec_bounds(C, lo, hi, x_lo, x_hi)
        for i in rows:
            _close(low[i].double().cpu().numpy(), want[i], f"{plan}, instance {i}")
