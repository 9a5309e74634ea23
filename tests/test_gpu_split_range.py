"""Operands that three bf16 parts do not hold: infinities, FP32 values past the largest bf16, and
rows so small that their last parts would be flushed.  The bf16 kernels form such tiles by FP32
instructions, and layers of such weights take the FP32 kernels: coefficients (no box) as on the
general kernels (BOUND_OPT_GEMM_ONLY), infinities and NaN at the same places, everything
else within 2e-6 of the row's largest (two FP32 sums of up to 1152 terms).
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _coeffs(net, target, C, lo, hi, options):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    n, R, _ = C.shape
    d0 = W.in_dim(net)
    t = lambda a: torch.as_tensor(a, device="cuda")
    bn = N.BoundNet(net, n, n * R)
    B.bound_set_options(bn.handle, options)
    co = torch.empty(n * R, d0, device="cuda")
    off, mag = torch.empty(n * R, device="cuda"), torch.empty(n * R, device="cuda")
    kw = {} if lo is None else dict(lo=t(lo), hi=t(hi), n_bounds=n)
    B.bound_backward(bn.handle, n, R, target, spec=t(C), coeff=co, offset=off, offset_mag=mag, **kw)
    return co.double().cpu().numpy()


def _same(a, b, what):
    for f in (np.isnan, np.isposinf, np.isneginf):
        assert np.array_equal(f(a), f(b)), f"{what}: {f.__name__} at other places"
    fin = np.isfinite(b)
    scale = np.where(fin, np.abs(b), 0).max(1, keepdims=True)
    off = np.where(fin, np.abs(np.where(fin, a, 0) - np.where(fin, b, 0)), 0)
    assert np.all(off <= 2e-6 * scale), f"{what}: {np.max(off / np.maximum(scale, 1e-300)):.2g} of the row's largest"


def _spec(shape, seed):
    """Normal rows, among them rows with +-inf, with a value past the largest bf16, tiny ones
    and one of a single tiny value."""
    C = np.random.default_rng(seed).normal(0, 1, shape).astype(np.float32)
    C[1, 0, 3] = np.inf
    C[2, 1, 0] = -np.inf
    C[3, 2, 5] = 3.4e38
    C[4] *= np.float32(2.0 ** -112)
    C[5, 3] *= np.float32(2.0 ** -120)
    C[6, 0] = 0
    C[6, 0, 2] = 1.5e-36
    return C


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -112, 3.0e37])
def test_dense_rows_and_weights(scale):
    """16384 rows (256 tiles), one layer (the concretising product) and two (the relaxing one,
    every neuron active); weights scaled out of the range too."""
    from paper_2412_09584_amd import binding as B
    net = W.mlp([270, 256], seed=261)
    net[0]["W"] = (net[0]["W"] * scale * (10 if scale > 1 else 1)).astype(np.float32)
    C = _spec((256, 64, 256), 262)
    if scale != 1.0:          # one thing at a time
        C = np.random.default_rng(263).normal(0, 1, C.shape).astype(np.float32)
    if scale > 1.0:
        C *= np.float32(1e-6)
    a, b = (_coeffs(net, 1, C, None, None, o) for o in (0, B.BOUND_OPT_GEMM_ONLY))
    _same(a, b, "one layer")
    if scale == 1.0:
        net = W.mlp([256, 300, 256], seed=264)
        lo = np.random.default_rng(265).uniform(0.1, 1, (256, 300)).astype(np.float32)
        C[1:4] = np.random.default_rng(266).normal(0, 1, C[1:4].shape)
        a, b = (_coeffs(net, 2, C, lo, lo + 1, o) for o in (0, B.BOUND_OPT_GEMM_ONLY))
        _same(a, b, "two layers")


@pytest.mark.parametrize("side", [8, 16, 32])
def test_convolution_rows(side):
    """Relaxing 3x3 products of 32 channels on whole layers: several images a block (8 x 8), one
    (16 x 16) and bands of one (32 x 32)."""
    from paper_2412_09584_amd import binding as B
    rng = np.random.default_rng(267)
    net = [W._conv(rng, (4, side, side), 32, 3, 1, 1), W._conv(rng, (32, side, side), 32, 3, 1, 1)]
    d, n, R = 32 * side * side, 7, 4
    C = _spec((n, R, d), 268)
    C[3, 2, 5] = 0
    lo = rng.uniform(0.1, 1, (n, d)).astype(np.float32)
    a, b = (_coeffs(net, 2, C, lo, lo + 1, o) for o in (0, B.BOUND_OPT_GEMM_ONLY))
    _same(a, b, "convolution")


def test_window_rows_and_weights():
    """Full CROWN (windows, pairs of phases): a layer scaled down by 2^112 and the next one up
    again gives the first network's bounds."""
    from paper_2412_09584_amd import net as N
    rng = np.random.default_rng(269)
    net = [W._conv(rng, (3, 16, 16), 16, 3, 1, 1), W._conv(rng, (16, 16, 16), 32, 4, 2, 1),
           W._conv(rng, (32, 8, 8), 32, 3, 1, 1), W._conv(rng, (32, 8, 8), 32, 3, 1, 1), W._linear(rng, 2048, 4)]
    x_lo, x_hi = W.linf_box(W.uniform_inputs(2, 768, 270), 0.02)
    s = np.float32(2.0 ** -112)
    tiny = [dict(l) for l in net]
    tiny[2] = dict(net[2], W=net[2]["W"] * s, b=net[2]["b"] * s)
    tiny[3] = dict(net[3], W=net[3]["W"] / s)
    out = [N.BoundNet(l, 2, 4096).crown_bounds(x_lo, x_hi) for l in (net, tiny)]
    a0, a1 = 16 * 256 + 32 * 64, 16 * 256 + 32 * 64 + 32 * 64        # z_3, scaled
    for p, q in zip(*out):
        q = q.clone()
        q[:, a0:a1] /= float(s)
        assert bool(((p - q).abs() <= 1e-5 * p.abs().clamp_min(1.0)).all())
