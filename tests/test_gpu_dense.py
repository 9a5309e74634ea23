"""The dense products' kernels (bound_set_plan tile configurations past the LDS-tiled GEMM's)
against those of BOUND_OPT_GEMM_ONLY and the FP64 oracle, at the sizes where they can go
wrong: one row, rows and columns around the 16 / 32 / 128 tiles, widths that are no multiple
of 4 (unaligned rows) or of the k chunks, and K below one chunk.  Bounds, gradients and
forward samples; the parity tolerance 1e-4 (of the largest gradient for gradients).
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import crown as O

pytestmark = pytest.mark.gpu

WIDTHS = [(5, 7, 3), (33, 31, 130, 17, 4), (64, 129, 16, 65, 10), (30, 300, 258, 2)]
CFGS = [11, 12, 13, 14, 15, 16, 17]


def _case(dims, n):
    net = W.mlp(list(dims), seed=21)
    x0 = W.uniform_inputs(n, dims[0], 22)
    x_lo, x_hi = W.linf_box(x0, 0.05)
    rng = np.random.default_rng(23)
    R = 3
    C = rng.normal(0, 1, (n, R, dims[-1])).astype(np.float32)
    return net, x_lo, x_hi, C


def _run(net, x_lo, x_hi, C, lo, hi, alpha, plan):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    n, R = C.shape[:2]
    bn = N.BoundNet(net, n, 4096, n * R)
    if plan is None:
        B.bound_set_options(bn.handle, B.BOUND_OPT_GEMM_ONLY)
    elif plan >= 0:
        for k in range(1, len(net) + 1):
            for p in "RCAF":
                B.bound_set_plan(bn.handle, p, k, 2, plan, 0)
    t = lambda a: torch.as_tensor(a, device="cuda")
    low, _ = bn.spec_bounds(C, t(lo), t(hi), x_lo, x_hi, alpha=t(alpha), both=False, save=True)
    ga, _ = bn.grad(torch.ones(n, R, device="cuda"))
    both = bn.spec_bounds(C, t(lo), t(hi), x_lo, x_hi)
    x = t((x_lo + x_hi) / 2)
    out = torch.empty(n, net[-1]["out_shape"][0], device="cuda")
    slo, shi = torch.empty(n, bn.n_relu, device="cuda"), torch.empty(n, bn.n_relu, device="cuda")
    B.bound_sample_bounds(bn.handle, n, 1, x, slo, shi, out)
    clo, chi = bn.crown_bounds(x_lo, x_hi)
    return [v.double().cpu().numpy() for v in (low, ga, *both, slo, out, clo, chi)]


@pytest.mark.parametrize("n", [1, 11, 43])
@pytest.mark.parametrize("dims", WIDTHS)
def test_dense_kernels_match_general_gemm_and_oracle(dims, n):
    net, x_lo, x_hi, C = _case(dims, n)
    bounds = [O.crown_bounds(net, x_lo[i], x_hi[i]) for i in range(n)]
    lo = np.stack([np.concatenate([b[0] for b in o]) for o in bounds]).astype(np.float32)
    hi = np.stack([np.concatenate([b[1] for b in o]) for o in bounds]).astype(np.float32)
    alpha = W.random_alpha(n, lo.shape[1], 24)
    ref = _run(net, x_lo, x_hi, C, lo, hi, alpha, None)
    for plan in [-1] + CFGS:
        got = _run(net, x_lo, x_hi, C, lo, hi, alpha, plan)
        for k, (a, b) in enumerate(zip(got, ref)):
            scale = np.abs(b).max() if k == 1 else np.maximum(np.abs(b), 1.0)
            assert np.all(np.abs(a - b) <= 1e-4 * scale), f"cfg {plan}, output {k}"
    i = n - 1
    b64 = [(O.per_layer(net, lo[i].astype(float)), O.per_layer(net, hi[i].astype(float)))]
    b64 = list(zip(*b64[0]))
    al = O.per_layer(net, alpha[i])
    want = O.spec_lower(net, len(net), C[i], b64, x_lo[i], x_hi[i], al)
    _, oga, _ = O.spec_lower_grad(net, len(net), C[i], b64, x_lo[i], x_hi[i], al)
    oga = np.concatenate(oga)
    assert np.all(np.abs(ref[0][i] - want) <= 1e-4 * np.maximum(np.abs(want), 1.0))
    assert np.abs(ref[1][i] - oga).max() <= 1e-4 * max(np.abs(oga).max(), 1e-30)


@pytest.mark.parametrize("n", [1, 50, 700, 9000])
def test_saving_pass_keeps_its_coefficients(n):
    """Automatic plans of a SAVE_FOR_GRAD pass give the general GEMM's coefficients bitwise, so
    the gradient takes the same branch at every neuron, and the adjoint's automatic plans
    add in the general GEMM's order: gradients are equal bitwise."""
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    dims, R = (40, 100, 530, 70, 17, 36, 6), 3
    net, x_lo, x_hi, C = _case(dims, n)
    bn = N.BoundNet(net, n, max(4096, n * R), n * R)
    lo, hi = bn.crown_bounds(x_lo, x_hi)
    alpha = torch.as_tensor(W.random_alpha(n, bn.n_relu, 25), device="cuda")
    out = []
    for pinned in (False, True):
        for k in range(1, len(net) + 1):
            for p in "RCA":
                B.bound_set_plan(bn.handle, p, k, 2 if pinned else 0, -1, 0)
        bn.spec_bounds(C, lo, hi, x_lo, x_hi, alpha=alpha, both=False, save=True)
        out.append(bn.grad(torch.ones(n, R, device="cuda"))[0])
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("n,dims,rows", [(1, (5, 7, 3, 2), 64), (3, (70, 130, 261, 9, 4), 300), (40, (16, 64, 33, 65, 3), 1500)])
def test_identity_rows_of_linear_targets(n, dims, rows):
    """Full CROWN's identity rows and box bounds of Linear layers: rows and columns around the
    waves' eight rows and 64 columns, instances cut by the workspace's chunks, both the
    row-per-block and the eight-rows-per-wave kernels, against the FP64 oracle (1e-4)."""
    from paper_2412_09584_amd import net as N
    net, x_lo, x_hi, _ = _case(dims, n)
    bn = N.BoundNet(net, n, rows)
    lo, hi = (t.double().cpu().numpy() for t in bn.crown_bounds(x_lo, x_hi))
    one = N.BoundNet(net, n, 1 << 16)
    olo, ohi = (t.double().cpu().numpy() for t in one.crown_bounds(x_lo, x_hi))
    for i in range(0, n, 13):
        ob = O.crown_bounds(net, x_lo[i], x_hi[i])
        for side, got in ((0, (lo, olo)), (1, (hi, ohi))):
            want = np.concatenate([b[side] for b in ob])
            for g in got:
                assert np.all(np.abs(g[i] - want) <= 1e-4 * np.maximum(np.abs(want), 1.0))
