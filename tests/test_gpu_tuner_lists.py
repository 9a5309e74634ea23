"""What the autotuner times, from its report: products that keep the FP32 order (the adjoint,
and forward samples) have no bf16 weights and are not timed on that tile.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _handle(dims, n, R, save):
    from paper_2412_09584_amd import net as N
    net = W.mlp(list(dims), seed=231)
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, dims[0], 232), 0.05)
    C = np.random.default_rng(233).normal(0, 1, (n, R, dims[-1])).astype(np.float32)
    bn = N.BoundNet(net, n, max(n * 2 * R, 2048), n * R if save else 0)
    lo, hi = bn.crown_bounds(x_lo, x_hi)
    t = lambda a: torch.as_tensor(a, device="cuda")
    args = dict(spec=t(C), lo=lo, hi=hi, n_bounds=n, x_lo=t(x_lo), x_hi=t(x_hi),
                lower=torch.empty(n, R, device="cuda"))
    return bn, net, args, (x_lo, x_hi, C)


def _tuned(bn, n, R, L, args, save):
    """{product: [(path, cfg)]} of one tuning run."""
    from paper_2412_09584_amd import binding as B
    kw = dict(args, flags=B.BOUND_SAVE_FOR_GRAD, grad_lower=torch.ones(n, R, device="cuda")) if save else args
    out = {}
    for line in B.bound_autotune(bn.handle, n, R, L, **kw).strip().splitlines():
        key, path, cfg = line.split()[:3]
        out.setdefault(key, []).append((path, int(cfg.split("=")[1])))
    return out


def test_adjoint_is_not_timed_on_the_bf16_tile():
    n, R = 40, 3
    bn, net, args, _ = _handle((40, 90, 70, 6), n, R, True)
    lists = _tuned(bn, n, R, len(net), args, True)
    assert any(k[0] == "A" for k in lists)
    for key, plans in lists.items():
        if key[0] == "A":
            assert ("gemm", 16) not in plans, key


def test_tuned_passes_of_both_kinds():
    """A tuned saving pass times no plan on the bf16 matrix cores; a tuned pass that saves
    nothing does, and its bounds are those of the automatic plans (1e-5: other orders of the
    same FP32 sums)."""
    n, R = 3000, 6                                  # 18000 rows x 260: 423 tiles
    bn, net, args, (x_lo, x_hi, C) = _handle((40, 260, 256, 6), n, R, True)
    ref, _ = bn.spec_bounds(C, args["lo"], args["hi"], x_lo, x_hi, both=False)
    saving = _tuned(bn, n, R, len(net), args, True)
    assert all(("gemm", c) not in plans for plans in saving.values() for c in (13, 14, 16))
    other = _tuned(bn, n, R, len(net), args, False)
    assert ("gemm", 16) in other["R2"] and ("auto", -1) in other["R2"]
    low, _ = bn.spec_bounds(C, args["lo"], args["hi"], x_lo, x_hi, both=False)
    assert bool(((low - ref).abs() <= 1e-5 * ref.abs().clamp_min(1.0)).all())
