"""Saving passes where the preparation's kernels leave their first round: layers of more
neurons than one sweep of the slot kernel holds (65536; up to three sweeps, and a
convolution whose sweeps end inside a pixel), and split lists longer than a wave (65 to 200
entries with repeated neurons in both signs).  Bounds and gradients against the FP64
oracle at the same bounds; 1e-4 (of the largest gradient for gradients).
"""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import crown as O

pytestmark = pytest.mark.gpu


def _check(net, n, R, seed, entries=None):
    from paper_2412_09584_amd import net as N
    rng = np.random.default_rng(seed)
    x_lo, x_hi = W.linf_box(W.uniform_inputs(n, W.in_dim(net), seed + 1), 0.05)
    C = rng.normal(0, 1, (n, R, net[-1]["out_shape"][0])).astype(np.float32)
    nr = sum(int(np.prod(l["out_shape"])) for l in net[:-1])
    z = rng.normal(0, 1, (n, nr))
    w = rng.uniform(0, 1, z.shape)
    lo, hi = (z - w).astype(np.float32), (z + w).astype(np.float32)
    alpha = W.random_alpha(n, nr, seed + 2)
    t = lambda a: torch.as_tensor(a, device="cuda")
    sp, beta, kw, nnz = None, None, {}, 0
    if entries:
        off, neu, sg = [0], [], []
        for i in range(n):
            un = np.nonzero((lo[i] < 0) & (hi[i] > 0))[0]
            neu += list(rng.choice(un[:entries // 2], entries))       # most neurons several times
            sg += list(rng.choice([-1, 1], entries))
            off.append(len(neu))
        sp = W.Splits(np.array(off, np.int32), np.array(neu, np.int32), np.array(sg, np.int8))
        nnz = sp.nnz
        beta = W.random_beta(nnz, R, seed + 3)
        kw = dict(splits=N.splits_to_device(sp), beta=t(beta))
    bn = N.BoundNet(net, n, n * R, n * R)
    low, _ = bn.spec_bounds(C, t(lo), t(hi), x_lo, x_hi, alpha=t(alpha), both=False, slack=False, save=True, **kw)
    ga, gb = bn.grad(torch.ones(n, R, device="cuda"), nnz)
    for i in range(n):
        b = list(zip(O.per_layer(net, lo[i]), O.per_layer(net, hi[i])))
        q = slice(sp.off[i], sp.off[i + 1]) if sp else slice(0, 0)
        args = (O.split_list(net, sp.neuron[q], sp.sign[q]), beta[q].astype(float)) if sp else ()
        want, oga, ogb = O.spec_lower_grad(net, len(net), C[i], b, x_lo[i], x_hi[i], O.per_layer(net, alpha[i]), *args)
        got = low[i].double().cpu().numpy()
        assert np.all(np.abs(got - want) <= 1e-4 * np.maximum(np.abs(want), 1.0)), f"bound {i}"
        oga = np.concatenate(oga)
        assert np.abs(ga[i].double().cpu().numpy() - oga).max() <= 1e-4 * np.abs(oga).max(), f"alpha {i}"
        if sp:
            assert np.abs(gb[q].double().cpu().numpy() - ogb).max() <= 1e-4 * np.abs(ogb).max(), f"beta {i}"


@pytest.mark.parametrize("width", [65537, 140003])
def test_wide_linear_layer(width):
    rng = np.random.default_rng(251)
    _check([W._linear(rng, 3, width), W._linear(rng, width, 4)], 2, 2, 252)


@pytest.mark.parametrize("channels,side", [(24, 60), (7, 150)])
def test_wide_convolution(channels, side):
    rng = np.random.default_rng(253)
    net = [W._conv(rng, (2, side, side), channels, 3, 1, 1), W._linear(rng, channels * side * side, 3)]
    _check(net, 2, 2, 254)


@pytest.mark.parametrize("entries", [65, 128, 200])
def test_long_split_lists(entries):
    _check(W.mlp([20, 90, 70, 80, 5], seed=255), 3, 2, 256, entries)
