"""Row sums of a pass (bias, intercept and concretised terms) keep terms far below the running
sum: every kernel adds partial sums of its tiles, and these additions may not round at the
size of the sum.  A network of one always-active hidden layer whose output bias of 2^20 is
cancelled by the input box leaves the sum of the hidden biases' terms, which are 2^-20 of
it.  Tolerance: 2^-20 of the terms' summed magnitude, 16 roundings of the FP32 partial sums (an
FP32 running sum is off by an eighth per addition).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BIG = float(2 ** 20)


def _linear(Wm, b):
    return {"kind": "linear", "W": Wm.astype(np.float32), "b": np.asarray(b, np.float32),
            "in_shape": (Wm.shape[1],), "out_shape": (Wm.shape[0],)}


@pytest.mark.parametrize("options", [0, 8])       # 8: deterministic sums
@pytest.mark.parametrize("n,width", [(1, 300), (40, 257), (12000, 300)])
def test_small_terms_survive_the_running_sum(n, width, options):
    from paper_2412_09584_amd import binding as B
    from paper_2412_09584_amd import net as N
    rng = np.random.default_rng(201)
    R = 3
    W1 = np.zeros((width, 8))
    W1[0, 0] = 1.0
    b1 = rng.uniform(0.5, 1.5, width)
    b1[0] = 0.0
    W2 = rng.normal(0, 1, (R, width))
    W2[:, 0] = -1.0
    net = [_linear(W1, b1), _linear(W2, np.full(R, BIG))]
    x = np.zeros((n, 8), np.float32)
    x[:, 0] = BIG
    z = np.tile(np.concatenate([[BIG], b1[1:]]).astype(np.float32), (n, 1))
    C = np.tile(np.eye(R, dtype=np.float32), (n, 1, 1))
    w2, bb = net[1]["W"].astype(float)[:, 1:], net[0]["b"].astype(float)[1:]
    want, tol = w2 @ bb, 2.0 ** -20 * (np.abs(w2) @ np.abs(bb))
    bn = N.BoundNet(net, n, n * 2 * R)
    B.bound_set_options(bn.handle, options)
    t = lambda a: torch.as_tensor(a, device="cuda")
    for cfg in [None, -1, 3, 10] + list(range(11, 18)):
        if cfg is not None:
            for p, k in (("R", 2), ("C", 1)):
                B.bound_set_plan(bn.handle, p, k, 2, cfg, 0)
        low, up = bn.spec_bounds(C, t(z), t(z), x, x, slack=False)
        for got in (low, up):
            off = np.abs(got.double().cpu().numpy() - want) / tol
            assert off.max() <= 1.0, f"plan {cfg}: {off.max():.3g} of the tolerance"
