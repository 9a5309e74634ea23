"""Pick-out and pruner of one block (up to 65536 subdomains, 4096 picks of either phase)
against the oracle, which gives the lists exactly: set sizes around the block's rounds and
its range's end, picks around the selection's ends, ties, non-finite bounds, and eta at both
ends; one size past each limit takes the device-wide sort.
"""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

from oracle import bab as OB  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n", [(1, 1), (7, 9), (1023, 64), (1024, 1), (1025, 600), (5000, 4999), (9000, 8192),
                                 (65535, 1024), (65536, 4097), (65537, 300)])
@pytest.mark.parametrize("eta", [0.0, 0.5, 1.0])
def test_pick_out_and_prune(N, n, eta):
    from paper_2412_09584_amd import binding as B
    rng = np.random.default_rng(N + n)
    f_lo = np.round(rng.normal(size=N), 2).astype(np.float32)          # many ties
    f_hi = np.round(rng.normal(size=N), 1).astype(np.float32)
    g = np.round(-np.log(-np.log(rng.random(N))), 1).astype(np.float32)
    f_lo[rng.random(N) < 0.05] = np.inf
    f_lo[rng.random(N) < 0.02] = np.nan
    f_hi[rng.random(N) < 0.02] = np.nan
    f_hi[rng.random(N) < 0.02] = -0.0
    f_hi[rng.random(N) < 0.02] = -np.inf

    def t(a):
        return torch.as_tensor(a, device="cuda")

    h = B.bound_bab_init(N, 2, 8)
    m = min(n, N)
    picked = torch.full((m,), -1, dtype=torch.int32, device="cuda")
    rest = torch.full((max(N - m, 1),), -1, dtype=torch.int32, device="cuda")
    B.bound_bab_pick_out(h, N, t(f_lo), t(f_hi), t(g), n, eta, 0.05, picked, rest)
    want, others = OB.pick_out(f_lo, f_hi, g, n, eta, 0.05)
    assert picked.cpu().tolist() == [int(i) for i in want]
    assert rest.cpu().tolist()[:N - m] == [int(i) for i in others]
    for best in (0.25, -9.0, np.inf):
        keep = torch.full((N,), -1, dtype=torch.int32, device="cuda")
        nk = torch.zeros(1, dtype=torch.int32, device="cuda")
        B.bound_bab_prune(h, N, t(f_lo), t(np.array([best], np.float32)), keep, nk)
        ref = [int(i) for i in OB.prune(np.where(np.isnan(f_lo), np.inf, f_lo), best)]   # NaN: no bound, +inf
        assert int(nk.item()) == len(ref) and keep.cpu().tolist()[:len(ref)] == ref
    B.bound_bab_destroy(h)
