"""FP64 value of blocks above the register capacity, by panels of four tile
columns: joint sizes around the edges of a tile and of a panel (a border row
that opens a tile of its own, one to four tile columns in the last panel, an odd
number of row tiles below a panel), against the numpy oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import loglik as OL

pytestmark = pytest.mark.gpu
# (block points, neighbours): joint sizes 176, 191, 192, 207, 208, 239, 240, 255, 256, 257, 320, 463
SIZES = [(1, 175), (15, 176), (92, 100), (7, 200), (8, 200), (38, 201), (40, 200), (255, 0), (1, 255), (3, 254),
         (20, 300), (13, 450)]


@pytest.mark.parametrize("d,nu,nt", [(1, 0.5, 1), (2, 1.5, 3), (3, 2.5, 1)])
def test_large_block_sizes_match_oracle(d, nu, nt):
    from paper_2410_04477_amd import api
    g = W.rng(640 + d)
    ls = [600] + [l for l, _ in SIZES]           # the first block (600 points, no neighbours) feeds the others
    bp = np.concatenate([[0], np.cumsum(ls)])
    nb = [np.empty(0, np.int64)] + [np.sort(g.choice(600, m, replace=False)) for _, m in SIZES]
    npt = np.concatenate([[0], np.cumsum([len(v) for v in nb])])
    nid = np.concatenate(nb)
    n = int(bp[-1])
    s, y = g.random((n, d)), g.standard_normal(n)
    ths = [W.Theta(1.3, 0.1 * (k + 1), 0.01, nu) for k in range(nt)]
    t = lambda a, dt=torch.float64: torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    plan = api.Plan(t(bp, torch.int32), t(npt, torch.int32), n, nt)
    assert plan.c.nlarge == len(ls)
    ll, _, part = api.loglik(plan, t(s), t(y), t(nid, torch.int32), ths, "fp64", want_partial=True)
    for k, th in enumerate(ths):
        ref = OL.block_terms(s, y, bp, npt, nid, th)
        np.testing.assert_allclose(part[k].cpu().numpy(), ref, rtol=1e-8, atol=1e-9)
        assert abs(float(ll[k]) - ref.sum()) <= 1e-8 * abs(ref.sum())

