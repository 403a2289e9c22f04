"""FP64 value of the size classes that the transposed-tile kernel runs (seven to
ten tile rows): joint sizes around the edges of tiles and of four-column panels,
smaller blocks that run in the same class, and the border row in every tile row,
against the numpy oracle."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import loglik as OL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g,d,nu", [(7, 2, 0.5), (8, 3, 1.5), (9, 1, 2.5), (10, 3, 2.5)])
def test_value_sizes_match_oracle(g, d, nu):
    from paper_2410_04477_amd import api
    rng = W.rng(700 + g)
    top = 16 * g - 1                     # largest joint size of the class
    sizes = [top, top - 1, top - 3, top - 4, top - 5, top - 14, top - 15] + list(range(1, 16 * (g - 1), 9))
    ls = [16] * 10                       # earlier points to condition on
    nb = [np.empty(0, np.int64)] * 10
    for k, p in enumerate(sizes):
        l = min(p, 1 + 5 * (k % 4))
        ls.append(l)
        nb.append(np.sort(rng.choice(160, p - l, replace=False)))
    bp = np.concatenate([[0], np.cumsum(ls)])
    npt = np.concatenate([[0], np.cumsum([len(v) for v in nb])])
    nid = np.concatenate(nb)
    n = int(bp[-1])
    s, y = rng.random((n, d)), rng.standard_normal(n)
    ths = [W.Theta(1.3, 0.1, 0.01, nu), W.Theta(0.7, 0.3, 0.05, nu)]
    t = lambda a, dt=torch.float64: torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    plan = api.Plan(t(bp, torch.int32), t(npt, torch.int32), n, 2)
    assert max(int(c) + 1 for c in plan.c.bucket_cfg[:plan.c.nbuckets]) == g
    ll, cnt, part = api.loglik(plan, t(s), t(y), t(nid, torch.int32), ths, "fp64", want_partial=True)
    for k, th in enumerate(ths):
        ref = OL.block_terms(s, y, bp, npt, nid, th)
        np.testing.assert_allclose(part[k].cpu().numpy(), ref, rtol=1e-8, atol=1e-9)
        assert abs(float(ll[k]) - ref.sum()) <= 1e-8 * abs(ref.sum())
    assert int(cnt.sum()) == 0
