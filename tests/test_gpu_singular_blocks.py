"""Blocks whose covariance is singular (a duplicate point, no nugget) in every FP64 value
kernel.  The exact pivot of the second copy is zero, so the computed one is rounding:
the block is NaN and counted if that comes out at zero or below, and finite and
not counted otherwise (about half of the blocks either way, in every kernel and the
kernels before them).  What has to hold: NaN and the counter agree, the FP32 guard
re-runs every such block with the same outcome, and the other blocks keep their values."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import loglik as OL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [3, 4, 6, 7, 8, 9, 10, 11, 14])
@pytest.mark.parametrize("nu", [0.5, 1.5])
def test_duplicate_point_without_nugget(tiles, nu):
    from paper_2410_04477_amd import api
    g = W.rng(70 + tiles)
    p, l, nblk = 16 * tiles - 5, 12, 24
    ls = [p] + [l] * nblk
    nb = [np.empty(0, np.int64)] + [np.sort(g.choice(p, p - l, replace=False)) for _ in range(nblk)]
    bp = np.concatenate([[0], np.cumsum(ls)])
    npt = np.concatenate([[0], np.cumsum([len(v) for v in nb])])
    nid, n = np.concatenate(nb), int(bp[-1])
    s, y = g.random((n, 2)), g.standard_normal(n)
    double = np.zeros(nblk + 1, bool)
    double[1::2] = True
    for b in np.flatnonzero(double):   # a copy inside the block, or of a neighbour
        j = int(g.integers(1, l))
        s[bp[b] + j] = s[bp[b] + int(g.integers(j))] if b % 4 == 1 else s[nb[b][int(g.integers(p - l))]]
    t = lambda a, dt=torch.float64: torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    plan = api.Plan(t(bp, torch.int32), t(npt, torch.int32), n, 1)
    assert max(int(c) + 1 for c in plan.c.bucket_cfg[:plan.c.nbuckets]) == (tiles if tiles <= 11 else 32)
    th = W.Theta(1.2, 0.2, 0.0, nu)
    args = (plan, t(s), t(y), t(nid, torch.int32), [th])
    ll, cnt, part = api.loglik(*args, "fp64", want_partial=True)
    part = part[0].cpu().numpy()
    bad = np.isnan(part)
    assert not bad[~double].any() and int(cnt[0, 1]) == bad.sum() and bool(torch.isnan(ll[0])) == bad.any()
    ref = OL.block_terms(s, y, bp, npt, nid, th, np.flatnonzero(~double))
    np.testing.assert_allclose(part[~double], ref, rtol=1e-8, atol=1e-9)
    _, cnt32, part32 = api.loglik(*args, "fp32", want_partial=True)
    part32 = part32[0].cpu().numpy()
    assert int(cnt32[0, 0]) >= double.sum() and int(cnt32[0, 1]) == bad.sum()
    np.testing.assert_array_equal(part32[double], part[double])
