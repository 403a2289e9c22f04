"""Distances far outside the exponential's range: points more than 2^31 range units
apart are independent, in every kernel that generates covariances."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _blocks(p, l, nblk, d, seed):
    """A first block of p points without neighbours, then nblk blocks of l points
    with p - l of its points as neighbours."""
    g = W.rng(seed)
    ls = [p] + [l] * nblk
    nb = [np.empty(0, np.int64)] + [np.sort(g.choice(p, p - l, replace=False)) for _ in range(nblk)]
    bp = np.concatenate([[0], np.cumsum(ls)])
    npt = np.concatenate([[0], np.cumsum([len(v) for v in nb])])
    n = int(bp[-1])
    return g.random((n, d)), g.standard_normal(n), bp, npt, np.concatenate(nb)


def _plan(api, pb, **kw):
    t = lambda a, dt=torch.float64: torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    s, y, bp, npt, nid = pb
    return api.Plan(t(bp, torch.int32), t(npt, torch.int32), s.shape[0], 1, **kw), t(s), t(y), t(nid, torch.int32)


@pytest.mark.parametrize("p", [9, 30, 60, 90, 110, 125, 140, 155, 170, 230])
@pytest.mark.parametrize("rng", [1e-12, 1e-100])
def test_far_points_are_independent(p, rng):
    from paper_2410_04477_amd import api
    pb = _blocks(p, 5, 6, 2, 900 + p)
    plan, *args = _plan(api, pb)
    for nu in (0.5, 1.5, 2.5) + ((1.3,) if p <= 175 else ()):
        th = W.Theta(1.5, rng, 0.25, nu)
        ref = -0.5 * (np.log(2 * np.pi * 1.75) + pb[1] ** 2 / 1.75)
        ref = np.add.reduceat(ref, pb[2][:-1])
        ll, cnt, part = api.loglik(plan, *args, [th], "fp64", want_partial=True)
        np.testing.assert_allclose(part[0].cpu().numpy(), ref, rtol=1e-12, atol=1e-12)
        assert int(cnt.sum()) == 0
