"""Coordinates at the ends of FP64: points more than 2^31 range units apart are
independent, and a block with a coordinate that is not finite has no likelihood, in
every kernel that generates covariances."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import loglik as OL

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


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("p,engine", [(p, "mfma") for p in (9, 30, 60, 90, 110, 125, 140, 155, 170, 230)]
                         + [(60, "mfma_wg"), (60, "tiles")])
def test_coordinate_that_is_not_finite(p, engine, bad):
    """The blocks that hold the point, or condition on it, are NaN and counted; the
    others keep their values."""
    from paper_2410_04477_amd import api
    s, y, bp, npt, nid = _blocks(p, 5, 8, 2, 930 + p)
    q, own = p // 2, int(bp[4]) + 1           # a point that some blocks condition on, one inside block 4
    s[q, 1] = s[own, 0] = bad
    hit = [b for b in range(9) if b in (0, 4) or q in nid[npt[b]:npt[b + 1]]]
    rest = [b for b in range(9) if b not in hit]
    if not rest:   # leave one block untouched
        nid[npt[8]:npt[9]][nid[npt[8]:npt[9]] == q] = 0
        hit, rest = [b for b in hit if b != 8], [8]
    plan, *args = _plan(api, (s, y, bp, npt, nid), engine=engine)
    for nu in (0.5, 1.5, 2.5) + ((1.3,) if p <= 175 and engine == "mfma" else ()):
        th = W.Theta(1.5, 0.3, 0.25, nu)
        ref = OL.block_terms(s, y, bp, npt, nid, th, rest)
        for precision in ("fp64", "fp32"):
            calls = [api.loglik] + ([api.loglik_grad] if p <= 175 else [])
            for call in calls:
                out = call(plan, *args, [th], precision, want_partial=True)
                ll, cnt, part = (out[0], out[1], out[2]) if call is api.loglik else (out[0], out[2], out[3])
                part = part[0].cpu().numpy()
                assert np.isnan(part[hit]).all() and torch.isnan(ll).all(), (nu, precision, call.__name__)
                assert int(cnt[0, 1]) == len(hit), (nu, precision, call.__name__, cnt)
                np.testing.assert_allclose(part[rest], ref, rtol=1e-9 if precision == "fp64" else 1e-4, atol=1e-4 if precision == "fp32" else 1e-9)
