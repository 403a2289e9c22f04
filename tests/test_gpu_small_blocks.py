"""Value and gradient of plans whose largest size class has one or two tile rows
(joint sizes up to 15 and 31), where the 16 x 16 transposition of the diagonal
inverses exceeds four panel columns: per block against the oracle, in FP64,
FP32-bulk and the Bessel form, with one point a block, many, and no neighbours."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import coracle, loglik as OL

pytestmark = pytest.mark.gpu
# (block points, neighbours)
ONE_TILE = [(1, 0), (9, 0), (15, 0), (1, 8), (4, 6), (9, 1), (1, 14), (14, 1), (8, 7), (5, 10)]
TWO_TILES = ONE_TILE + [(16, 0), (1, 15), (6, 10), (31, 0), (1, 30), (30, 1), (15, 16), (20, 11), (2, 14), (16, 15)]


def _problem(sizes, d, seed):
    g = W.rng(seed)
    ls, nb = [10] * 4, [np.empty(0, np.int64)] * 4        # 40 points to condition on
    for l, m in sizes:
        ls.append(l)
        nb.append(np.sort(g.choice(40, m, replace=False)))
    bp = np.concatenate([[0], np.cumsum(ls)])
    npt = np.concatenate([[0], np.cumsum([len(v) for v in nb])])
    n = int(bp[-1])
    return g.random((n, d)), g.standard_normal(n), bp, npt, np.concatenate(nb)


def _run(call, pb, thetas, precision):
    from paper_2410_04477_amd import api
    t = lambda a, dt=torch.float64: torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")
    s, y, bp, npt, nid = pb
    plan = api.Plan(t(bp, torch.int32), t(npt, torch.int32), s.shape[0], len(thetas))
    ll, g, _, part, gpart = getattr(api, call)(plan, t(s), t(y), t(nid, torch.int32), thetas, precision,
                                               want_partial=True)
    tiles = max(int(c) + 1 for c in plan.c.bucket_cfg[:plan.c.nbuckets])
    return [v.cpu().numpy() for v in (ll, g, part, gpart)] + [tiles]


@pytest.mark.parametrize("sizes,tiles", [(ONE_TILE, 1), (TWO_TILES, 2)])
@pytest.mark.parametrize("d,nu", [(1, 0.5), (2, 1.5), (3, 2.5)])
def test_gradient_of_small_blocks_matches_oracle(sizes, tiles, d, nu):
    pb = _problem(sizes, d, 310 + tiles)
    ths = [W.Theta(1.3, 0.15, 0.02, nu), W.Theta(0.8, 0.3, 0.05, nu)]
    ll, g, part, gpart, got = _run("loglik_grad", pb, ths, "fp64")
    _, g32, part32, gpart32, _ = _run("loglik_grad", pb, ths, "fp32")
    assert got == tiles
    for k, th in enumerate(ths):
        val, ref = coracle.block_terms(*pb, th), coracle.grad_terms(*pb, th)
        np.testing.assert_allclose(part[k], val, rtol=1e-8, atol=1e-9)
        np.testing.assert_allclose(gpart[k], ref, rtol=1e-7, atol=1e-8 * np.abs(ref).max())
        assert abs(ll[k] - val.sum()) <= 1e-8 * abs(val.sum())
        assert np.linalg.norm(g[k] - ref.sum(0)) <= 1e-8 * np.linalg.norm(ref.sum(0))
        np.testing.assert_allclose(part32[k], val, rtol=1e-3, atol=1e-3)
        assert np.linalg.norm(gpart32[k] - ref) <= 1e-3 * np.linalg.norm(ref)
        assert np.all(np.abs(g32[k] - ref.sum(0)) <= 1e-3 * np.abs(ref).sum(0))


@pytest.mark.parametrize("sizes,tiles", [(ONE_TILE, 1), (TWO_TILES, 2)])
@pytest.mark.parametrize("nu", [0.8, 1.5])
def test_four_derivatives_of_small_blocks_match_oracle(sizes, tiles, nu):
    pb = _problem(sizes, 2, 320 + tiles)
    th = W.Theta(1.3, 0.15, 0.02, nu)
    ref = np.concatenate([OL.grad_trace(*pb, th), OL.grad_nu_trace(*pb, th)[:, None]], 1)
    val = OL.block_terms(*pb, th)
    _, _, part, gpart, got = _run("loglik_grad_nu", pb, [th], "fp64")
    _, _, part32, gpart32, _ = _run("loglik_grad_nu", pb, [th], "fp32")
    assert got == tiles
    np.testing.assert_allclose(part[0], val, rtol=1e-8, atol=1e-9)
    np.testing.assert_allclose(gpart[0], ref, rtol=1e-7, atol=1e-8 * np.abs(ref).max())
    np.testing.assert_allclose(part32[0], val, rtol=1e-3, atol=1e-3)
    assert np.linalg.norm(gpart32[0] - ref) <= 1e-3 * np.linalg.norm(ref)
