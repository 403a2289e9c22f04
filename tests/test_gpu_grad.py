"""GPU adjoint gradient and simulator against the oracle.

Gradient tolerances (norm-wise, ||dg|| / ||g||): FP64 adjoint vs the oracle's
trace-formula gradient <= 1e-8; vs central finite differences of the FP64
log-likelihood (h = 1e-5 absolute on the natural parameters) within their
own step-halving truncation estimate, and vs the Richardson-extrapolated
difference <= 1e-6; FP32-bulk gradient vs FP64 <= 1e-3 (norm-wise on per-block
terms, or per component on the cancellation-free scale sum_i |dl_i| for
totals near the truth)."""
import numpy as np
import pytest
import torch

import workloads as W
from cases import oracle_terms, problem, workload_problem
from oracle import coracle

pytestmark = pytest.mark.gpu
# one-wave matrix-core (default), four-wave matrix-core, vector-ALU register tiles
ENGINES = ["mfma", "mfma_wg", "tiles"]
DEV = "cuda"


def _model(pb, nu, aniso=(1.0, 1.0, 1.0), max_theta=1, engine="mfma"):
    from paper_2410_04477_amd.model import BlockVecchia
    t = lambda a, dt: torch.tensor(np.asarray(a), dtype=dt, device=DEV)
    nidx = pb["nbr_idx"] if len(pb["nbr_idx"]) else np.zeros(1)
    return BlockVecchia.from_prepared(t(pb["locs_perm"], torch.float64), t(pb["y_perm"], torch.float64),
                                      t(pb["block_ptr"], torch.int32), t(pb["nbr_ptr"], torch.int32),
                                      t(nidx, torch.int32), nu, aniso, max_theta, engine)


def _oracle_grad(pb, th):
    return coracle.grad_terms(pb["locs_perm"], pb["y_perm"], pb["block_ptr"], pb["nbr_ptr"], pb["nbr_idx"], th)


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


@pytest.mark.parametrize("m,bc,nu,d", [(0, 60, 1.5, 2), (12, 60, 0.5, 2), (30, 100, 1.5, 2), (60, 100, 2.5, 3),
                                       (100, 120, 1.5, 2), (140, 300, 2.5, 3), (160, 600, 0.5, 2)])
@pytest.mark.parametrize("engine", ENGINES)
def test_adjoint_matches_oracle_per_block(m, bc, nu, d, engine):
    aniso = (1.0, 1.0, 0.3) if d == 3 else (1.0, 1.0, 1.0)
    th = W.Theta(1.2, 0.06, 2e-3, nu, aniso)
    pb = problem(f"g{m}", 1500, d, bc, m, th, 50 + m, zmax=0.3)
    mod = _model(pb, nu, aniso, engine=engine)
    ll, g, cnt, part, gpart = mod.loglik_grad([mod.theta(th.sigma2, th.beta, th.nugget)], "fp64", True)
    ref = _oracle_grad(pb, th)
    gp = gpart[0].cpu().numpy()
    np.testing.assert_allclose(gp, ref, rtol=1e-7, atol=1e-8 * np.abs(ref).max())
    assert _rel(g[0].cpu().numpy(), ref.sum(0)) <= 1e-8
    # the value path of the adjoint kernel equals the forward kernel's
    llf = mod.loglik([mod.theta(th.sigma2, th.beta, th.nugget)])[0]
    assert abs(float(ll[0]) - float(llf[0])) <= 1e-12 * abs(float(llf[0]))


@pytest.mark.parametrize("engine", ENGINES)
@pytest.mark.parametrize("bc,m", [(18, 20), (40, 0)])
def test_adjoint_many_right_hand_sides(bc, m, engine):
    """Blocks of about 40-85 points, so l_i + 2 right-hand sides exceed one
    32-column pass of the one-wave adjoint (several passes, the factor kept in
    the tiles).  Engines that hold the right-hand sides whole in LDS either fit
    or report VECCHIA_EUNSUPPORTED, never a wrong value."""
    from paper_2410_04477_amd._lib import VecchiaError
    th = W.Theta(1.1, 0.08, 1e-3, 1.5)
    pb = problem(f"rhs{bc}", 1500, 2, bc, m, th, 71 + bc)
    assert np.diff(pb["block_ptr"]).max() + 2 > 32   # at least two passes of 32
    mod = _model(pb, 1.5, engine=engine)
    t = [mod.theta(th.sigma2, th.beta, th.nugget)]
    try:
        ll, g, cnt, part, gpart = mod.loglik_grad(t, "fp64", True)
    except VecchiaError as e:
        assert engine != "mfma" and "unsupported" in str(e), str(e)
        return
    ref = _oracle_grad(pb, th)
    np.testing.assert_allclose(gpart[0].cpu().numpy(), ref, rtol=1e-7, atol=1e-8 * np.abs(ref).max())
    np.testing.assert_allclose(part[0].cpu().numpy(), oracle_terms(pb, th), rtol=1e-9, atol=1e-9)
    _, _, _, _, gpart32 = mod.loglik_grad(t, "fp32", True)
    assert _rel(gpart32[0].cpu().numpy(), ref) <= 1e-3


def test_fp32_gradient_large_classes_vs_oracle():
    """p_i + 1 in (144, 176]: the FP32 gradient of these size classes runs the
    register-resident kernel at one wave per SIMD (G = 10) or two launches
    (G = 11: factorisation + tiles, then the adjoint from the tiles); the FP64
    one, direct or as the forced re-run of every block, the left-looking
    factorisation launch and the adjoint launch.  Per-block FP32 terms within
    1e-3 (norm-wise) of the FP64 oracle, FP32 values within 1e-3 per block and
    1e-4 on the total; the forced-refactor path reproduces FP64 exactly."""
    th = W.Theta(1.0, 0.1, 2e-3, 1.5)
    pb = problem("big32", 3000, 2, 150, 130, th, 81)
    p = np.diff(pb["block_ptr"]) + np.diff(pb["nbr_ptr"])
    assert ((p + 1 > 144) & (p + 1 <= 176)).sum() > 50
    mod = _model(pb, 1.5)
    assert any(cfg >= 9 for cfg, _ in mod.plan.buckets())
    t = [mod.theta(th.sigma2, th.beta, th.nugget)]
    ll, g, cnt, part, gpart = mod.loglik_grad(t, "fp32", True)
    ref = _oracle_grad(pb, th)
    big = (p + 1 > 144)
    assert _rel(gpart[0].cpu().numpy()[big], ref[big]) <= 1e-3
    assert _rel(gpart[0].cpu().numpy(), ref) <= 1e-3
    rterms = np.asarray(oracle_terms(pb, th))
    np.testing.assert_allclose(part[0].cpu().numpy(), rterms, rtol=1e-3, atol=1e-3)
    assert abs(float(ll[0]) - rterms.sum()) <= 1e-4 * abs(rterms.sum())
    l64, g64, _, _, _ = mod.loglik_grad(t, "fp64")
    lf, gf, cf, _, _ = mod.loglik_grad(t, "fp32_force_refactor")
    assert int(cf[0, 0]) == len(p)
    assert torch.equal(g64, gf) and torch.equal(l64, lf)


def test_adjoint_vs_central_fd_and_fp32():
    """Central differences with h = 1e-5 (absolute, natural parameters).  Their
    truncation error is O(h^2 f3) (f3 the third derivative), which grows like
    1/nugget^2 relative, so the check uses the step-halving estimate of that
    error and a Richardson-extrapolated difference (error O(h^4))."""
    th = W.Theta(1.5, 0.08, 0.01, 1.5)
    pb = problem("fd", 6000, 2, 600, 50, th, 61, ysim="block")
    mod = _model(pb, 1.5)
    base = (th.sigma2, th.beta, th.nugget)
    _, g, _, _, _ = mod.loglik_grad([mod.theta(*base)], "fp64")
    g = g[0].cpu().numpy()

    def fd(h):
        out = []
        for k in range(3):
            up, dn = list(base), list(base)
            up[k] += h
            dn[k] -= h
            lu = float(mod.loglik([mod.theta(*up)])[0][0])
            ld = float(mod.loglik([mod.theta(*dn)])[0][0])
            out.append((lu - ld) / (2 * h))
        return np.array(out)

    f1, f2 = fd(1e-5), fd(0.5e-5)
    rich = (4 * f2 - f1) / 3
    trunc = np.abs(f1 - f2) * 4 / 3
    print("adjoint", g, "fd(1e-5)", f1, "richardson", rich)
    assert np.all(np.abs(g - f1) <= 1.5 * trunc + 1e-7 * np.linalg.norm(g))
    assert _rel(g, rich) <= 1e-6
    # FP32-bulk at the generating theta, where the block terms cancel in the
    # sum: within 1e-3 of the cancellation-free scale sum_i |dl_i| per component
    _, _, _, _, gp64 = mod.loglik_grad([mod.theta(*base)], "fp64", want_partial=True)
    _, g32, _, _, _ = mod.loglik_grad([mod.theta(*base)], "fp32")
    scale = gp64[0].abs().sum(0).cpu().numpy()
    assert np.all(np.abs(g32[0].cpu().numpy() - g) <= 1e-3 * scale), (g32[0], g, scale)


@pytest.mark.parametrize("engine", ENGINES)
def test_fp32_forced_refactor_gradient_equals_fp64(engine):
    th = W.Theta(1.0, 0.05, 1e-3, 2.5)
    pb = problem("gforce", 2000, 2, 200, 40, th, 62, ysim="block")
    mod = _model(pb, 2.5, engine=engine)
    t = [mod.theta(th.sigma2, th.beta, th.nugget)]
    l64, g64, _, _, _ = mod.loglik_grad(t, "fp64")
    lf, gf, cnt, _, _ = mod.loglik_grad(t, "fp32_force_refactor")
    assert int(cnt[0, 0]) == 200
    assert torch.equal(g64, gf) and torch.equal(l64, lf)


def test_c4_full_size_gradient_vs_oracle():
    """n = 200,000, 20,000 blocks, m = 100: adjoint at theta0 and at the truth."""
    w = W.C4
    pb = workload_problem(w, ysim="block")
    mod = _model(pb, 1.5, max_theta=2)
    thetas = [W.Theta(*W.C4_THETA0, 1.5), w.theta]
    ll, g, cnt, _, _ = mod.loglik_grad([mod.theta(t.sigma2, t.beta, t.nugget) for t in thetas], "fp64")
    ll32, g32, _, _, _ = mod.loglik_grad([mod.theta(t.sigma2, t.beta, t.nugget) for t in thetas], "fp32")
    for i, th in enumerate(thetas):
        terms = _oracle_grad(pb, th)
        ref = terms.sum(0)
        assert _rel(g[i].cpu().numpy(), ref) <= 1e-8
        # FP32: each block's terms carry a relative error of order kappa * u32; near
        # the truth the block terms cancel in the sum, so the bound is taken on the
        # cancellation-free scale sum_i |dl_i|, per component
        scale = np.abs(terms).sum(0)
        assert np.all(np.abs(g32[i].cpu().numpy() - ref) <= 1e-3 * scale), (g32[i], ref, scale)
        ref_ll = coracle.loglik(pb["locs_perm"], pb["y_perm"], pb["block_ptr"], pb["nbr_ptr"], pb["nbr_idx"], th)
        assert abs(float(ll[i]) - ref_ll) <= 1e-8 * abs(ref_ll)
        assert abs(float(ll32[i]) - ref_ll) <= 1e-4 * abs(ref_ll)
        print(f"C4 theta {i}: loglik rel err fp64 {abs(float(ll[i]) - ref_ll) / abs(ref_ll):.2e} fp32-bulk "
              f"{abs(float(ll32[i]) - ref_ll) / abs(ref_ll):.2e}; gradient rel err fp64 "
              f"{_rel(g[i].cpu().numpy(), ref):.2e}, fp32-bulk per component vs sum|dl_i| "
              f"{np.array2string(np.abs(g32[i].cpu().numpy() - ref) / scale, precision=2)}")


@pytest.mark.parametrize("engine", ENGINES)
def test_value_of_gradient_call_on_a_fresh_plan(engine):
    """vecchia_loglik_grad on a plan that never ran vecchia_loglik: its values
    (total and per block) come from the gradient kernels alone and equal the
    oracle's, in FP64 and FP32-bulk, for classes that keep the factor in
    registers and classes that go through the tile buffer."""
    th = W.Theta(1.2, 0.07, 3e-3, 1.5)
    for m, bc in ((40, 400), (120, 150)):
        pb = problem(f"fresh{m}", 3000, 2, bc, m, th, 55 + m, ysim="exact")
        ref = oracle_terms(pb, th)
        for prec, tol in (("fp64", 1e-8), ("fp32", 1e-4)):
            mod = _model(pb, 1.5, engine=engine)
            ll, _, _, part, _ = mod.loglik_grad([mod.theta(th.sigma2, th.beta, th.nugget)], prec, want_partial=True)
            assert abs(float(ll[0]) - ref.sum()) <= tol * abs(ref.sum()), (m, prec, float(ll[0]), ref.sum())
            if prec == "fp64":
                np.testing.assert_allclose(part[0].cpu().numpy(), ref, rtol=1e-8, atol=1e-9)


def test_c4_full_size_mle_end_point_judged_by_oracle():
    """n = 200,000, 20,000 blocks, m = 100: L-BFGS from theta0 = (1, 0.05, 0.05)
    with the FP64 adjoint, then the oracle's own gradient at the end point:
    stationary to 1e-3 of the cancellation-free scale sum_i |dl_i| per
    component, and the oracle's log-likelihood there at least its value at
    the generating theta."""
    from paper_2410_04477_amd import mle
    w = W.C4
    pb = workload_problem(w, ysim="block")
    mod = _model(pb, 1.5)
    res = mle.fit(mod, W.C4_THETA0, "fp64", max_evals=120)
    th_hat = W.Theta(*res.theta, 1.5)
    terms = _oracle_grad(pb, th_hat)
    g, scale = terms.sum(0), np.abs(terms).sum(0)
    args = (pb["locs_perm"], pb["y_perm"], pb["block_ptr"], pb["nbr_ptr"], pb["nbr_idx"])
    ll_hat, ll_true = coracle.loglik(*args, th_hat), coracle.loglik(*args, w.theta)
    ll0 = coracle.loglik(*args, W.Theta(*W.C4_THETA0, 1.5))
    print(f"C4 MLE: theta {np.array2string(np.asarray(res.theta), precision=5)} after {res.evals} evaluations "
          f"({res.seconds:.2f} s); oracle l: start {ll0:.3f}, truth {ll_true:.3f}, end {ll_hat:.3f}; "
          f"gradient / sum|dl_i| {np.array2string(np.abs(g) / scale, precision=2)}", flush=True)
    assert abs(res.loglik - ll_hat) <= 1e-8 * abs(ll_hat)
    assert ll_hat >= ll_true and ll_hat > ll0
    assert np.all(np.abs(g) <= 1e-3 * scale), (g, scale)


def test_simulator_matches_oracle():
    from paper_2410_04477_amd import api
    from oracle.preprocess import point_neighbors
    n, m = 4000, 150
    th = W.Theta(1.0, 0.05, 1e-3, 2.5, (1.0, 1.0, 0.2))
    s = W.rng(71).random((n, 3)) * [1, 1, 0.2]
    order = W.point_permutation(n, 71)
    so = s[order]
    w = [1.0, 1.0, 5.0]
    ptr, idx = point_neighbors(so * w, m)
    z = W.standard_normal(n, 72)
    ref = coracle.simulate(so, np.arange(n + 1), ptr, idx, th, z)
    t = lambda a, dt: torch.tensor(np.asarray(a), dtype=dt, device=DEV)
    y = api.simulate(t(so, torch.float64), t(ptr, torch.int32), t(idx, torch.int32), th, t(z, torch.float64))
    np.testing.assert_allclose(y.cpu().numpy(), ref, rtol=1e-9, atol=1e-9)


@pytest.mark.parametrize("n,m,sets", [(1, 5, 1), (40, 60, 2), (300, 14, 3), (700, 15, 24), (400, 142, 2), (400, 143, 1),
                                      (400, 158, 2), (400, 174, 1)])
def test_simulator_sizes_match_oracle(n, m, sets):
    """Every tile count of the coefficient kernels (from 1 to 10 tile rows in one
    wave, 11 in four), one and many data sets in one data flow.  Weights carry a
    relative error of cond(K_N) u, below 1e-11 here (nugget 1e-3), and the
    recursion keeps it: 1e-9."""
    from paper_2410_04477_amd import api
    from oracle.preprocess import point_neighbors
    x = W.rng(90 + n + m).random((n, 2))
    ptr, idx = point_neighbors(x, m)
    z = W.rng(5).standard_normal((sets, n))
    ths = [W.Theta(1.0 + 0.1 * k, 0.1, 1e-3, (0.5, 1.5, 2.5)[k % 3]) for k in range(sets)]
    t = lambda a, dt: torch.tensor(np.asarray(a), dtype=dt, device=DEV)
    ip = t(idx if len(idx) else np.zeros(1), torch.int32)
    y = api.simulate(t(x, torch.float64), t(ptr, torch.int32), ip, ths, t(z, torch.float64)).cpu().numpy()
    for k in range(sets):
        ref = coracle.simulate(x, np.arange(n + 1), ptr, idx, ths[k], z[k])
        np.testing.assert_allclose(y[k], ref, rtol=1e-9, atol=1e-9)


def test_simulator_neighbour_that_is_not_earlier():
    """A list without cycles whose neighbours are not all earlier still runs (in
    passes), and equals the same design renumbered; a cycle is refused."""
    from paper_2410_04477_amd import api
    from paper_2410_04477_amd._lib import VecchiaError
    n, th = 60, W.Theta(1.0, 0.2, 1e-2, 1.5)
    x = W.rng(3).random((n, 2))
    z = W.standard_normal(n, 4)
    t = lambda a, dt: torch.tensor(np.ascontiguousarray(a), dtype=dt, device=DEV)
    run = lambda xs, p, i, zs: api.simulate(t(xs, torch.float64), t(p, torch.int32), t(i, torch.int32), th,
                                            t(zs, torch.float64)).cpu().numpy()
    ptr = np.arange(n + 1) - 1
    ptr[0] = 0
    fwd = run(x, ptr, np.arange(n - 1), z)              # point i given point i - 1
    rptr = np.minimum(np.arange(n + 1), n - 1)          # the same chain numbered backwards
    back = run(x[::-1], rptr, np.arange(1, n), z[::-1])
    np.testing.assert_allclose(back[::-1], fwd, rtol=1e-12, atol=1e-12)
    with pytest.raises(VecchiaError):
        run(x[:2], np.array([0, 1, 2]), np.array([1, 0]), z[:2])


def test_mle_recovers_parameters_and_beats_start():
    from paper_2410_04477_amd import mle
    th = W.Theta(1.5, 0.08, 0.01, 1.5)
    pb = problem("mle", 8000, 2, 800, 40, th, 81, ysim="block")
    mod = _model(pb, 1.5)
    res = mle.fit(mod, W.C4_THETA0, "fp64", max_evals=80)
    ll_true = float(mod.loglik([mod.theta(th.sigma2, th.beta, th.nugget)])[0][0])
    ll0 = float(mod.loglik([mod.theta(*W.C4_THETA0)])[0][0])
    assert res.loglik >= ll_true - 1e-6 * abs(ll_true)   # the MLE is at least as likely as the truth
    assert res.loglik > ll0
    assert 0.5 < res.theta[0] / th.sigma2 < 2.0 and 0.5 < res.theta[1] / th.beta < 2.0
