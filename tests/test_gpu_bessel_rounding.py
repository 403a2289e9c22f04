"""The Bessel form's correlation and its two derivatives against 80-bit arithmetic:
rounding errors of rho by range of the distance, the derivatives one pair a block
on both sides of every line between the evaluation rules, and gradients at orders
below 1/2."""
import numpy as np
import pytest
import torch
from scipy import special

import workloads as W
from cases import problem
from oracle import loglik as OL

pytestmark = pytest.mark.gpu
L = np.longdouble


def _t(a, dt=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dt, device="cuda")


def _functions(x, nu):
    """rho, x d K-form (d rho / d range at range 1) and d rho / d nu by the trapezoidal rule on the
    integral representation, step 1/24, in 80 bits."""
    x, v = np.asarray(x, L)[:, None], L(nu)
    t = np.arange(900, dtype=L)[None] / 24
    w = np.exp(-x * (np.cosh(t) - 1)) / 24
    w[:, 0] /= 2
    k, k1, dk = [(w * f).sum(1) for f in (np.cosh(v * t), np.cosh((v - 1) * t), t * np.sinh(v * t))]
    x = x[:, 0]
    c = np.exp((1 - v) * np.log(L(2)) + v * np.log(x) - x - L(special.gammaln(nu)))
    return c * k, c * x * k1, c * (k * (np.log(x) - np.log(L(2)) - L(special.digamma(nu))) + dk)


@pytest.mark.parametrize("nu", [0.3, 0.8, 1.0, 2.0])
@pytest.mark.parametrize("lo,hi,bound", [(1e-3, 2.0, 4e-16), (2.0, 16.0, 4e-16), (16.0, 72.0, 1.6e-15)])
def test_rounding_errors_of_rho(nu, lo, hi, bound):
    """One neighbour's conditional mean is rho.  The distances have 24 bits, so that
    their squares and the distances found are exact; root mean square of the relative
    error over 512 of them (the rules that evaluate them, emulated on the CPU, keep
    3e-16, 3e-16 and 1.2e-15)."""
    from paper_2410_04477_amd import api
    x = np.geomspace(lo, hi, 512).astype(np.float32).astype(np.float64)
    s_obs = np.stack([np.arange(x.size) * 1024.0, np.zeros(x.size)], 1)
    s_new = s_obs + np.stack([np.zeros(x.size), x], 1)
    step = np.arange(x.size + 1)
    plan = api.Plan(_t(step, torch.int32), _t(step, torch.int32), x.size, 1, "mfma", predict=True)
    mean, _, _ = api.predict(plan, _t(s_obs), _t(np.ones(x.size)), _t(s_new), _t(step[:-1], torch.int32),
                             W.Theta(1.0, 1.0, 0.0, nu))
    rho = _functions(x, nu)[0]
    err = (mean.cpu().numpy().astype(L) - rho) / rho
    rms = float(np.sqrt((err ** 2).mean()))
    print(f"nu {nu} x in [{lo}, {hi}]: {rms:.1e}")
    assert rms <= bound


X = [1e-7, 1e-5, 3e-4, 0.0038, 0.0040, 0.0311, 0.0314, 0.5, 1.99, 2.01, 15.9, 16.1, 30.0, 71.9, 72.1, 80.0]


@pytest.mark.parametrize("nu", [0.1, 0.3, 0.49, 0.8, 1.2, 2.3, 10.0])
def test_derivatives_of_one_pair(nu):
    """Blocks of one point with one neighbour and y = 0, whose term is
    -log(a - rho^2 / a) / 2 and a constant (a = sigma2 + nugget): d l / d range = d l / d rho
    d rho / d range and the same in nu, without any cancellation in d l / d rho =
    rho / (a^2 - rho^2).  The distance is off by 2^-52 of itself at most, which moves rho
    and its derivatives by up to 80 times that, 1.8e-14, each; d rho / d nu is the sum
    of two terms of which each has such an error."""
    from paper_2410_04477_amd import api
    x = np.array(X + ([5e-8] if nu > 0.5 else []))
    n = x.size
    s = np.zeros((2 * n, 2))
    s[:n, 0] = s[n:, 0] = np.arange(n) * 1e4
    s[n:, 1] = x
    th = W.Theta(1.0, 1.0, 0.25, nu)
    bp, npt = np.arange(2 * n + 1), np.concatenate([np.zeros(n + 1, np.int64), np.arange(1, n + 1)])
    plan = api.Plan(_t(bp, torch.int32), _t(npt, torch.int32), 2 * n, 1)
    args = (plan, _t(s), _t(np.zeros(2 * n)), _t(np.arange(n), torch.int32), [th])
    got = api.loglik_grad_nu(*args, "fp64", want_partial=True)[4][0].cpu().numpy()[n:]
    got3 = api.loglik_grad(*args, "fp64", want_partial=True)[4][0].cpu().numpy()[n:]
    rho, dr, dn = _functions(x, nu)
    dl = rho / (L(1.25) ** 2 - rho ** 2)
    tol = 1e-13
    np.testing.assert_allclose(got[:, 1], (dl * dr).astype(np.float64), rtol=tol)
    np.testing.assert_allclose(got3[:, 1], (dl * dr).astype(np.float64), rtol=tol)
    terms = np.abs(dn) + 2 * rho * np.abs(np.log(x) - np.log(2) - special.digamma(nu))
    assert np.all(np.abs(got[:, 3] - dl * dn) <= tol * dl * terms), (got[:, 3], dl * dn)


@pytest.mark.parametrize("nu", [0.1, 0.3, 0.49])
def test_gradient_at_orders_below_one_half(nu):
    from paper_2410_04477_amd import api
    th = W.Theta(1.2, 0.08, 1e-2, nu)
    pb = problem("gnu-adj-2", 700, 2, 50, 30, W.Theta(1.2, 0.08, 1e-3, 1.5), 97)
    args = (pb["locs_perm"], pb["y_perm"], pb["block_ptr"], pb["nbr_ptr"], pb["nbr_idx"])
    ref = np.concatenate([OL.grad_trace(*args, th), OL.grad_nu_trace(*args, th)[:, None]], 1)
    plan = api.Plan(_t(pb["block_ptr"], torch.int32), _t(pb["nbr_ptr"], torch.int32), 700, 1)
    call = (plan, _t(pb["locs_perm"]), _t(pb["y_perm"]), _t(pb["nbr_idx"], torch.int32), [th])
    gp4 = api.loglik_grad_nu(*call, "fp64", want_partial=True)[4][0].cpu().numpy()
    gp3 = api.loglik_grad(*call, "fp64", want_partial=True)[4][0].cpu().numpy()
    scale = np.abs(ref).max(0)
    np.testing.assert_allclose(gp4, ref, rtol=1e-8, atol=1e-8 * scale.max())
    np.testing.assert_allclose(gp3, ref[:, :3], rtol=1e-8, atol=1e-8 * scale.max())
    gp32 = api.loglik_grad_nu(*call, "fp32", want_partial=True)[4][0].cpu().numpy()
    assert np.linalg.norm(gp32 - ref) <= 1e-3 * np.linalg.norm(ref)
