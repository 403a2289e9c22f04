"""Performance cases of the block Vecchia library: the calls that programs built
on it make, with inputs drawn like the ones they meet, the work each call
cannot do without, and the value of its outputs in plain 64-bit arithmetic.

Inputs are seeded and made on the device with torch alone: uniform points, a
random field with the Matern spectrum plus noise for the observations, ragged
blocks around a jittered lattice in random order, and for each block the
nearest points of earlier blocks."""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2410_04477_amd import api, model, warmstart

DEVICE = "cuda"
SIGMA2, NUGGET = 1.0, {"rough": 1e-2, "fine": 1e-3}


# ------------------------------------------------------------------ the cases


def listed():
    return [
        # one likelihood of a small data set (2,000 points, 30 neighbours): the
        # call whose latency a line search over a few thousand points waits for
        dict(name="value_n2k", op="value", n=2000, d=2, bc=200, m=30, nu=0.5, nt=1, precision="fp64", partial=False),
        # a grid of parameter vectors on 100,000 points in the mixed precision,
        # as a likelihood surface is scanned
        dict(name="grid_n100k_fp32", op="value", n=100_000, d=2, bc=10_000, m=60, nu=1.5, nt=10, precision="fp32",
             partial=False),
        # one objective evaluation of a maximum-likelihood fit in the default
        # precision: value and backward through autograd (an odd point count)
        dict(name="fit_n100k", op="fit", n=100_003, d=2, bc=10_000, m=60, nu=1.5, nt=1, precision="fp64",
             partial=False),
        # value and gradient of the million-point 3-D field in the mixed
        # precision: the benchmark's step
        dict(name="grad_n1m_fp32", op="grad", n=1_000_000, d=3, bc=50_000, m=120, nu=2.5, nt=1, precision="fp32",
             partial=False),
        # the likelihood of the same field in the default precision
        dict(name="value_n1m", op="value", n=1_000_000, d=3, bc=50_000, m=120, nu=2.5, nt=1, precision="fp64",
             partial=False),
        # blocks above the one-wave limit: 450 neighbours, the accuracy study's
        # setting, with the per-block terms
        dict(name="large_n20k_m450", op="value", n=20_000, d=2, bc=1500, m=450, nu=1.5, nt=1, precision="fp64",
             partial=True),
        # a fit that estimates the smoothness too: value and all four derivatives
        # through the Bessel form
        dict(name="smoothness_n20k", op="grad_nu", n=20_000, d=2, bc=2000, m=30, nu=1.0, nt=1, precision="fp64",
             partial=False),
        # kriging of 100,000 new points from 1,000,000 observations, and draws of
        # the conditional field at them
        dict(name="predict_n100k", op="predict", n=1_000_000, d=3, bc=10_000, m=120, nu=2.5, new=100_000, draws=100),
        # setting a data set up: K-means blocks, block order, neighbours, schedule
        dict(name="setup_n200k", op="setup", n=200_000, d=2, bc=20_000, m=100, iters=30, ordering="random"),
        # training data for the learned warm start: fields drawn on one design
        dict(name="simulate_n20k", op="simulate", n=20_000, d=2, m=150, nu=1.5, nt=24),
        # their variogram features (a subset of 4,096 points of each)
        dict(name="features_k4096", op="features", k=4096, sets=64),
        # one training step of the warm-start network
        dict(name="train_b256", op="train", batch=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges of the listed ones: point counts from 500 to the
    listed largest, spread over their logarithm, any remainder of the block and
    neighbour counts modulo the kernels' tiles."""
    op = rng.choice(["value", "value", "fit", "grad", "grad", "large", "grad_nu", "predict", "setup", "simulate",
                     "features", "train"])
    d = rng.choice([2, 3])
    per = rng.uniform(7.0, 20.0)   # points per block
    nu = rng.choice([0.5, 1.5, 2.5])
    if op in ("value", "fit", "grad"):
        n = _log_int(rng, 500, 1_000_000 if op == "value" else 600_000)
        nt = 1 if op == "fit" else max(1, min(rng.choice([1, 1, 3, 10]), 600_000 // n))
        return dict(op=op, n=n, d=d, bc=min(50_000, max(4, int(n / per))), m=rng.randint(10, 120), nu=nu, nt=nt,
                    precision="fp64" if op == "fit" else rng.choice(["fp64", "fp32"]), partial=rng.random() < 0.2)
    if op == "large":
        n = _log_int(rng, 4000, 20_000)
        return dict(op="value", n=n, d=d, bc=int(n / rng.uniform(13.0, 18.0)), m=rng.randint(190, 450), nu=nu, nt=1,
                    precision=rng.choice(["fp64", "fp32"]), partial=rng.random() < 0.5)
    if op == "grad_nu":
        n = _log_int(rng, 500, 20_000)
        return dict(op=op, n=n, d=2, bc=max(4, int(n / rng.uniform(8.0, 12.0))), m=rng.randint(10, 30),
                    nu=rng.choice([0.8, 1.0, 1.25, 2.0]), nt=1, precision=rng.choice(["fp64", "fp32"]), partial=False)
    if op == "predict":
        new = _log_int(rng, 300, 100_000)
        return dict(op=op, n=10 * new, d=d, bc=max(4, int(new / per)), m=rng.randint(10, 120), nu=nu, new=new,
                    draws=rng.randint(30, 100))
    if op == "setup":
        n = _log_int(rng, 1000, 200_000)
        return dict(op=op, n=n, d=d, bc=max(4, int(n / rng.uniform(10.0, 20.0))), m=rng.randint(20, 120),
                    iters=rng.choice([10, 30]), ordering=rng.choice(["random", "random", "morton", "hilbert", "kdtree"]))
    if op == "simulate":
        return dict(op=op, n=_log_int(rng, 1000, 20_000), d=2, m=rng.randint(30, 150), nu=nu, nt=rng.randint(1, 24))
    if op == "features":
        return dict(op=op, k=_log_int(rng, 300, 4096), sets=rng.randint(1, 64))
    return dict(op="train", batch=_log_int(rng, 16, 512))


# --------------------------------------------------------------------- inputs


def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1_000_003 * int(seed) + 17)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEVICE, dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEVICE, dtype=torch.float64)


def _aniso(d):
    return (1.0, 1.0, 0.2) if d == 3 else (1.0, 1.0, 1.0)


def _points(g, n, d):
    s = _rand(g, n, d)
    if d == 3:
        s[:, 2] *= 0.2
    return s


def _scaled(s, d):
    return s / torch.tensor(_aniso(d)[:d], dtype=torch.float64, device=DEVICE)


def _truth(case):
    """(sigma2, range, nugget) of the field: ranges of a tenth to a twentieth of
    the domain, a larger nugget for rough fields."""
    nu = case.get("nu", 1.5)
    return SIGMA2, {0.5: 0.1, 2.5: 0.05}.get(nu, 0.07), NUGGET["rough" if nu < 1.0 else "fine"]


def _thetas(case, seed):
    """Parameter vectors around the truth, as an optimiser or a grid visits them."""
    s2, rg, nug = _truth(case)
    rng = np.random.default_rng(int(seed) + 5)
    f = rng.uniform(0.8, 1.25, (case.get("nt", 1), 3))
    return [(s2 * a, rg * b, nug * c, case["nu"], _aniso(case["d"])) for a, b, c in f.tolist()]


def _field(g, s, case):
    """Random field with the Matern spectrum (256 random waves) plus white noise."""
    s2, rg, nug = _truth(case)
    d, waves = case["d"], 256
    dof = max(1, round(2 * case.get("nu", 1.5)))
    w = _randn(g, waves, d) / (rg * _randn(g, waves, dof).square().sum(1, keepdim=True).sqrt())
    phase = _rand(g, waves) * (2 * math.pi)
    u, y = _scaled(s, d), torch.empty(s.shape[0], dtype=torch.float64, device=DEVICE)
    for a in range(0, s.shape[0], 200_000):
        arg = phase.expand(u[a:a + 200_000].shape[0], waves).clone()
        for k in range(d):
            arg += u[a:a + 200_000, k, None] * w[:, k]
        y[a:a + 200_000] = torch.cos(arg).sum(1)
    return y * math.sqrt(2 * s2 / waves) + math.sqrt(nug) * _randn(g, s.shape[0])


def _blocks(g, u, bc):
    """Ragged blocks in random order: each point with the nearest centre of a
    jittered lattice of about bc cells (u: scaled coordinates in the unit cube).
    Returns (order of the points, block_ptr)."""
    n, d = u.shape
    if bc >= n:
        return torch.randperm(n, generator=g, device=DEVICE), torch.arange(n + 1, dtype=torch.int64, device=DEVICE)
    side = max(1, int(round(bc ** (1.0 / d))))
    dims = [side] * (d - 1) + [max(1, bc // side ** (d - 1))]
    total = math.prod(dims)
    cell = torch.arange(total, device=DEVICE)
    axes, rest = [], cell
    for k in reversed(range(d)):
        axes.insert(0, rest % dims[k])
        rest = rest // dims[k]
    dd = torch.tensor(dims, dtype=torch.float64, device=DEVICE)
    cen = (torch.stack(axes, 1) + 0.5 + 0.3 * (_rand(g, total, d) - 0.5)) / dd
    at = torch.minimum((u * dd).long().clamp_min(0), torch.tensor(dims, device=DEVICE) - 1)
    best = torch.full((n,), math.inf, dtype=torch.float64, device=DEVICE)
    label = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    for off in range(3 ** d):
        c, flat, ok = off, torch.zeros(n, dtype=torch.int64, device=DEVICE), None
        for k in range(d):
            q = at[:, k] + (c % 3 - 1)
            c //= 3
            inside = (q >= 0) & (q < dims[k])
            ok = inside if ok is None else ok & inside
            flat = flat * dims[k] + q.clamp(0, dims[k] - 1)
        dist = (u - cen[flat]).square().sum(1)
        take = ok & (dist < best)
        best = torch.where(take, dist, best)
        label = torch.where(take, flat, label)
    pos = torch.randperm(total, generator=g, device=DEVICE)[label]
    key, order = torch.sort(pos, stable=True)
    cnt = torch.bincount(key, minlength=total)
    cnt = cnt[cnt > 0]
    return order, torch.cat([cnt.new_zeros(1), cnt.cumsum(0)])


def _nearest(u_pts, bp_pts, u_blk, bp_blk, m, earlier):
    """For each block of u_blk, up to m of the nearest points of u_pts among the
    points of its nearest blocks of u_pts (earlier: only blocks before it), by
    the distance from its centroid.  Returns (nbr_ptr, nbr_idx)."""
    def centroids(u, bp):
        cs = torch.cat([u.new_zeros(1, u.shape[1]), u.cumsum(0)])
        return ((cs[bp[1:]] - cs[bp[:-1]]) / (bp[1:] - bp[:-1])[:, None].double()).float()
    cp, cb = centroids(u_pts, bp_pts), centroids(u_blk, bp_blk)
    nb, npb, d = cb.shape[0], cp.shape[0], cb.shape[1]
    size = bp_pts[1:] - bp_pts[:-1]
    lmax = int(size.max())
    k = min(npb, int(1.5 * m / (u_pts.shape[0] / npb)) + 8 if lmax > 1 else m)
    ar = torch.arange(lmax, device=DEVICE)
    cnts, idxs = [], []
    rows = max(1, int(1.2e8 // max(npb, k * lmax)))
    for a in range(0, nb, rows):
        e = min(nb, a + rows)
        cols = min(npb, e) if earlier else npb
        dist = torch.zeros((e - a, cols), dtype=torch.float32, device=DEVICE)
        for q in range(d):
            dist += (cb[a:e, None, q] - cp[None, :cols, q]).square()
        if earlier:
            dist.masked_fill_(torch.arange(cols, device=DEVICE)[None] >= torch.arange(a, e, device=DEVICE)[:, None],
                              math.inf)
        near, j = torch.topk(dist, min(k, cols), dim=1, largest=False)
        pts = bp_pts[j][:, :, None] + ar
        ok = (near < math.inf)[:, :, None] & (ar < size[j][:, :, None])
        pts, ok = pts.reshape(e - a, -1), ok.reshape(e - a, -1)
        pts = pts.clamp_max(u_pts.shape[0] - 1)
        dp = torch.zeros(pts.shape, dtype=torch.float32, device=DEVICE)
        for q in range(d):
            dp += (u_pts[:, q].float()[pts] - cb[a:e, None, q]).square()
        dp.masked_fill_(~ok, math.inf)
        dv, sel = torch.topk(dp, min(m, dp.shape[1]), dim=1, largest=False, sorted=True)
        good = dv < math.inf
        cnts.append(good.sum(1))
        idxs.append(torch.gather(pts, 1, sel)[good])
    cnt = torch.cat(cnts)
    return torch.cat([cnt.new_zeros(1), cnt.cumsum(0)]), torch.cat(idxs)


def _data(case, seed):
    """Points, observations, blocks and neighbours of a likelihood case, in block order."""
    g = _gen(seed)
    s = _points(g, case["n"], case["d"])
    y = _field(g, s, case)
    order, bp = _blocks(g, _scaled(s, case["d"]), case["bc"])
    s, y = s[order].contiguous(), y[order].contiguous()
    u = _scaled(s, case["d"])
    nptr, nidx = _nearest(u, bp, u, bp, case["m"], True)
    return s, y, bp, nptr, nidx


def _pred_data(case, seed):
    """Observations in block order, new locations in blocks, and the nearest
    observations of each of those blocks; normals for the draws."""
    g = _gen(seed)
    n, d, new = case["n"], case["d"], case["new"]
    s = _points(g, n, d)
    y = _field(g, s, case)
    order, bp = _blocks(g, _scaled(s, d), max(4, n // 12))
    s, y = s[order].contiguous(), y[order].contiguous()
    t = _points(g, new, d)
    torder, tbp = _blocks(g, _scaled(t, d), case["bc"])
    t = t[torder].contiguous()
    nptr, nidx = _nearest(_scaled(s, d), bp, _scaled(t, d), tbp, case["m"], False)
    return s, y, t, tbp, nptr, nidx, _randn(g, case["draws"], new)


def _sim_data(case, seed):
    """A design in random order with its nearest earlier points, and normals."""
    g = _gen(seed)
    s = _points(g, case["n"], case["d"])
    unit = torch.arange(case["n"] + 1, dtype=torch.int64, device=DEVICE)
    nptr, nidx = _nearest(s, unit, s, unit, case["m"], True)
    return s, nptr, nidx, _randn(g, case["nt"], case["n"])


def _set_data(case, seed):
    """Subsets of simulated fields on one design: locations, values, smoothness slots."""
    g = _gen(seed)
    s = _rand(g, case["k"], 2)
    y = torch.stack([_field(g, s, dict(d=2, nu=(0.5, 1.5, 2.5)[q % 3])) for q in range(case["sets"])])
    slot = torch.arange(case["sets"], device=DEVICE, dtype=torch.int32) % 3
    return s, y, slot


def _net_data(case, seed):
    """A batch of variogram features (32 rising bins in one of three slots) with
    standardised targets, and a network's seed."""
    g = _gen(seed)
    b = case["batch"]
    bins = torch.linspace(0.0, 1.0, 32, device=DEVICE, dtype=torch.float64)
    curve = 1.0 - torch.exp(-bins[None] / (0.05 + 0.4 * _rand(g, b, 1))) + 0.05 * _randn(g, b, 32)
    x = torch.zeros(b, 3, 32, device=DEVICE, dtype=torch.float64)
    x[torch.arange(b, device=DEVICE), torch.arange(b, device=DEVICE) % 3] = curve
    return x.reshape(b, 96).float().contiguous(), _randn(g, b, 3).float(), int(seed) % 1000 + 1


def _i32(t):
    return t.to(torch.int32).contiguous()


def prepare(case, seed):
    op = case["op"]
    if op in ("value", "fit", "grad", "grad_nu"):
        s, y, bp, nptr, nidx = _data(case, seed)
        mod = model.BlockVecchia.from_prepared(s, y, _i32(bp), _i32(nptr), _i32(nidx), case["nu"],
                                               _aniso(case["d"])[:case["d"]], max_theta=case["nt"])
        st = dict(op=op, model=mod, thetas=_thetas(case, seed), precision=case["precision"], partial=case["partial"])
        if op == "fit":
            st["params"] = torch.tensor(st["thetas"][0][:3], dtype=torch.float64, requires_grad=True)
        return st
    if op == "predict":
        s, y, t, tbp, nptr, nidx, z = _pred_data(case, seed)
        plan = api.Plan(_i32(tbp), _i32(nptr), case["new"], 1, "mfma", predict=True)
        return dict(op=op, plan=plan, s=s, y=y, t=t, nidx=_i32(nidx), z=z, theta=_thetas(case, seed)[0])
    if op == "setup":
        g = _gen(seed)
        s = _points(g, case["n"], case["d"])
        y = _randn(g, case["n"])
        init = torch.randperm(case["n"], generator=g, device=DEVICE)[:case["bc"]].sort().values
        order = torch.randperm(case["bc"], generator=g, device=DEVICE)
        return dict(op=op, s=s, y=y, init=init, order=order, case=case)
    if op == "simulate":
        s, nptr, nidx, z = _sim_data(case, seed)
        return dict(op=op, s=s, nptr=_i32(nptr), nidx=_i32(nidx), z=z, thetas=_thetas(case, seed))
    if op == "features":
        s, y, slot = _set_data(case, seed)
        return dict(op=op, s=s, y=y, slot=slot)
    x, t, net = _net_data(case, seed)
    return dict(op=op, net=warmstart.MLP(net, DEVICE), x=x, t=t)


# ----------------------------------------------------------------- one pass


def run(st):
    op = st["op"]
    if op == "value":
        ll, cnt, part = st["model"].loglik(st["thetas"], st["precision"], st["partial"])
        return dict(loglik=ll, counters=cnt, partial=part)
    if op == "fit":
        p = st["params"]
        p.grad = None
        ll = model.vecchia_loglik(p, st["model"], st["precision"])
        ll.backward()
        return dict(loglik=ll.detach(), grad=p.grad)
    if op == "grad":
        ll, g, cnt, part, gpart = st["model"].loglik_grad(st["thetas"], st["precision"], st["partial"])
        return dict(loglik=ll, grad=g, counters=cnt, partial=part, gpartial=gpart)
    if op == "grad_nu":
        ll, g, cnt, _, _ = st["model"].loglik_grad_nu(st["thetas"], st["precision"])
        return dict(loglik=ll, grad=g, counters=cnt)
    if op == "predict":
        mean, var, _ = api.predict(st["plan"], st["s"], st["y"], st["t"], st["nidx"], st["theta"])
        return dict(mean=mean, var=var, **api.condsim(mean, var, st["z"]))
    if op == "setup":
        c = st["case"]
        mod = model.BlockVecchia(st["s"], st["y"], c["bc"], c["m"], 1.5, st["init"], st["order"],
                                 _aniso(c["d"])[:c["d"]], c["iters"], ordering=c["ordering"])
        # the lists at their capacities: the lengths depend on the drawn points
        fill = lambda t, size: torch.nn.functional.pad(t, (0, size - t.numel()), value=-1)  # noqa: E731
        return dict(perm=mod.perm, block_ptr=fill(mod.block_ptr, c["bc"] + 1), nbr_ptr=fill(mod.nbr_ptr, c["bc"] + 1),
                    nbr_idx=fill(mod.nbr_idx, c["bc"] * c["m"]), locs=mod.locs_perm, y=mod.y_perm)
    if op == "simulate":
        return dict(y=api.simulate(st["s"], st["nptr"], st["nidx"], st["thetas"], st["z"]))
    if op == "features":
        feat, gamma = api.variogram(st["s"], st["y"], st["slot"], warmstart.NBINS, warmstart.HMAX, 3,
                                    shared_design=True)
        return dict(features=feat, gamma=gamma)
    net = st["net"]
    part = net.train_step(st["x"], st["t"], 1e-3)
    return dict(loss=part, params=net.params, m=net.m, v=net.v)


# -------------------------------------------------------------------- the work


def work(case):
    """Inputs read once and outputs written once; the joint factorisations and
    solves (p^3 / 3 + p^2), the covariance entries at 30 operations, and the
    adjoint's right-hand sides (3 m^2 l + 2 m^2), per block and parameter vector."""
    op = case["op"]
    if op == "features":
        k, sets = case["k"], case["sets"]
        return dict(bytes=8.0 * k * (2 + sets) + 12.0 * 32 * sets, flops=k * (k - 1) / 2 * (8.0 + 3.0 * sets))
    if op == "train":
        b, layers = case["batch"], [(96, 256), (256, 256), (256, 3)]
        par = sum(i * o + o for i, o in layers)
        return dict(bytes=4.0 * (b * 99 + 6 * par), flops=b * (sum(6.0 * i * o for i, o in layers) - 2.0 * 96 * 256))
    n, d = case["n"], case["d"]
    if op == "setup":
        return dict(bytes=16.0 * n * (d + 1) + 8.0 * n + 4.0 * case["bc"] * (case["m"] + 2), flops=10.0 * n * case["iters"])
    if op == "simulate":
        m, nt = case["m"], case["nt"]
        return dict(bytes=8.0 * n * d + 4.0 * n * m + 16.0 * n * nt, flops=nt * n * (m ** 3 / 3.0 + 2.0 * m * m + 15.0 * m * m))
    new = case.get("new", n)
    bc, m, nt = case["bc"], case["m"], case.get("nt", 1)
    l = new / bc
    p = m + l
    out = 8.0 * nt * (4 + (bc if case.get("partial") else 0))
    if op == "predict":
        return dict(bytes=8.0 * bc * m * (d + 1) + 4.0 * bc * m + 8.0 * new * (d + case["draws"] + 6),
                    flops=bc * (m ** 3 / 3.0 + m * m * (l + 1) + m * (l + 1) ** 2 + 15.0 * p * p) + 5.0 * new * case["draws"])
    flops = p ** 3 / 3.0 + p * p + 15.0 * p * p
    if op != "value":
        flops += 3.0 * m * m * l + 2.0 * m * m + 15.0 * p * p
    return dict(bytes=8.0 * n * (d + 1) + 4.0 * bc * m + 8.0 * bc + out, flops=float(nt * bc) * flops)


# --------------------------------------------------------- the same in 64 bits


def _bessel(x, nu):
    """rho, -x drho/dx and drho/dnu of the Matern correlation of any order, from
    K_v(x) = int_0^inf exp(-x cosh t) cosh(v t) dt and its derivative in v by the
    trapezoidal rule (its error falls exponentially with the step)."""
    pos = x > 0
    z = torch.where(pos, x, torch.ones_like(x))
    h = 1.0 / 16
    top = math.acosh(60.0 / float(z.min()) + 10.0) + 1.0
    k0, k1, k2 = torch.zeros_like(z), torch.zeros_like(z), torch.zeros_like(z)
    for q in range(int(top / h) + 1):
        t = q * h
        e = torch.exp(-z * math.cosh(t)) * (h * (0.5 if q == 0 else 1.0))
        k0 += e * math.cosh(nu * t)
        k1 += e * math.cosh((nu - 1.0) * t)
        k2 += e * t * math.sinh(nu * t)
    c = 2.0 ** (1.0 - nu) / math.gamma(nu) * z ** nu
    psi = float(torch.special.digamma(torch.tensor(nu, dtype=torch.float64)))
    one = torch.ones_like(x)
    rho = torch.where(pos, c * k0, one)
    g = torch.where(pos, c * z * k1, 0 * one)
    dn = torch.where(pos, c * (k0 * (torch.log(z) - math.log(2.0) - psi) + k2), 0 * one)
    return rho, g, dn


def _corr(x, nu, grad):
    """rho(x), -x rho'(x) and, for a general order, drho/dnu (else None)."""
    if nu not in (0.5, 1.5, 2.5):
        return _bessel(x, nu)
    e = torch.exp(-x)
    if nu == 0.5:
        return e, x * e if grad else None, None
    if nu == 1.5:
        return (1 + x) * e, x * x * e if grad else None, None
    return (1 + x + x * x / 3) * e, x * x * (1 + x) / 3 * e if grad else None, None


def _dist(u, v):
    r = torch.zeros(u.shape[0], u.shape[1], v.shape[1], dtype=torch.float64, device=DEVICE)
    for k in range(u.shape[2]):
        r += (u[:, :, None, k] - v[:, None, :, k]).square()
    return r.sqrt()


def _joint(bp, nptr, nidx, a, e, shift):
    """Padded index table of blocks a..e-1: neighbours, then the block's points
    (offset by `shift`); returns (index, valid, neighbour count, block size)."""
    m, l = nptr[a + 1:e + 1] - nptr[a:e], bp[a + 1:e + 1] - bp[a:e]
    width = int((m + l).max())
    q = torch.arange(width, device=DEVICE)[None].expand(e - a, width)
    nb = q < m[:, None]
    idx = torch.where(nb, nidx[(nptr[a:e, None] + q).clamp_max(max(0, nidx.numel() - 1))] if nidx.numel() else q,
                      shift + (bp[a:e, None] + q - m[:, None]))
    ok = q < (m + l)[:, None]
    return torch.where(ok, idx, torch.zeros_like(idx)), ok, m, l


def _exact_likelihood(case, seed, grad):
    s, y, bp, nptr, nidx = _data(case, seed)
    nb, nu = bp.numel() - 1, case["nu"]
    u = _scaled(s, case["d"])
    gen = grad and nu not in (0.5, 1.5, 2.5)
    parts, gparts = [], []
    pm = int((nptr[1:] - nptr[:-1]).max() + (bp[1:] - bp[:-1]).max())
    step = max(1, int(6e7 // (pm * pm)))
    for s2, rg, nug, _, _ in _thetas(case, seed):
        ll, gg = torch.empty(nb, dtype=torch.float64, device=DEVICE), torch.zeros(nb, 4, dtype=torch.float64, device=DEVICE)
        for a in range(0, nb, step):
            e = min(nb, a + step)
            idx, ok, m, l = _joint(bp, nptr, nidx, a, e, 0)
            w = idx.shape[1]
            x = _dist(u[idx], u[idx]) / rg
            rho, dr, dn = _corr(x, nu, grad)
            both = ok[:, :, None] & ok[:, None, :]
            eye = torch.eye(w, dtype=torch.float64, device=DEVICE)
            K = torch.where(both, s2 * rho + nug * eye, eye)
            L = torch.linalg.cholesky(K)
            yv = torch.where(ok, y[idx], torch.zeros_like(y[idx]))
            wv = torch.linalg.solve_triangular(L, yv[:, :, None], upper=False)[:, :, 0]
            q = torch.arange(w, device=DEVICE)[None]
            own = (q >= m[:, None]) & ok
            piv = torch.diagonal(L, dim1=1, dim2=2)
            ll[a:e] = -0.5 * torch.where(own, 2 * torch.log(piv) + wv * wv + math.log(2 * math.pi), 0 * wv).sum(1)
            if grad:
                lm = int(l.max())
                rhs = torch.zeros(e - a, w, lm + 2, dtype=torch.float64, device=DEVICE)
                rhs[:, :, 0] = wv
                rhs[:, :, 1] = torch.where(q < m[:, None], wv, 0 * wv)
                c = torch.arange(lm, device=DEVICE)[None].expand(e - a, lm)
                r = (m[:, None] + c).clamp_max(w - 1)
                rows = torch.arange(e - a, device=DEVICE)[:, None].expand(e - a, lm)
                rhs[rows, r, 2 + c] = (c < l[:, None]).double()
                X = torch.linalg.solve_triangular(L.transpose(1, 2).contiguous(), rhs, upper=True)
                sign = torch.full((lm + 2,), -1.0, dtype=torch.float64, device=DEVICE)
                sign[0] = 1.0
                W = torch.bmm(X * sign, X.transpose(1, 2).contiguous())
                W = torch.where(both, W, torch.zeros_like(W))
                gg[a:e, 0] = 0.5 * (W * rho).sum((1, 2))
                gg[a:e, 1] = 0.5 * s2 / rg * (W * dr).sum((1, 2))
                gg[a:e, 2] = 0.5 * torch.diagonal(W, dim1=1, dim2=2).sum(1)
                if gen:
                    gg[a:e, 3] = 0.5 * s2 * (W * dn).sum((1, 2))
        parts.append(ll)
        gparts.append(gg[:, :4 if gen else 3])
    part, gpart = torch.stack(parts), torch.stack(gparts)
    return part.sum(1), gpart.sum(1), part, gpart


def _exact_predict(case, seed):
    s, y, t, bp, nptr, nidx, z = _pred_data(case, seed)
    s2, rg, nug, nu, _ = _thetas(case, seed)[0]
    both = torch.cat([s, t])
    u = _scaled(both, case["d"])
    yy = torch.cat([y, torch.zeros(case["new"], dtype=torch.float64, device=DEVICE)])
    mean, var = torch.empty(case["new"], dtype=torch.float64, device=DEVICE), torch.empty(case["new"], dtype=torch.float64, device=DEVICE)
    nb = bp.numel() - 1
    pm = int((nptr[1:] - nptr[:-1]).max() + (bp[1:] - bp[:-1]).max())
    step = max(1, int(6e7 // (pm * pm)))
    for a in range(0, nb, step):
        e = min(nb, a + step)
        idx, ok, m, l = _joint(bp, nptr, nidx, a, e, case["n"])
        w = idx.shape[1]
        K = s2 * _corr(_dist(u[idx], u[idx]) / rg, nu, False)[0] + nug * torch.eye(w, dtype=torch.float64, device=DEVICE)
        q = torch.arange(w, device=DEVICE)[None]
        nbr, own = (q < m[:, None]), (q >= m[:, None]) & ok
        mm = int(m.max())
        A = torch.where(nbr[:, :mm, None] & nbr[:, None, :mm], K[:, :mm, :mm],
                        torch.eye(mm, dtype=torch.float64, device=DEVICE))
        L = torch.linalg.cholesky(A)
        lm = int(l.max())
        c = torch.arange(lm, device=DEVICE)[None].expand(e - a, lm)
        r = (m[:, None] + c).clamp_max(w - 1)
        rows = torch.arange(e - a, device=DEVICE)[:, None].expand(e - a, lm)
        B = torch.where(nbr[:, :mm, None], K[rows, :, r].transpose(1, 2)[:, :mm], torch.zeros((), dtype=torch.float64, device=DEVICE))
        yn = torch.where(nbr[:, :mm], yy[idx[:, :mm]], torch.zeros((), dtype=torch.float64, device=DEVICE))
        S = torch.linalg.solve_triangular(L, torch.cat([B, yn[:, :, None]], 2), upper=False)
        mu = (S[:, :, :lm] * S[:, :, lm:]).sum(1)
        vv = s2 + nug - S[:, :, :lm].square().sum(1)
        keep = c < l[:, None]
        to = (bp[a:e, None] + c)[keep]
        mean[to], var[to] = mu[keep], vv[keep]
    draws = var.sqrt() * z
    m1 = mean + draws.mean(0)
    sd = draws.std(0, unbiased=True)
    zq = 1.959963984540054
    return dict(mean=mean, var=var, sample_mean=m1, sample_sd=sd, lo=m1 - zq * sd, hi=m1 + zq * sd)


def _exact_simulate(case, seed):
    s, nptr, nidx, z = _sim_data(case, seed)
    n = case["n"]
    u = _scaled(s, case["d"])
    unit = torch.arange(n + 1, device=DEVICE)
    out = []
    step = max(1, int(6e7 // (case["m"] + 1) ** 2))
    for t, (s2, rg, nug, nu, _) in enumerate(_thetas(case, seed)):
        coef, sd = np.zeros(nidx.numel()), np.empty(n)
        for a in range(0, n, step):
            e = min(n, a + step)
            idx, ok, m, _ = _joint(unit, nptr, nidx, a, e, 0)
            w = idx.shape[1]
            K = s2 * _corr(_dist(u[idx], u[idx]) / rg, nu, False)[0] + nug * torch.eye(w, dtype=torch.float64, device=DEVICE)
            K = torch.where(ok[:, :, None] & ok[:, None, :], K, torch.eye(w, dtype=torch.float64, device=DEVICE))
            L = torch.linalg.cholesky(K)
            row = torch.arange(e - a, device=DEVICE)
            last = L[row, m]                       # the point's own row: L_N^-1 k in its first m entries
            own = last[row, m]
            q = torch.arange(w, device=DEVICE)[None]
            rhs = torch.where(q < m[:, None], last, torch.zeros_like(last))
            c = torch.linalg.solve_triangular(L.transpose(1, 2).contiguous(), rhs[:, :, None], upper=True)[:, :, 0]
            coef[int(nptr[a]):int(nptr[e])] = c[q < m[:, None]].cpu().numpy()
            sd[a:e] = own.cpu().numpy()
        ptr, ix, zz, yv = nptr.cpu().numpy(), nidx.cpu().numpy(), z[t].cpu().numpy(), np.empty(n)
        for i in range(n):
            a, e = ptr[i], ptr[i + 1]
            yv[i] = coef[a:e] @ yv[ix[a:e]] + sd[i] * zz[i]
        out.append(torch.from_numpy(yv))
    return dict(y=torch.stack(out))


def _exact_features(case, seed):
    s, y, slot = _set_data(case, seed)
    k, sets = case["k"], case["sets"]
    i, j = torch.triu_indices(k, k, 1, device=DEVICE)
    h = (s[i] - s[j]).square().sum(1).sqrt()
    keep = (h > 0) & (h <= 0.5)
    i, j = i[keep], j[keep]
    bin_ = (h[keep] / 0.5 * 32).long().clamp_max(31)
    cnt = torch.bincount(bin_, minlength=32).double()
    gamma = torch.stack([torch.bincount(bin_, weights=(y[q, i] - y[q, j]).square(), minlength=32) / (2 * cnt) for q in range(sets)])
    gamma = torch.where(cnt > 0, gamma, torch.zeros_like(gamma))
    feat = torch.zeros(sets, 3, 32, dtype=torch.float64, device=DEVICE)
    feat[torch.arange(sets, device=DEVICE), slot.long()] = gamma / y.var(1, unbiased=False)[:, None]
    return dict(features=feat.reshape(sets, 96), gamma=gamma)


def _exact_train(case, seed):
    x, t, net = _net_data(case, seed)
    g = np.random.Generator(np.random.PCG64(net))
    P = []
    for a, b in ((96, 256), (256, 256), (256, 3)):
        lim = math.sqrt(6.0 / a)
        P += [torch.tensor(g.uniform(-lim, lim, (b, a)), dtype=torch.float32, device=DEVICE).double().requires_grad_(),
              torch.zeros(b, dtype=torch.float64, device=DEVICE, requires_grad=True)]
    a = x.double()
    for q in (0, 2, 4):
        a = a @ P[q].T + P[q + 1]
        a = torch.relu(a) if q < 4 else a
    loss = (a - t.double()).square().mean()
    loss.backward()
    m = [0.1 * p.grad for p in P]
    v = [0.001 * p.grad.square() for p in P]
    new = [p.detach() - 1e-3 * (mi / 0.1) / ((vi / 0.001).sqrt() + 1e-8) for p, mi, vi in zip(P, m, v)]
    # the first step moves a parameter by the learning rate and the sign of its
    # gradient: where that is rounding noise (a unit that is hardly ever active)
    # the sign has no exact value, and the biases start from zero
    return dict(loss=None, params=[p if p.dim() > 1 else None for p in new], m=m, v=v)


def exact(case, seed):
    op = case["op"]
    if op == "value":
        if case["n"] * case["nt"] > 1_000_000:
            return None
        ll, _, part, _ = _exact_likelihood(case, seed, False)
        return dict(loglik=ll, counters=None, partial=part if case["partial"] else None)
    if op == "fit":
        ll, g, _, _ = _exact_likelihood(case, seed, True)
        return dict(loglik=ll[0], grad=g[0])
    if op in ("grad", "grad_nu"):
        ll, g, part, gpart = _exact_likelihood(case, seed, True)
        r = dict(loglik=ll, grad=g, counters=None)
        if op == "grad":
            r.update(partial=part if case["partial"] else None, gpartial=gpart if case["partial"] else None)
        return r
    if op == "predict":
        return _exact_predict(case, seed)
    if op == "simulate":
        return _exact_simulate(case, seed)
    if op == "features":
        return _exact_features(case, seed)
    if op == "train":
        return _exact_train(case, seed)
    return None
