"""The work that users of the library have it do, as timed cases.

Every case is one call of a public entry point of ``Context`` on a field of n
locations: one likelihood, one likelihood with its score, a simulated field,
kriging, the Fisher information, or a capped maximisation.  The sizes are those
of the library's own studies: 400 (20 x 20 grid) and 1,600 points, 10,000 (100
x 100, tile 512) and 40,000 (the headline workload and the 200 x 200 grid),
with odd sizes between them.

``listed()`` names twelve cases, ``draw(rng)`` gives another one of the same
ranges, ``prepare`` makes what a program holds before the call (locations,
observations, a context), ``run`` is the call, ``exact`` the same numbers from
dense 64-bit torch on the GPU.

Locations are the jittered grid of ``inputgen`` (n of its points at random
where n is no square), uniform points, or a patch of the sphere in degrees.
Observations are a zero-mean field with the case's own Matern spectrum (a sum
of plane waves with random frequencies), so that z^T Sigma^-1 z is near n.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1908_06936_amd as exa

DEV = "cuda"
WAVES = 384


def _case(name, op, n, ts=768, layout="grid", theta=(1.0, 0.1, 0.5), precision="fp64", **more):
    c = {"name": name, "op": op, "n": n, "ts": ts, "layout": layout, "s2": theta[0], "beta": theta[1],
         "nu": theta[2], "precision": precision, "nugget": 0.0, "band": 0, "m": 0, "mse": False, "evals": 0}
    c.update(more)
    return c


def listed():
    return [
        # one likelihood of the paper's own example size (20 x 20 grid): a script's inner call
        _case("loglik_400", "loglik", 400),
        # the derivative-free estimate of that example, whole call, capped as the paper caps its timings
        _case("mle_400", "mle", 400, evals=60),
        # a gradient step on the paper's n = 1,600 field
        _case("grad_1600", "grad", 1600, theta=(1.0, 0.1, 1.0)),
        # geostatistics on the sphere: great-circle distances, noisy observations, an odd size
        _case("grad_sphere_2501", "grad", 2501, ts=512, layout="sphere", theta=(1.5, 150.0, 0.8), nugget=0.05),
        # the n = 10,000 study (100 x 100 grid, tile 512)
        _case("loglik_10000", "loglik", 10000, ts=512, theta=(1.0, 0.1, 1.0)),
        # a gradient step of an ordinary estimation, n a prime, scattered stations
        _case("grad_9973", "grad", 9973, layout="uniform"),
        # kriging with variances at 1,000 new points
        _case("predict_10000", "predict", 10000, theta=(1.0, 0.1, 0.8), m=1000, mse=True),
        # standard errors of an estimate
        _case("fisher_6400", "fisher", 6400, ts=512, theta=(1.0, 0.08, 0.5)),
        # one simulated field (150 x 150 grid)
        _case("simulate_22500", "simulate", 22500, theta=(1.0, 0.1, 1.0)),
        # the diagonal-super-tile approximation at full size
        _case("dst_40000", "loglik", 40000, theta=(1.0, 0.005, 0.5), band=4),
        # a mixed-precision gradient step at full size
        _case("mixed_grad_40000", "grad", 40000, theta=(1.0, 0.03, 0.5), precision="mixed"),
        # the headline workload: one FP64 (l, grad l) at n = 40,000
        _case("grad_40000", "grad", 40000, layout="uniform", theta=(1.0, 0.1, 1.0)),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["loglik", "loglik", "grad", "grad", "mixed_loglik", "mixed_grad", "sphere", "dst", "predict",
                     "simulate", "fisher", "mle"])
    ts = rng.choice([256, 512, 768])
    layout = rng.choice(["grid", "grid", "uniform"])
    beta = round(math.exp(rng.uniform(math.log(0.02), math.log(0.12))), 4)
    # uniform points hold close pairs: rough fields only
    nu = 0.5 if layout == "uniform" else rng.choice([0.5, 0.8, 1.0])
    th = (round(rng.uniform(0.5, 2.0), 3), beta, nu)
    if op in ("loglik", "grad"):
        n = _size(rng, 300, 40000)
        if n > 12000:
            ts = rng.choice([512, 768])
        return _case("", op, n, ts=ts, layout=layout, theta=th, nugget=rng.choice([0.0, 0.0, 0.02]))
    if op in ("mixed_loglik", "mixed_grad"):
        return _case("", op[6:], _size(rng, 10000, 40000), ts=rng.choice([512, 768]), theta=(th[0], min(beta, 0.04), 0.5),
                     precision="mixed")
    if op == "sphere":
        return _case("", rng.choice(["loglik", "grad"]), _size(rng, 400, 10000), ts=ts, layout="sphere",
                     theta=(th[0], round(rng.uniform(60.0, 200.0), 1), rng.choice([0.5, 0.8])), nugget=0.05)
    if op == "dst":
        return _case("", "loglik", _size(rng, 5000, 40000), ts=rng.choice([512, 768]), theta=(th[0], 0.005, 0.5),
                     band=rng.choice([2, 4, 8]))
    if op == "predict":
        return _case("", "predict", _size(rng, 400, 20000), ts=ts, layout=layout, theta=th, m=_size(rng, 1, 2000),
                     mse=rng.choice([True, False]))
    if op == "simulate":
        return _case("", "simulate", _size(rng, 400, 30000), ts=rng.choice([512, 768]), layout=layout, theta=th)
    if op == "fisher":
        return _case("", "fisher", _size(rng, 300, 12000), ts=ts, layout=layout, theta=th)
    return _case("", "mle", _size(rng, 250, 1600), ts=ts, evals=rng.choice([20, 40, 60]))


# ------------------------------------------------------------------ inputs
def _locations(n, layout, rng):
    if layout == "sphere":  # a 20 x 20 degree patch, stations on a jittered grid
        x, y = _locations(n, "grid", rng)
        return -60.0 + 20.0 * x, 30.0 + 20.0 * y
    if layout == "uniform":
        return rng.random(n), rng.random(n)
    m = math.isqrt(n - 1) + 1
    c = (np.arange(m) + 0.5) / m
    gx, gy = np.meshgrid(c, c, indexing="ij")
    x = gx.ravel() + rng.uniform(-0.4, 0.4, m * m) / m
    y = gy.ravel() + rng.uniform(-0.4, 0.4, m * m) / m
    if n < m * m:
        keep = np.sort(rng.permutation(m * m)[:n])
        x, y = x[keep], y[keep]
    return x, y


def _inputs(case, seed):
    """x, y, z, new locations and normal draws, float64 on the host, from the seed alone."""
    rng = np.random.default_rng([seed, case["n"]])
    n, m = case["n"], case["m"]
    x, y = _locations(n, case["layout"], rng)
    box = (x.min(), x.max(), y.min(), y.max())
    xn, yn = rng.uniform(box[0], box[1], m), rng.uniform(box[2], box[3], m)
    # plane waves with frequencies of the Matern spectrum (a bivariate t)
    px, py, beta = x, y, case["beta"]
    if case["layout"] == "sphere":  # local kilometres
        k = 6371.0 * math.pi / 180.0
        px, py = (x + 50.0) * k * math.cos(math.radians(40.0)), (y - 40.0) * k
    g = rng.gamma(case["nu"], 1.0, WAVES)
    w = rng.standard_normal((2, WAVES)) / (beta * np.sqrt(2.0 * g))
    ph = rng.uniform(0.0, 2.0 * math.pi, WAVES)
    P = torch.as_tensor(np.stack([px, py], 1), device=DEV)
    W = torch.as_tensor(w, device=DEV)
    z = torch.zeros(n, dtype=torch.float64, device=DEV)
    for a in range(0, n, 8192):
        z[a:a + 8192] = torch.cos(P[a:a + 8192, :1] * W[0] + P[a:a + 8192, 1:] * W[1]
                                  + torch.as_tensor(ph, device=DEV)).sum(1)
    z = z * math.sqrt(2.0 * case["s2"] / WAVES)
    if case["nugget"]:
        z = z + math.sqrt(case["nugget"]) * torch.as_tensor(rng.standard_normal(n), device=DEV)
    e = rng.standard_normal(n)
    return [torch.as_tensor(np.ascontiguousarray(a), device=DEV) for a in (x, y)] + [z] + \
        [torch.as_tensor(np.ascontiguousarray(a), device=DEV) for a in (xn, yn, e)]


def prepare(case, seed):
    x, y, z, xn, yn, e = _inputs(case, seed)
    ctx = exa.Context(ts=case["ts"])
    if case["layout"] == "sphere":
        ctx.set_distance("great_circle")
    if case["nugget"]:
        ctx.set_nugget(case["nugget"])
    if case["band"]:
        ctx.set_dst_band(case["band"])
    return {"case": case, "ctx": ctx, "x": x, "y": y, "z": z, "xn": xn, "yn": yn, "e": e,
            "theta": (case["s2"], case["beta"], case["nu"])}


def run(s):
    c, ctx, x, y, z, th = s["case"], s["ctx"], s["x"], s["y"], s["z"], s["theta"]
    op = c["op"]
    if op == "loglik":
        return {"loglik": np.float64(ctx.loglik(x, y, z, th, c["precision"]))}
    if op == "grad":
        ll, g = ctx.loglik_grad(x, y, z, th, c["precision"])
        return {"loglik": np.float64(ll), "grad": np.asarray(g)}
    if op == "predict":
        mean, mse = ctx.predict(x, y, z, th, s["xn"], s["yn"], with_mse=c["mse"])
        return {"mean": mean, "mse": mse} if c["mse"] else {"mean": mean}
    if op == "simulate":
        return {"z": ctx.simulate(x, y, th, s["e"])}
    if op == "fisher":
        return {"fisher": ctx.fisher(x, y, th)}
    theta, ll, stats = ctx.mle(x, y, z, [0.01, 0.01, 0.1], [5.0, 2.0, 3.0], theta0=[0.5, 0.3, 0.5], tol=1e-4,
                               max_iters=c["evals"], method="dfo")
    return {"theta": np.asarray(theta), "loglik": np.float64(ll), "evals": stats["n_evals"]}


def work(case):
    """Inputs and outputs once, and the dense linear algebra of the exact path:
    n^3 / 3 for a factorisation, n^3 / 3 more each for the inverse factor and
    for Sigma^-1 in a score, n^2 per new point of a kriging variance, n^3 per
    parameter of the Fisher information, n w^2 for a band of w rows."""
    n, m = float(case["n"]), float(case["m"])
    op = case["op"]
    chol = n * n * n / 3.0
    if case["band"]:
        w = min(n, float(case["band"] * case["ts"]))
        chol = min(chol, n * w * w)
    by, fl = 24.0 * n + 8.0, chol + n * n
    if op == "grad":
        by, fl = by + 24.0, 3.0 * chol
    elif op == "predict":
        by, fl = by + 16.0 * m + 8.0 * m * (2 if case["mse"] else 1), fl + (n * n * m if case["mse"] else 2.0 * n * m)
    elif op == "simulate":
        by += 8.0 * n
    elif op == "fisher":
        by, fl = 16.0 * n + 72.0, 2.0 * chol + 2.0 * n * n * n
    elif op == "mle":
        fl *= case["evals"]
    return {"bytes": by, "flops": fl}


# ------------------------------------------- the same numbers, dense, 64 bits
def _bessel(x, nu, deriv):
    """(e^x K_nu, e^x K_{nu-1}, e^x dK_nu/dnu) by the trapezoidal rule on
    int exp(-x (cosh t - 1)) cosh(nu t) dt (and its derivatives), x > 0."""
    k0 = torch.zeros_like(x)
    k1 = torch.zeros_like(x) if deriv else None
    kd = torch.zeros_like(x) if deriv else None
    h = 1.0 / 32.0
    tmax = math.acosh(1.0 + 60.0 / max(float(x.min()), 1e-9)) + 1.0
    for k in range(int(tmax / h) + 2):
        t = k * h
        w = 0.5 * h if k == 0 else h
        f = torch.exp(x * -(2.0 * math.sinh(0.5 * t) ** 2))
        k0.add_(f, alpha=w * math.cosh(nu * t))
        if deriv:
            k1.add_(f, alpha=w * math.cosh((nu - 1.0) * t))
            kd.add_(f, alpha=w * t * math.sinh(nu * t))
    return k0, k1, kd


def _dist(xa, ya, xb, yb, sphere):
    if not sphere:
        return torch.sqrt((xa[:, None] - xb[None]) ** 2 + (ya[:, None] - yb[None]) ** 2)
    r = math.pi / 180.0
    sp, sl = torch.sin((ya[:, None] - yb[None]) * (r / 2)), torch.sin((xa[:, None] - xb[None]) * (r / 2))
    a = sp * sp + torch.cos(ya * r)[:, None] * torch.cos(yb * r)[None] * sl * sl
    a = a.clamp(0.0, 1.0)
    return 2.0 * 6371.0 * torch.atan2(torch.sqrt(a), torch.sqrt(1.0 - a))


def _cov(case, xa, ya, xb, yb, deriv=False, rows=2048):
    """Sigma between two sets of locations (and its derivatives in beta, nu)."""
    s2, beta, nu = case["s2"], case["beta"], case["nu"]
    c = 2.0 ** (1.0 - nu) / math.gamma(nu)
    psi = float(torch.digamma(torch.tensor(nu, dtype=torch.float64)))
    out = [torch.empty(len(xa), len(xb), dtype=torch.float64, device=DEV) for _ in range(3 if deriv else 1)]
    for a in range(0, len(xa), rows):
        d = _dist(xa[a:a + rows], ya[a:a + rows], xb, yb, case["layout"] == "sphere") / beta
        zero = d == 0
        x = torch.where(zero, torch.ones_like(d), d)
        ex = torch.exp(-x)
        if nu == 0.5 and not deriv:
            v = [s2 * ex]
        else:
            k0, k1, kd = _bessel(x, nu, deriv)
            xn = s2 * c * torch.pow(x, nu) * ex
            v = [xn * k0]
            if deriv:
                v += [xn * x * k1 / beta, v[0] * (-math.log(2.0) - psi + torch.log(x)) + xn * kd]
        for k, o in enumerate(out):
            o[a:a + rows] = torch.where(zero, torch.full_like(x, s2 if k == 0 else 0.0), v[k])
    return out


def _z_order(x, y):
    """The order in which the library factorises: 16-bit Z-order over the bounding box, ties by index."""
    x, y = x.cpu().numpy(), y.cpu().numpy()

    def bits(v):
        w = v.max() - v.min()
        q = ((v - v.min()) * (65535.999 / w if w > 0 else 0.0)).astype(np.uint64)
        s = np.zeros(v.size, dtype=np.uint64)
        for b in range(16):
            s |= ((q >> np.uint64(b)) & np.uint64(1)) << np.uint64(2 * b)
        return s

    code = bits(x) | (bits(y) << np.uint64(1))
    return torch.as_tensor(np.lexsort((np.arange(x.size), code)), device=DEV)


def exact(case, seed):
    op, n = case["op"], case["n"]
    # an optimiser's path has no value of its own; the rest by what dense torch does in a few seconds
    if op == "mle" or n > (12000 if op in ("grad", "fisher", "predict") else 30000) and case["nu"] != 0.5:
        return None
    x, y, z, xn, yn, e = _inputs(case, seed)
    ll_only = n > 12000
    if op == "fisher" and ll_only:
        return None
    order = _z_order(x, y)
    x, y, z = x[order], y[order], z[order]
    deriv = op in ("grad", "fisher") and not ll_only
    S = _cov(case, x, y, x, y, deriv)
    A = S[0]
    if case["nugget"]:
        A.diagonal().add_(case["nugget"])
    if case["band"]:
        t = torch.arange(n, device=DEV) // case["ts"]
        for a in range(0, n, 4096):
            A[a:a + 4096].masked_fill_((t[a:a + 4096, None] - t[None]).abs() >= case["band"], 0.0)
    if case["nugget"] and op == "fisher":
        return None
    L = torch.linalg.cholesky(A)
    if op == "simulate":
        out = torch.empty_like(z)
        out[order] = L @ e[order]
        return {"z": out}
    v = torch.linalg.solve_triangular(L, z[:, None], upper=False)
    ll = np.float64(-0.5 * (n * math.log(2.0 * math.pi) + 2.0 * torch.log(L.diagonal()).sum() + (v * v).sum()).item())
    if op == "loglik":
        return {"loglik": ll}
    if op == "grad" and ll_only:
        return {"loglik": ll, "grad": None}
    if op == "predict":
        C = _cov(case, x, y, xn, yn)[0]
        V = torch.linalg.solve_triangular(L, C, upper=False)
        out = {"mean": (V * v).sum(0)}
        if case["mse"]:
            out["mse"] = case["s2"] - (V * V).sum(0)
        return out
    if op == "grad":
        al = torch.linalg.solve_triangular(L.t(), v, upper=True)[:, 0]
        Si = torch.cholesky_inverse(L)
        if case["nugget"]:
            S[0].diagonal().sub_(case["nugget"])
        g = []
        for k, d in enumerate((S[0] / case["s2"], S[1], S[2])):
            g.append(float(0.5 * (al @ (d @ al)) - 0.5 * (Si * d).sum()))
        return {"loglik": ll, "grad": np.asarray(g)}
    A3 = [torch.cholesky_solve(d, L) for d in (S[1], S[2])]
    s2 = case["s2"]
    f = np.empty((3, 3))
    f[0, 0] = 0.5 * n / s2 ** 2
    for j in range(2):
        f[0, j + 1] = f[j + 1, 0] = 0.5 * float(A3[j].diagonal().sum()) / s2
        for k in range(2):
            f[j + 1, k + 1] = 0.5 * float((A3[j] * A3[k].t()).sum())
    return {"fisher": f}
