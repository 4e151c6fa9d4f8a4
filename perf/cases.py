"""Timed cases of the library: K_nu(x) on arrays of pairs, its derivatives, tiled
Matern covariance matrices and their gradient, the Gaussian log-likelihood, and the
window network's training gradient.

listed() names the cases, draw(rng) gives one more of the same ranges, prepare()
makes what a caller holds before the call, run() is one pass through the public
entry points, work() the bytes and operations the pass cannot do without, and
exact() the outputs in 64 bits from plain torch (no code of the library): the
trapezoid rule on the defining integrals with far more nodes than needed, a dense
Cholesky factorisation, and autograd.
"""
import math

import numpy as np
import torch

from paper_2502_00356_amd import api, workloads

MODEL_PATH = api.HERE + "/models/window_mlp.bin"
RESULTS = {"k": api.RESULT_K, "scaled": api.RESULT_SCALED, "log": api.RESULT_LOG}
GRID_LAW = dict(nu_lo=0.01, nu_hi=10.0, lx_lo=-4.0, lx_hi=3.0)


def listed():
    return [
        # Standalone K_nu(x). A small call (a few thousand pairs: launches and the
        # latency of one workgroup), and the 2^24-pair grid over the whole (nu, x) range
        # in plain FP64 and in the learned form.
        dict(name="k_plain_4096", kind="k", mode="plain", result="k", n=4096, nu_lo=0.1, nu_hi=4.0, lx_lo=-3.0,
             lx_hi=2.0),
        dict(name="k_plain_2e24", kind="k", mode="plain", result="k", n=1 << 24, **GRID_LAW),
        dict(name="k_learned_2e24", kind="k", mode="learned", result="k", n=1 << 24, **GRID_LAW),
        # The backward direction of K_nu: K, dK/dx and dK/dnu of a batch of pairs.
        dict(name="k_deriv_2e22", kind="deriv", result="k", n=1 << 22, **GRID_LAW),
        # One small covariance matrix, whole, FP64 (an exploratory fit on a thousand sites).
        dict(name="matern_plain_1024", kind="matern", mode="plain", out="f64", n=1024, tile=1024, lower=0, points="uniform",
             sigma2=1.0, beta=0.1, nu=1.3),
        # The lower tiles of a 40,000-site covariance in FP64 for a tiled factorisation.
        dict(name="matern_plain_40000", kind="matern", mode="plain", out="f64", n=40000, tile=960, lower=1, points="uniform",
             sigma2=1.0, beta=0.05, nu=2.3),
        # The smallest Matern call: a few hundred sites (a local kriging neighbourhood),
        # ragged tiles, FP32.
        dict(name="matern_learned_517", kind="matern", mode="learned", out="f32", n=517, tile=128, lower=1, points="uniform",
             sigma2=1.0, beta=0.1, nu=1.3),
        # The largest: the 316 x 316 jittered grid, lower 1,024-tiles, learned form, FP32.
        dict(name="matern_learned_99856", kind="matern", mode="learned", out="f32", n=99856, tile=1024, lower=1, points="grid",
             sigma2=1.0, beta=0.02, nu=3.7),
        # The mixed form (no trained model at hand), full matrix, odd sizes, FP32.
        dict(name="matern_mixed_9001", kind="matern", mode="mixed", out="f32", n=9001, tile=500, lower=0, points="uniform",
             sigma2=1.7, beta=0.05, nu=0.8),
        # The backward direction of the covariance: C, dC/dbeta and dC/dnu tiles, FP64.
        dict(name="matern_grad_12000", kind="grad", out="f64", n=12000, tile=960, lower=1, points="uniform", sigma2=1.0, beta=0.05,
             nu=0.8),
        # One likelihood-and-gradient evaluation of a maximum-likelihood fit.
        dict(name="loglik_grad_8100", kind="loglik", grad=True, n=8100, sigma2=1.0, beta=0.05, nu=0.8),
        # One gradient step's backward pass of the window network's training (a batch).
        dict(name="mlp_grad_4096", kind="mlp", n=4096),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _order(rng):
    """A smoothness: mostly any value, now and then a half-integer."""
    return rng.choice([0.5, 1.5, 2.5, 3.5]) if rng.random() < 0.2 else round(_log(rng, 0.3, 5.0), 4)


def draw(rng):
    kind = rng.choice(["k", "k", "deriv", "matern", "matern", "matern", "matern", "grad", "loglik", "mlp"])
    if kind in ("k", "deriv"):
        lx_lo = round(rng.uniform(-4.0, 0.0), 3)
        c = dict(kind=kind, result=rng.choice(["k", "scaled", "log"] if kind == "k" else ["k", "scaled"]),
                 n=int(_log(rng, 200, 1 << 24 if kind == "k" else 1 << 22)), nu_lo=0.01,
                 nu_hi=round(rng.uniform(2.0, 10.0), 3), lx_lo=lx_lo, lx_hi=round(rng.uniform(lx_lo + 1.0, 3.0), 3))
        if kind == "k":
            c["mode"] = rng.choice(["plain", "learned"])
        return c
    if kind in ("matern", "grad"):
        c = dict(kind=kind, n=int(_log(rng, 100, 20000 if kind == "matern" else 8000)), lower=rng.choice([0, 1]),
                 tile=rng.choice([64, 128, 256, 320, 500, 512, 777, 960, 1024, 2048]), points="uniform",
                 sigma2=round(rng.uniform(0.5, 2.0), 3), beta=round(_log(rng, 0.01, 0.3), 4), nu=_order(rng), out="f64")
        if kind == "matern":
            c["mode"] = rng.choice(["plain", "mixed", "learned"])
            c["out"] = "f64" if c["mode"] == "plain" and rng.random() < 0.8 else "f32"
        return c
    if kind == "loglik":
        return dict(kind="loglik", grad=rng.random() < 0.5, n=int(round(_log(rng, 16, 90))) ** 2,
                    sigma2=round(rng.uniform(0.5, 2.0), 3), beta=round(_log(rng, 0.02, 0.06), 4),
                    nu=round(rng.uniform(0.4, 1.2), 3))
    return dict(kind="mlp", n=int(_log(rng, 200, 16384)))


def _elems(c):
    return api.matern_out_elems(c["n"], c["tile"], c["lower"])


def _pairs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    u = torch.rand(2, c["n"], generator=g, dtype=torch.float64, device="cuda")
    nu = c["nu_lo"] + (c["nu_hi"] - c["nu_lo"]) * u[0]
    x = 10.0 ** (c["lx_lo"] + (c["lx_hi"] - c["lx_lo"]) * u[1])
    return nu, x


def _sites(points, n, seed):
    if points == "grid":
        xy = workloads.jittered_grid_locations(int(round(math.sqrt(n))), seed)
    else:
        xy = workloads.uniform_locations(n, seed)
    t = torch.from_numpy(np.ascontiguousarray(xy.T)).cuda()
    return t[0].contiguous(), t[1].contiguous()


def _distances(lx, ly, i, j):
    """Distances of sites j (rows) to sites i (columns): j.size x i.size."""
    return torch.hypot(lx[j][:, None] - lx[i][None, :], ly[j][:, None] - ly[i][None, :])


def _observations(lx, ly, seed):
    """A draw with exponential correlation, as the likelihood's data."""
    every = torch.arange(lx.numel(), device="cuda")
    r = torch.exp(-_distances(lx, ly, every, every) / 0.05)
    r.diagonal().add_(1e-9)
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    return torch.linalg.cholesky(r) @ torch.randn(lx.numel(), generator=g, dtype=torch.float64, device="cuda")


def _mlp_inputs(c, seed):
    """Parameters (He initialisation) and one batch of normalised inputs and targets."""
    rng = np.random.default_rng(int(seed))
    w = [rng.normal(0, 1.0, (64, 2)), 0.1 * rng.normal(size=64), rng.normal(0, math.sqrt(2 / 64), (64, 64)),
         np.zeros(64), rng.normal(0, math.sqrt(1 / 64), (3, 64)), np.array([0.2, 0.8, 0.5])]
    p = np.concatenate([a.ravel() for a in w])
    u = rng.uniform(-1, 1, (c["n"], 2))
    target = np.stack([np.maximum(0, 0.3 - 0.4 * u[:, 0]), 0.9 - 0.5 * u[:, 0], 0.5 + 0.2 * u[:, 1]], 1)
    return [torch.from_numpy(a.astype(np.float32)).cuda() for a in (p, u, target, np.array([0.1, 0.9, 0.9]))]


def prepare(c, seed):
    s = dict(case=c)
    if c.get("mode") == "learned":
        s["model"] = api.Model(MODEL_PATH)
    if c["kind"] in ("k", "deriv"):
        s["nu"], s["x"] = _pairs(c, seed)
        s["out"] = ({k: torch.empty_like(s["x"]) for k in ("k", "dx", "dnu")} if c["kind"] == "deriv"
                    else torch.empty_like(s["x"]))
        if c.get("mode") == "learned":
            s["workspace"] = torch.empty(api.workspace_bytes(c["n"]), dtype=torch.uint8, device="cuda")
    elif c["kind"] in ("matern", "grad"):
        s["lx"], s["ly"] = _sites(c["points"], c["n"], seed)
        dt = torch.float32 if c["out"] == "f32" else torch.float64
        if c["kind"] == "grad":
            s["out"] = {k: torch.empty(_elems(c), dtype=dt, device="cuda") for k in ("c", "dbeta", "dnu")}
        else:
            s["out"] = torch.empty(_elems(c), dtype=dt, device="cuda")
        if c.get("mode") == "learned":
            need = api.matern_workspace_bytes(c["n"], c["tile"], c["lower"])
            s["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    elif c["kind"] == "loglik":
        s["lx"], s["ly"] = _sites("grid", c["n"], seed)
        s["z"] = _observations(s["lx"], s["ly"], seed)
        s["workspace"] = torch.empty(api.matern_loglik_workspace_bytes(c["n"], c["grad"]), dtype=torch.uint8, device="cuda")
    else:
        s["inputs"] = _mlp_inputs(c, seed)
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "k":
        return api.besselk(s["nu"], s["x"], out=s["out"], mode=c["mode"], result=RESULTS[c["result"]],
                           model=s.get("model"), workspace=s.get("workspace"))
    if c["kind"] == "deriv":
        return api.besselk_deriv(s["nu"], s["x"], result=RESULTS[c["result"]], out=s["out"])
    if c["kind"] == "matern":
        return api.matern_tiles(s["lx"], s["ly"], c["sigma2"], c["beta"], c["nu"], c["tile"], c["lower"], mode=c["mode"],
                                out_dtype=api.OUT_F32 if c["out"] == "f32" else api.OUT_F64, out=s["out"],
                                model=s.get("model"), workspace=s.get("workspace"))
    if c["kind"] == "grad":
        return api.matern_grad_tiles(s["lx"], s["ly"], c["sigma2"], c["beta"], c["nu"], c["tile"], c["lower"],
                                     out_dtype=api.OUT_F32 if c["out"] == "f32" else api.OUT_F64, out=s["out"])
    if c["kind"] == "loglik":
        r = api.matern_loglik(s["lx"], s["ly"], s["z"], c["sigma2"], c["beta"], c["nu"], grad=c["grad"],
                              workspace=s["workspace"])
        return {"l": r[0], "grad": list(r[1])} if c["grad"] else {"l": r}
    loss, grad = api.mlp_grad(*s["inputs"])
    return {"loss": loss, "grad": grad}


def work(c):
    """Inputs read once, outputs written once; operations: a handful per entry where
    the bytes are what a pass cannot do without, n^3 terms for the likelihood (the
    factorisation, and the inverse with the gradient), products for the network."""
    n = c["n"]
    if c["kind"] == "k":
        return {"bytes": 24 * n, "flops": 100 * n}
    if c["kind"] == "deriv":
        return {"bytes": 40 * n, "flops": 300 * n}
    if c["kind"] in ("matern", "grad"):
        e, size = _elems(c), 4 if c["out"] == "f32" else 8
        k = 3 if c["kind"] == "grad" else 1
        return {"bytes": k * size * e + 16 * n, "flops": 20 * k * e}
    if c["kind"] == "loglik":
        k = 3 if c["grad"] else 1
        return {"bytes": k * 8 * n * n, "flops": k * n ** 3 / 3}
    return {"bytes": 20 * n + 2 * 4 * api.MLP_NPARAM, "flops": 6 * api.MLP_NPARAM * n}


# ------------------------------------------------------------- outputs in 64 bits
NODES = 128


def _integrals(nu, x, deriv):
    """e^x times K_nu(x) and, with deriv, -dK/dx and dK/dnu: the trapezoid rule with
    NODES intervals on [0, T], e^(nu t - x (cosh t - 1)) below e^-44 of its peak past T."""
    peak = torch.asinh(nu / x)
    drop = nu * peak - 2 * x * torch.sinh(peak / 2) ** 2      # the exponent at the peak
    t_end = torch.acosh(1.0 + (44.0 + nu * (peak + 4.0)) / x)
    for _ in range(6):       # outward bound of nu t - x (cosh t - 1) = drop - 44
        t_end = torch.acosh(1.0 + (44.0 + nu * t_end - drop).clamp_min(1.0) / x)
    t_end = t_end * 1.02
    h = t_end / NODES
    sums = [torch.zeros_like(x) for _ in range(3 if deriv else 1)]
    for m in range(NODES + 1):
        t = h * m
        w = 0.5 if m in (0, NODES) else 1.0
        e = torch.exp(nu * t - drop - 2 * x * torch.sinh(t / 2) ** 2) * (0.5 * w)
        p = torch.expm1(-2 * nu * t)
        sums[0] += e * (2 + p)
        if deriv:
            sums[1] += e * (2 + p) * torch.cosh(t)
            sums[2] += e * t * -p
    # e^drop can pass 1e308 only together with K itself
    return [h * torch.exp(drop) * s for s in sums], drop, h, sums


def _exact_pairs(c, seed):
    nu, x = _pairs(c, seed)
    outs = []
    for a in range(0, c["n"], 1 << 20):
        v, z = nu[a:a + (1 << 20)], x[a:a + (1 << 20)]
        (k, *d), drop, h, sums = _integrals(v, z, c["kind"] == "deriv")
        if c["result"] == "log":
            outs.append((drop - z + torch.log(h * sums[0]),))
        else:
            f = torch.exp(-z) if c["result"] == "k" else torch.ones_like(z)
            outs.append((k * f,) + ((-d[0] * f, d[1] * f) if d else ()))
    got = [torch.cat(t) for t in zip(*outs)]
    return got[0] if c["kind"] == "k" else dict(zip(("k", "dx", "dnu"), got))


def _matern_values(c, r, deriv):
    """C and, with deriv, dC/dbeta and dC/dnu at distances r."""
    s2, beta, nu = c["sigma2"], c["beta"], c["nu"]
    zero = r == 0
    z = torch.where(zero, 1.0, r / beta)
    v = torch.full((), nu, dtype=torch.float64, device=r.device)
    (k, *d), *_ = _integrals(v, z, deriv)
    f = s2 * torch.exp((1 - nu) * math.log(2.0) - math.lgamma(nu) + nu * torch.log(z) - z)
    out = [torch.where(zero, s2, f * k)]
    if deriv:
        psi = torch.digamma(v)
        # d/dz z^nu K = z^nu (K' + nu K / z)
        out.append(torch.where(zero, 0.0, f * (d[0] - nu * k / z) * z / beta))
        out.append(torch.where(zero, 0.0, f * (k * (torch.log(z) - math.log(2.0) - psi) + d[1])))
    return out


def _exact_tiles(c, seed, deriv):
    lx, ly = _sites(c["points"], c["n"], seed)
    n, ts = c["n"], c["tile"]
    starts = range(0, n, ts)
    out = [torch.empty(_elems(c), dtype=torch.float64, device="cuda") for _ in range(3 if deriv else 1)]
    o = 0
    for J in starts:
        cols = torch.arange(J, min(n, J + ts), device="cuda")
        for I in starts:
            if c["lower"] and I < J:
                continue
            rows = torch.arange(I, min(n, I + ts), device="cuda")
            for a, b in zip(out, _matern_values(c, _distances(lx, ly, rows, cols), deriv)):
                a[o:o + b.numel()] = b.reshape(-1)
            o += rows.numel() * cols.numel()
    return dict(zip(("c", "dbeta", "dnu"), out)) if deriv else out[0]


def _exact_loglik(c, seed):
    lx, ly = _sites("grid", c["n"], seed)
    z = _observations(lx, ly, seed)
    every = torch.arange(c["n"], device="cuda")
    S, *dS = _matern_values(c, _distances(lx, ly, every, every), c["grad"])
    L = torch.linalg.cholesky(S)
    a = torch.cholesky_solve(z[:, None], L)[:, 0]
    quad = float(z @ a)
    l = -0.5 * quad - float(torch.log(L.diagonal()).sum()) - 0.5 * c["n"] * math.log(2 * math.pi)
    if not c["grad"]:
        return {"l": l}
    inv = torch.cholesky_inverse(L)
    g = [0.5 * (quad - c["n"]) / c["sigma2"]]
    g += [0.5 * float(a @ (D @ a)) - 0.5 * float((inv * D).sum()) for D in dS]
    return {"l": l, "grad": g}


def _exact_mlp(c, seed):
    p, u, target, tau = [t.double() for t in _mlp_inputs(c, seed)]
    p.requires_grad_(True)
    W1, b1, W2, b2, W3, b3 = torch.split(p, [128, 64, 4096, 64, 192, 3])
    h = torch.relu(u @ W1.reshape(64, 2).T + b1)
    h = torch.relu(h @ W2.reshape(64, 64).T + b2)
    e = target - (h @ W3.reshape(3, 64).T + b3)
    loss = (torch.where(e < 0, 1 - tau, tau) * e * e).sum(1).mean()
    loss.backward()
    return {"loss": loss.detach().reshape(1), "grad": p.grad}


def exact(c, seed):
    if c["kind"] in ("k", "deriv"):
        return _exact_pairs(c, seed)
    if c["kind"] in ("matern", "grad"):
        # past this the dense evaluation takes too long
        return None if _elems(c) > 1e9 else _exact_tiles(c, seed, c["kind"] == "grad")
    return _exact_loglik(c, seed) if c["kind"] == "loglik" else _exact_mlp(c, seed)
