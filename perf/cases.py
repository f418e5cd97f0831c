"""Workloads of the likelihood library, through its public entry points.

What a user of this package has it do: evaluate the exact log-likelihood l(θ)
of measurements at n locations (once per optimiser step, so at every size from
a few hundred points to tens of thousands, eager or as a replayed graph, in
binary64 or in a mixed-precision mode), many such evaluations at once through
the request queue, the independent-blocks approximation on a large field,
kriging at new locations from a kept factor (with and without variances),
k-fold cross-validation, and covariance blocks between two point sets.

A case is a dict of plain values; `kind` names the entry point.  Locations are
a jittered grid in the unit square (or the same grid as longitude and latitude
over a 15 degree square for the great-circle distance).  Measurements are draws
of a Gaussian field with the Matérn covariance of the case, made by summing
random cosines whose frequencies follow the Matérn spectral density.
"""
import math

import numpy as np
import torch

import paper_1708_02835_amd as gl

_RADIUS = 6371.0  # great-circle distances in km
_LON0, _LAT0, _SPAN = -100.0, 30.0, 15.0
_KM = _SPAN * math.pi / 180.0 * _RADIUS  # side of the great-circle square, north-south


def listed():
    return [
        # one optimiser step on a station network of a few hundred points: latency and launches
        dict(name="eval_n400", kind="eval", n=400, t1=1.0, t2=0.1, t3=0.5, precision="fp64", metric=0, graph=0),
        # the smallest synthetic size of the paper's experiments
        dict(name="eval_n1600", kind="eval", n=1600, t1=1.0, t2=0.1, t3=0.5, precision="fp64", metric=0, graph=0),
        # maximum-likelihood estimation replays one size under changing θ: the replayed graph
        dict(name="eval_n8100_graph", kind="eval", n=8100, t1=1.2, t2=0.03, t3=1.5, precision="fp64", metric=0,
             graph=1),
        # geographic data: great-circle distance, general smoothness, a size no tile divides
        dict(name="eval_n15877_gcd", kind="eval", n=15877, t1=0.8, t2=0.05, t3=0.9, precision="fp64", metric=1,
             graph=0),
        # the largest binary64 size that is repeated often
        dict(name="eval_n40000", kind="eval", n=40000, t1=1.0, t2=0.1, t3=0.5, precision="fp64", metric=0, graph=0),
        # the headline field size in the mixed mode made for it
        dict(name="eval_n100000_fp16", kind="eval", n=100000, t1=1.0, t2=0.1, t3=0.5, precision="fp16", metric=0,
             graph=0),
        # independent-blocks approximation of a field too large to factor at every step
        dict(name="ind_n100000", kind="ind", n=100000, t1=1.0, t2=0.1, t3=0.5, tiles=4),
        # clients of the request queue, sizes as in the serving benchmark
        dict(name="queue_16", kind="queue", requests=16, n_lo=1000, n_hi=16000, field=3),
        # prediction maps: 1,000 held-out locations from a kept factor
        dict(name="krige_n40000_m1000", kind="krige", n=40000, m=1000, t1=1.0, t2=0.03, t3=1.5, var=0),
        # the same with the prediction variances
        dict(name="krige_var_n16000_m1000", kind="krige", n=16000, m=1000, t1=1.0, t2=0.1, t3=0.5, var=1),
        # 10-fold cross-validation of a medium field
        dict(name="cv_n4000_k10", kind="cv", n=4000, k=10, t1=1.0, t2=0.1, t3=0.5),
        # Σ12 between a field and held-out points, general smoothness
        dict(name="sigma12_40000x1000", kind="sigma12", n1=40000, n2=1000, t1=1.0, t2=0.1, t3=1.0, metric=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _theta(rng, n, metric=0):
    """θ of the serving benchmark's ranges, the range capped so that Σ stays well conditioned (and the
    smoothness on the sphere, where the smoother Matérn functions of the distance are no covariances)."""
    t3 = rng.choice([0.5, 0.5, 1.0, 1.5, 2.5, round(rng.uniform(0.4, 2.0), 3)])
    t3 = min(t3, 0.9) if metric else t3
    cap = {True: 25.0, False: 25.0 ** (3.0 / (2.0 * t3 + 2.0))}[t3 <= 0.5]
    t2 = round(min(rng.uniform(0.02, 0.15), max(0.004, cap / math.sqrt(n))), 5)
    return dict(t1=round(rng.uniform(0.5, 2.0), 4), t2=t2, t3=t3)


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "eval", "mixed", "ind", "queue", "krige", "krige", "cv", "sigma12"])
    if kind == "eval":
        n = _log_int(rng, 300, 30000)
        metric = 1 if rng.random() < 0.25 else 0
        graph = 1 if rng.random() < 0.25 else 0
        return dict(kind="eval", n=n, precision="fp64", metric=metric, graph=graph, **_theta(rng, n, metric))
    if kind == "mixed":
        n = _log_int(rng, 20000, 60000)
        return dict(kind="eval", n=n, t1=round(rng.uniform(0.5, 2.0), 4), t2=0.1, t3=0.5,
                    precision=rng.choice(["fp32", "bf16", "fp16"]), metric=0, graph=0)
    if kind == "ind":
        n = _log_int(rng, 10000, 100000)
        return dict(kind="ind", n=n, t1=1.0, t2=0.1, t3=0.5, tiles=rng.choice([1, 2, 4, 8]))
    if kind == "queue":
        hi = _log_int(rng, 2000, 16000)
        return dict(kind="queue", requests=rng.randint(4, 16), n_lo=max(300, hi // 16), n_hi=hi,
                    field=rng.randint(0, 1 << 20))
    if kind == "krige":
        n = _log_int(rng, 1000, 30000)
        return dict(kind="krige", n=n, m=_log_int(rng, 100, 3000), var=rng.randint(0, 1), **_theta(rng, n))
    if kind == "cv":
        n = _log_int(rng, 500, 5000)
        return dict(kind="cv", n=n, k=rng.choice([5, 10]), **_theta(rng, n))
    n1, n2 = _log_int(rng, 1000, 40000), _log_int(rng, 100, 1000)
    metric = rng.randint(0, 1)
    return dict(kind="sigma12", n1=n1, n2=n2, metric=metric, **_theta(rng, n1, metric))


# ------------------------------------------------------------------ inputs --

_shared = {}


def _context():
    """The one context a program keeps for its device."""
    if "ctx" not in _shared:
        _shared["ctx"] = gl.Context(0)
    return _shared["ctx"]


def _queue():
    """The one request queue a serving program keeps."""
    if "queue" not in _shared:
        _shared["queue"] = gl.lq_create(_context())
    return _shared["queue"]


def _grid(n, g, metric):
    side = math.isqrt(n - 1) + 1
    r = torch.arange(side, device="cuda", dtype=torch.float64)
    jit = torch.rand((2, side, side), generator=g, device="cuda", dtype=torch.float64) * 0.8 - 0.4
    x = ((r[:, None] + 0.5 + jit[0]) / side).reshape(-1)[:n].contiguous()
    y = ((r[None, :] + 0.5 + jit[1]) / side).reshape(-1)[:n].contiguous()
    return _place(x, y, metric)


def _place(x, y, metric):
    return (_LON0 + _SPAN * x, _LAT0 + _SPAN * y) if metric else (x, y)


def _scale(metric):
    """Unit of θ2: the side of the square."""
    return _KM if metric else 1.0


def _field(x, y, theta, seed, metric=0, waves=512):
    """Measurements: sqrt(2 θ1 / M) Σ cos(ω_m · s + φ_m) with ω_m from the Matérn spectral density
    (a t distribution), a field whose covariance over the draws is the Matérn one exactly."""
    t1, t2, t3 = theta
    rng = np.random.default_rng([seed, 17])
    w = rng.standard_normal((2, waves)) / np.sqrt(rng.chisquare(2.0 * t3, waves)) / t2
    ph = rng.uniform(0.0, 2.0 * math.pi, waves)
    w = torch.as_tensor(w).cuda()
    ph = torch.as_tensor(ph).cuda()
    if metric:
        x, y = (x - _LON0) / _SPAN, (y - _LAT0) / _SPAN
    z = torch.empty_like(x)
    for a in range(0, x.numel(), 16384):
        s = slice(a, a + 16384)
        z[s] = torch.cos(x[s, None] * w[0] + y[s, None] * w[1] + ph).sum(1)
    return z * math.sqrt(2.0 * t1 / waves)


_PREC = {"fp64": gl.GL_FP64, "fp32": gl.GL_MIXED_FP32, "bf16": gl.GL_MIXED_BF16, "fp16": gl.GL_MIXED_FP16}


class _Factor:
    """A kept Cholesky factor, released with its owner."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        gl.gl_factor_release(_context(), self.handle)


class _Datasets:
    """Datasets registered for the request queue, dropped with their owner."""

    def __init__(self, ids):
        self.ids = ids

    def __del__(self):
        for d in self.ids:
            gl.gl_dataset_release(_context(), d)


def _queue_fields(case):
    """Sizes and parameters of the queue's clients (the same for every seed)."""
    rng = np.random.default_rng([case["field"], 5])
    out = []
    for _ in range(case["requests"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
        t3 = float(rng.choice([0.5, 1.0, 1.5, 2.5]))
        cap = 25.0 ** (3.0 / (2.0 * t3 + 2.0)) / math.sqrt(n)
        out.append((n, (float(rng.uniform(0.5, 2.0)), min(float(rng.uniform(0.02, 0.15)), cap), t3)))
    return out


def prepare(case, seed):
    ctx = _context()
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    kind = case["kind"]
    if kind == "queue":
        jobs, ids = [], []
        for i, (n, th) in enumerate(_queue_fields(case)):
            x, y = _grid(n, g, 0)
            z = _field(x, y, th, seed + 1000 * i)
            torch.cuda.current_stream().synchronize()
            ids.append(gl.gl_dataset_register(ctx, x, y, z))
            jobs.append((ids[-1], th))
        return dict(kind=kind, queue=_queue(), jobs=jobs, owner=_Datasets(ids))
    metric = case.get("metric", 0)
    unit = _scale(metric)
    th1 = (case["t1"], case["t2"], case["t3"])  # in units of the square's side
    th = (case["t1"], case["t2"] * unit, case["t3"])
    dist = dict(metric=gl.GL_GREAT_CIRCLE, radius=_RADIUS) if metric else {}
    if kind == "sigma12":
        x, y = _grid(case["n1"], g, metric)
        u = torch.rand((2, case["n2"]), generator=g, device="cuda", dtype=torch.float64)
        xn, yn = _place(u[0].contiguous(), u[1].contiguous(), metric)
        return dict(kind=kind, x=x, y=y, xn=xn, yn=yn, theta=th, opts=gl.gl_opts_default(**dist))
    n = case["n"]
    x, y = _grid(n, g, metric)
    z = _field(x, y, th1, seed, metric)
    s = dict(kind=kind, x=x, y=y, z=z, theta=th)
    if kind == "eval":
        s["opts"] = gl.gl_opts_default(precision=_PREC[case["precision"]], graph=case["graph"], **dist)
        s["fp64"] = case["precision"] == "fp64"
    elif kind == "ind":
        s["opts"] = gl.gl_opts_default(ind_tiles=case["tiles"])
    elif kind == "krige":
        r = gl.loglik_eval(ctx, x, y, z, th, gl.gl_opts_default(keep_factor=1))
        if r["status"] != gl.GL_OK:
            raise RuntimeError("the field's covariance is not positive definite")
        u = torch.rand((2, case["m"]), generator=g, device="cuda", dtype=torch.float64)
        s.update(owner=_Factor(r["factor"]), xn=u[0].contiguous(), yn=u[1].contiguous(), var=bool(case["var"]))
    elif kind == "cv":
        s["folds"] = _folds(n, case["k"], seed)
        s["pred"] = torch.empty(n, device="cuda", dtype=torch.float64)
        s["opts"] = gl.gl_opts_default()
    return s


def _folds(n, k, seed):
    """A random assignment of n points to k folds of equal size (to one)."""
    return np.random.default_rng([seed, 23]).permutation(np.arange(n, dtype=np.int32) % k)


# --------------------------------------------------------------------- run --

def _scalars(r):
    """l, log|Σ| and the quadratic form, in the binary64 they are computed in."""
    return {k: np.float64(r[k]) for k in ("loglik", "logdet", "quad")}


def run(s):
    ctx, kind = _context(), s["kind"]
    if kind in ("eval", "ind"):
        r = gl.loglik_eval(ctx, s["x"], s["y"], s["z"], s["theta"], s["opts"])
        if s.get("fp64", True):
            return _scalars(r)
        # the mixed modes hold the trailing matrix in 32 bits: plain numbers
        return {k: r[k] for k in ("loglik", "logdet", "quad")}
    if kind == "queue":
        tickets = [gl.lq_submit(s["queue"], ds, th) for ds, th in s["jobs"]]
        return [_scalars(gl.lq_wait(s["queue"], t)) for t in tickets]
    if kind == "krige":
        return gl.krige_predict(ctx, s["owner"].handle, s["xn"], s["yn"], return_variance=s["var"])
    if kind == "cv":
        mse, _ = gl.krige_cv(ctx, s["x"], s["y"], s["z"], s["theta"], s["folds"], s["opts"], pred=s["pred"])
        return {"mse": np.array(mse), "pred": s["pred"]}
    return gl.matern_generate(ctx, s["x"], s["y"], s["xn"], s["yn"], s["theta"], s["opts"])


# -------------------------------------------------------------------- work --

def work(case):
    """The least a pass has to do.  A likelihood: n³/3 flops of the factorisation and n² of the solve, the
    locations and measurements read, three numbers written.  Kriging: the factor read once per solve
    direction (mean) and n² flops per new location (variances).  Σ12: every entry written."""
    kind = case["kind"]

    def eval_flops(n):
        return n ** 3 / 3.0 + float(n) ** 2

    if kind == "eval":
        return {"bytes": 24.0 * case["n"] + 24, "flops": eval_flops(case["n"])}
    if kind == "ind":
        n = case["n"]
        block = case["tiles"] * gl.gl_pick_tile(n)
        full, rest = divmod(n, block)
        return {"bytes": 24.0 * n + 24, "flops": full * eval_flops(block) + eval_flops(rest)}
    if kind == "queue":
        ns = [n for n, _ in _queue_fields(case)]
        return {"bytes": sum(24.0 * n + 24 for n in ns), "flops": sum(eval_flops(n) for n in ns)}
    if kind == "krige":
        n, m = float(case["n"]), float(case["m"])
        f = {"bytes": 4.0 * n * n + 24 * n + 24 * m, "flops": n * n + 2.0 * n * m}
        if case["var"]:
            f["bytes"] += 8 * m
            f["flops"] += n * n * m
        return f
    if kind == "cv":
        n, k = case["n"], case["k"]
        known = n - n / k
        return {"bytes": 32.0 * n + 8 * k, "flops": k * (eval_flops(known) + known ** 2 + 2.0 * known * n / k)}
    n1, n2 = float(case["n1"]), float(case["n2"])
    return {"bytes": 8.0 * n1 * n2 + 16 * (n1 + n2), "flops": 20.0 * n1 * n2}


# ------------------------------------------------------------------- exact --

def _bessel_k(nu, x):
    """K_ν(x) = ∫_0^∞ exp(-x cosh t) cosh(νt) dt by the trapezoidal rule, times e^x."""
    top = torch.acosh(1.0 + (40.0 + 8.0 * nu) / x)
    steps = 80
    h = top / steps
    acc = torch.full_like(x, 0.5)
    for i in range(1, steps + 1):
        t = h * i
        sh = torch.sinh(0.5 * t)
        acc += torch.exp(-2.0 * x * sh * sh) * torch.cosh(nu * t)
    return acc * h


def _matern(r, theta):
    t1, t2, t3 = theta
    x = r / t2
    if t3 == 0.5:
        c = torch.exp(-x)
    elif t3 == 1.5:
        c = (1.0 + x) * torch.exp(-x)
    elif t3 == 2.5:
        c = (1.0 + x + x * x / 3.0) * torch.exp(-x)
    else:
        xs = x.clamp_min(1e-12)
        c = 2.0 ** (1.0 - t3) / math.gamma(t3) * torch.exp(t3 * torch.log(xs) - xs) * _bessel_k(t3, xs)
        c = torch.where(x == 0.0, torch.ones_like(c), c)
    return t1 * c


def _cov(x1, y1, x2, y2, theta, metric=0):
    out = torch.empty((x1.numel(), x2.numel()), device="cuda", dtype=torch.float64)
    rows = max(1, (1 << 25) // x2.numel())
    deg = math.pi / 180.0
    for a in range(0, x1.numel(), rows):
        xa, ya = x1[a:a + rows, None], y1[a:a + rows, None]
        if metric:
            sp = torch.sin(0.5 * deg * (ya - y2))
            sl = torch.sin(0.5 * deg * (xa - x2))
            h = (sp * sp + torch.cos(deg * ya) * torch.cos(deg * y2) * sl * sl).clamp(0.0, 1.0)
            r = 2.0 * _RADIUS * torch.asin(torch.sqrt(h))
        else:
            r = torch.sqrt((xa - x2) ** 2 + (ya - y2) ** 2)
        out[a:a + rows] = _matern(r, theta)
    return out


def _tri(L, b, upper=False):
    b = b if b.ndim == 2 else b[:, None]
    return torch.linalg.solve_triangular(L.T if upper else L, b, upper=upper)


def _exact_eval(x, y, z, theta, metric=0):
    L = torch.linalg.cholesky(_cov(x, y, x, y, theta, metric))
    w = _tri(L, z)
    logdet = 2.0 * torch.log(torch.diagonal(L)).sum().item()
    quad = (w * w).sum().item()
    n = x.numel()
    return {"loglik": np.float64(-0.5 * n * math.log(2.0 * math.pi) - 0.5 * logdet - 0.5 * quad),
            "logdet": np.float64(logdet), "quad": np.float64(quad)}


def _exact_krige(x, y, z, xn, yn, theta, var):
    L = torch.linalg.cholesky(_cov(x, y, x, y, theta))
    u = _tri(L, _cov(x, y, xn, yn, theta))
    w = _tri(L, z)
    mean = (u * w).sum(0)
    return (mean, theta[0] - (u * u).sum(0)) if var else mean


def exact(case, seed):
    """The same in plain torch, in 64 bits: dense covariance, LAPACK-style Cholesky, triangular solves."""
    kind = case["kind"]
    if work(case)["flops"] > 8e12 or (kind == "eval" and case["precision"] != "fp64"):
        return None
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    if kind == "queue":
        out = []
        for i, (n, th) in enumerate(_queue_fields(case)):
            x, y = _grid(n, g, 0)
            out.append(_exact_eval(x, y, _field(x, y, th, seed + 1000 * i), th))
        return out
    metric = case.get("metric", 0)
    th1 = (case["t1"], case["t2"], case["t3"])
    th = (case["t1"], case["t2"] * _scale(metric), case["t3"])
    if kind == "sigma12":
        x, y = _grid(case["n1"], g, metric)
        u = torch.rand((2, case["n2"]), generator=g, device="cuda", dtype=torch.float64)
        xn, yn = _place(u[0], u[1], metric)
        return _cov(xn, yn, x, y, th, metric)
    n = case["n"]
    if n > 20000 and kind != "ind":
        return None
    x, y = _grid(n, g, metric)
    z = _field(x, y, th1, seed, metric)
    if kind == "eval":
        return _exact_eval(x, y, z, th, metric)
    if kind == "ind":
        block = case["tiles"] * gl.gl_pick_tile(n)
        parts = [_exact_eval(x[a:a + block], y[a:a + block], z[a:a + block], th) for a in range(0, n, block)]
        return {k: np.float64(math.fsum(p[k] for p in parts)) for k in ("loglik", "logdet", "quad")}
    if kind == "krige":
        u = torch.rand((2, case["m"]), generator=g, device="cuda", dtype=torch.float64)
        return _exact_krige(x, y, z, u[0], u[1], th, bool(case["var"]))
    folds = torch.as_tensor(_folds(n, case["k"], seed)).cuda()
    pred = torch.empty_like(z)
    mse = []
    for f in range(case["k"]):
        o, m = folds != f, folds == f
        pred[m] = _exact_krige(x[o], y[o], z[o], x[m], y[m], th, False)
        mse.append(((pred[m] - z[m]) ** 2).mean().item())
    return {"mse": np.array(mse), "pred": pred}
