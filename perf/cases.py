"""Performance cases of the graph-form solver: what users have it do, through
its public entry points, from the smallest calls to the largest.

A case is a dict of plain values; its ``kind`` says which call it times:

  solve    one whole problem on a matrix that is new: pogs_init (copy,
           equilibration, Gram matrix, factor), pogs_solve, pogs_free
  resolve  pogs_solve on a context that is kept (new right-hand sides, warm
           starts, fixed iteration budgets on the same matrix)
  path     pogs_solve_path: R values of lambda on a kept context
  batch    pogs_solve_batch: independent problems from host memory
  serve    the serving engine: requests submitted, waited for and collected
  project  pogs_project on a kept context (device vectors)

``exact`` computes the same outputs in float64 with plain torch.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_1503_08366_amd import pogs as P
from paper_1503_08366_amd.workloads import Fn

EPS_ABS, EPS_REL = 1e-4, 1e-3  # Section 5 defaults of the method
ALPHA, DELTA, TAU, SWEEPS = 1.7, 1.05, 0.8, 10
CG_TOL, CG_CAP = 0.1, 10
NOMINAL_ITERS = 50  # iterations that work() counts where the data decide how many run


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def _case(kind, problem, m, n, dtype="float32", order="row", projection="direct", cap=2000, warm=False):
    return {"kind": kind, "problem": problem, "m": m, "n": n, "dtype": dtype, "order": order,
            "projection": projection, "cap": cap, "warm": warm}


def _named(name, case):
    return dict(case, name=name)


def listed():
    return [
        # the smallest whole problem a user solves (the small float64 Lasso of the tests): launches and host latency
        _named("lasso_200x100_f64", _case("solve", "lasso", 200, 100, "float64")),
        # a model refitted on a kept matrix, warm-started from the last coefficients, odd sizes
        _named("logistic_refit_1999x503", _case("resolve", "logistic", 1999, 503, warm=True)),
        # an ordinary float64 fit handed over column-major (robust regression from a statistics package)
        _named("huber_3000x700_f64_col", _case("solve", "huber", 3000, 700, "float64", "col")),
        # more unknowns than rows (feature selection): the wide form of the projection
        _named("wide_lasso_1000x5000", _case("solve", "lasso", 1000, 5000)),
        # the benchmark's headline problem, whole
        _named("lasso_20000x2000", _case("solve", "lasso", 20000, 2000)),
        # treatment planning: a new dose target on a kept 400 MB matrix, fixed iteration budget
        _named("dose_100000x1000", _case("resolve", "dose", 100000, 1000, cap=200)),
        # the indirect projection, for matrices whose factor is not wanted
        _named("cgls_lasso_20000x2000", _case("solve", "lasso", 20000, 2000, projection="cgls")),
        # the benchmark's sparse problem on a kept context
        _named("sparse_lasso_2000000x200000", dict(_case("resolve", "sparse", 2000000, 200000, projection="cgls"),
                                                   per_row=16)),
        # cross-validation: 64 values of lambda on one matrix
        _named("path64_8000x1000", dict(_case("path", "lasso", 8000, 1000), count=64)),
        # many small independent fits in one call, from host memory
        _named("batch32_mixed", dict(_case("batch", "mixed", 4096, 1024), count=32, shapes=3)),
        # mixed requests through the serving engine, from host memory
        _named("serve16_mixed", dict(_case("serve", "mixed", 50000, 5000), count=16, shapes=4)),
        # the projection alone, inside somebody's own splitting method
        _named("project_20000x2000", _case("project", "lasso", 20000, 2000)),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choice(["solve", "solve", "solve", "resolve", "resolve", "path", "batch", "serve", "project", "sparse"])
    if kind == "batch":
        return dict(_case("batch", "mixed", 4096, 1024), count=_log_int(rng, 4, 32), shapes=rng.randrange(1 << 30))
    if kind == "serve":
        return dict(_case("serve", "mixed", 20000, 2000), count=_log_int(rng, 4, 16), shapes=rng.randrange(1 << 30))
    if kind == "path":
        return dict(_case("path", "lasso", _log_int(rng, 1000, 8000), _log_int(rng, 100, 1000)),
                    count=_log_int(rng, 4, 64))
    if kind == "sparse":
        m = _log_int(rng, 20000, 1000000)
        return dict(_case("resolve", "sparse", m, max(1000, m // rng.choice([4, 7, 10])), projection="cgls"),
                    per_row=rng.randrange(6, 25))
    dtype = "float64" if rng.random() < 0.25 else "float32"
    big, small = (4000, 1000) if dtype == "float64" else (20000, 2000)
    n = _log_int(rng, 50, small)
    m = max(n, _log_int(rng, 100, big))
    wide = rng.random() < 0.25
    if wide:  # rows and columns change places; as many unknowns as the serving requests have
        m, n = n, min(m, 5000)
        m = min(m, n)
    if kind == "project":
        return _case("project", "lasso", m, n, dtype, rng.choice(["row", "col"]))
    problem = rng.choice(["lasso", "svm"]) if wide else rng.choice(["lasso", "nnls", "logistic", "huber", "svm"])
    if kind == "resolve":
        return _case("resolve", problem, m, n, dtype, "row", cap=400, warm=rng.random() < 0.5)
    projection = "cgls" if not wide and problem in ("lasso", "nnls") and rng.random() < 0.25 else "direct"
    return _case("solve", problem, m, n, dtype, rng.choice(["row", "row", "col"]), projection, cap=400)


def _shapes(case):
    """Problem kinds and sizes of a batch or of a stream of requests: fixed by the case, the data by the seed."""
    rng = random.Random(case["shapes"])
    out = []
    for i in range(case["count"]):
        if case["kind"] == "batch":  # the 512-problem mix: m ~ U{64..4096}, n ~ U{32..1024}, Lasso and logistic in turn
            out.append((("lasso", "logistic")[i % 2], rng.randint(64, case["m"]), rng.randint(32, case["n"])))
        else:  # the serving mix: log-uniform sizes
            out.append((rng.choice(["lasso", "nnls", "svm"]), _log_int(rng, 100, case["m"]), _log_int(rng, 50, case["n"])))
    return out


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)


def _mul(A, x):
    return torch.cat([(a.double() * x).sum(1) for a in A.split(8192)])


def _mul_t(A, v):
    acc = torch.zeros(A.shape[1], dtype=torch.float64, device=A.device)
    for a, w in zip(A.split(8192), v.split(8192)):
        acc += (a.double() * w[:, None]).sum(0)
    return acc


def _fn(h, a=1.0, b=0.0, c=1.0, d=0.0, e=0.0):
    """One separable function: its base function and the parameters of c h(a y - b) + d y + (e/2) y^2."""
    return {"h": h, "a": a, "b": b, "c": c, "d": d, "e": e}


def _truth(g, n):
    x = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    return x * (torch.rand(n, generator=g, device="cuda", dtype=torch.float64) < 0.1)


def _dense(problem, m, n, dtype, seed):
    """(A, f, g, x0): the matrix (m x n, on the GPU) and the functions of one problem, and a guess of its solution."""
    g = _gen(seed)
    dt = torch.float64 if dtype == "float64" else torch.float32
    A = torch.randn((m, n), generator=g, device="cuda", dtype=dt)
    if problem == "dose":
        A = A.abs_() * (torch.rand((m, n), generator=g, device="cuda", dtype=dt) < 0.3)
        t = 0.5 + torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
        return A, _fn("abs", b=t.cpu().numpy(), c=0.6, d=0.4), _fn("ind_ge0"), None
    if problem == "svm":  # two clusters, the label folded into the rows
        s = torch.where(torch.arange(m, device="cuda") < m // 2, 1.0, -1.0).to(dt)
        A = s[:, None] * (A / math.sqrt(n) + s[:, None] / n)
        return A, _fn("hinge", a=-1.0, b=-1.0), _fn("square", c=2.0), None
    A /= math.sqrt(n)
    x = _truth(g, n)
    x0 = (x + 0.05 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)).cpu().numpy()
    y = _mul(A, x)
    noise = torch.randn(m, generator=g, device="cuda", dtype=torch.float64)
    if problem == "logistic":
        b01 = ((y + 0.01 * noise) > 0).double()
        lam = 0.1 * float(_mul_t(A, 0.5 - b01).abs().max())
        return A, _fn("logistic", d=-b01.cpu().numpy()), _fn("abs", c=lam), x0
    if problem == "huber":
        far = torch.rand(m, generator=g, device="cuda", dtype=torch.float64) >= 0.95
        b = y + torch.where(far, 10.0 * noise.abs(), 0.5 * noise)
        return A, _fn("huber", a=-1.0, b=-b.cpu().numpy()), _fn("square", c=0.1), x0
    b = y + 0.01 * noise
    f = _fn("square", b=b.cpu().numpy())
    if problem == "nnls":
        return A, f, _fn("ind_ge0"), x0
    return A, f, _fn("abs", c=0.1 * float(_mul_t(A, b).abs().max())), x0


def _lambdas(case, A, f):
    top = float(_mul_t(A, torch.from_numpy(f["b"]).cuda()).abs().max())
    return [_fn("abs", c=float(top * 10.0 ** t)) for t in np.linspace(-3.0, 0.0, case["count"])]


def _sparse(case, seed):
    """Row pointers, columns, values of a matrix with per_row entries a row, and the Lasso's functions on it."""
    g = _gen(seed)
    m, n, k = case["m"], case["n"], case["per_row"]
    cols = torch.randint(0, n, (m, k), generator=g, device="cuda").sort(1).values
    vals = torch.randn((m, k), generator=g, device="cuda") / math.sqrt(k)
    x = _truth(g, n)
    b = (vals.double() * x[cols]).sum(1) + 0.01 * torch.randn(m, generator=g, device="cuda", dtype=torch.float64)
    back = torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, cols.reshape(-1),
                                                                        (vals.double() * b[:, None]).reshape(-1))
    rows = torch.arange(0, m * k + 1, k, device="cuda")
    return rows, cols.reshape(-1), vals.reshape(-1), _fn("square", b=b.cpu().numpy()), _fn(
        "abs", c=0.1 * float(back.abs().max()))


def _user_fn(f, size):
    return Fn(f["h"], size, a=f["a"], b=f["b"], c=f["c"], d=f["d"], e=f["e"])


class _HostProblem:
    """One problem in host memory, as the batch call and the engine take it."""

    def __init__(self, A, f, g, cap):
        self.A, (self.m, self.n) = A.cpu().numpy(), A.shape
        self.f, self.g = _user_fn(f, self.m), _user_fn(g, self.n)
        self.eps_abs, self.eps_rel, self.max_iter = EPS_ABS, EPS_REL, cap


def prepare(case, seed):
    kind, m, n = case["kind"], case["m"], case["n"]
    if kind in ("batch", "serve"):
        probs = []
        for i, (problem, pm, pn) in enumerate(_shapes(case)):
            A, f, g, _ = _dense(problem, pm, pn, "float32", 1000 * seed + i)
            probs.append(_HostProblem(A, f, g, case["cap"]))
        return {"kind": kind, "problems": probs, "engine": P.BatchEngine() if kind == "serve" else None}
    params = P.default_params(max_iter=case["cap"], projection=case["projection"])
    s = {"kind": kind, "params": params}
    if case["problem"] == "sparse":
        rows, cols, vals, f, g = _sparse(case, seed)
        s["ctx"] = P.SparseContext(torch.sparse_csr_tensor(rows, cols, vals, (m, n)), params)
        s["f"], s["g"], s["x0"] = _user_fn(f, m), _user_fn(g, n), None
        return s
    A, f, g, x0 = _dense(case["problem"], m, n, case["dtype"], seed)
    if case["order"] == "col":
        A = A.t().contiguous().t()
    s["f"], s["g"] = _user_fn(f, m), _user_fn(g, n)
    s["x0"] = x0 if case["warm"] else None
    if kind == "solve":
        s["A"] = A
        return s
    s["ctx"] = P.Context(A, params)
    if kind == "path":
        lams = _lambdas(case, A, f)
        s["fs"], s["gs"] = [s["f"]] * len(lams), [_user_fn(h, n) for h in lams]
    elif kind == "project":
        s["c"], s["d"] = _vectors(case, seed)
    return s


def _vectors(case, seed):
    g = _gen(seed + 77)
    dt = torch.float64 if case["dtype"] == "float64" else torch.float32
    return tuple(torch.randn(k, generator=g, device="cuda", dtype=dt) for k in (case["n"], case["m"]))


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _one(r):
    return {"x": r.x, "y": r.y, "mu": r.mu, "nu": r.nu, "optval": float(r.optval), "iters": int(r.iters),
            "status": int(r.status)}


def _many(rs):
    out = {k: np.concatenate([getattr(r, k) for r in rs]) for k in ("x", "y", "mu", "nu")}
    out["optval"] = np.array([r.optval for r in rs])
    out["iters"] = np.array([r.iters for r in rs])
    out["status"] = np.array([r.status for r in rs])
    return out


def run(state):
    kind = state["kind"]
    if kind == "solve":
        with P.pogs_init(state["A"], state["params"]) as ctx:
            return _one(ctx.solve(state["f"], state["g"], state["params"]))
    if kind == "resolve":
        return _one(state["ctx"].solve(state["f"], state["g"], state["params"], x0=state["x0"]))
    if kind == "path":
        return _many(state["ctx"].solve_path(state["fs"], state["gs"], state["params"]))
    if kind == "batch":
        return _many(P.pogs_solve_batch(state["problems"]))
    if kind == "serve":
        eng = state["engine"]
        tickets = [eng.submit(p) for p in state["problems"]]
        eng.wait_all()
        return _many([eng.poll(t) for t in tickets])
    x, y = state["ctx"].project(state["c"], state["d"])
    return {"x": x, "y": y}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _work_one(m, n, size, setup, iters, cgls=False, nnz=None):
    a = m * n if nnz is None else nnz
    q, p = min(m, n), max(m, n)
    read = a * size + (a + m + 1) * 4 * (nnz is not None) + 8 * (m + n)
    flops = 4.0 * a * iters * (3 if cgls else 1)
    if setup:
        flops += 4.0 * a * SWEEPS
    if not cgls:
        flops += 2.0 * q * q * iters + (p * q * q + q ** 3 if setup else 0.0)
    return read + 2 * size * (m + n), flops


def work(case):
    m, n = case["m"], case["n"]
    size = 8 if case["dtype"] == "float64" else 4
    kind = case["kind"]
    if kind in ("batch", "serve"):
        each = [_work_one(pm, pn, 4, True, NOMINAL_ITERS) for _, pm, pn in _shapes(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    if kind == "project":
        q = min(m, n)
        return {"bytes": size * (m * n + q * q + 2 * (m + n)), "flops": 4.0 * m * n + 2.0 * q * q}
    iters = case["cap"] if case["problem"] == "dose" else NOMINAL_ITERS
    nnz = m * case["per_row"] if case["problem"] == "sparse" else None
    b, f = _work_one(m, n, size, kind == "solve", iters, case["projection"] == "cgls", nnz)
    if kind == "path":
        R = case["count"]
        return {"bytes": b + (R - 1) * (8 * n + 2 * size * (m + n)), "flops": f * R}
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The same outputs in float64 with plain torch
# ---------------------------------------------------------------------------
class _DenseOp:
    def __init__(self, A):
        self.A = A.double()
        self.m, self.n = A.shape

    def mul(self, x):
        return self.A @ x

    def mul_t(self, v):
        return self.A.t() @ v

    def squared(self):
        op = _DenseOp.__new__(_DenseOp)
        op.A, op.m, op.n = self.A * self.A, self.m, self.n
        return op

    def scale(self, D, E):
        self.A = D[:, None] * self.A * E


class _SparseOp:
    def __init__(self, rows, cols, vals, m, n):
        r = torch.arange(m, device="cuda").repeat_interleave(rows[1:] - rows[:-1])
        self.r, self.c, self.v, self.m, self.n = r, cols, vals.double(), m, n
        back = torch.argsort(cols, stable=True)
        self.back = back
        self.crow_t = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"),
                                 torch.bincount(cols, minlength=n).cumsum(0)])
        self.crow = rows
        self._pack()

    def _pack(self):
        self.S = torch.sparse_csr_tensor(self.crow, self.c, self.v, (self.m, self.n))
        self.T = torch.sparse_csr_tensor(self.crow_t, self.r[self.back], self.v[self.back], (self.n, self.m))

    def mul(self, x):
        return self.S @ x

    def mul_t(self, v):
        return self.T @ v

    def squared(self):
        op = _SparseOp.__new__(_SparseOp)
        op.__dict__.update(self.__dict__)
        op.v = self.v * self.v
        op._pack()
        return op

    def scale(self, D, E):
        self.v = D[self.r] * self.v * E[self.c]
        self._pack()


def _equilibrate(op, eps):
    """Section 4.2's Algorithm 2 (p = 2) and the Frobenius normalisation; op becomes D A E."""
    m, n = op.m, op.n
    sq = op.squared()
    gamma = (m + n) * math.sqrt(eps)
    e = torch.ones(n, dtype=torch.float64, device="cuda")
    for _ in range(SWEEPS):
        d = n / (sq.mul(e) + gamma / m)
        col = sq.mul_t(d)
        e = m / (col + gamma / n)
    s = torch.sqrt((e * col).sum() / min(m, n))
    D, E = torch.sqrt(d / s), torch.sqrt(e / s)
    del sq
    op.scale(D, E)
    return D, E


def _inverse(op):
    A = op.A
    G = A.t() @ A if op.m >= op.n else A @ A.t()
    G += torch.eye(G.shape[0], dtype=torch.float64, device="cuda")
    return torch.cholesky_inverse(torch.linalg.cholesky(G))


def _project(op, Kinv, c, d):
    if op.m >= op.n:
        x = Kinv @ (c + op.mul_t(d))
        y = op.mul(x)
    else:
        y = d + Kinv @ (op.mul(c) - d)
        x = c + op.mul_t(d - y)
    return x, y, c - x, d - y


def _cgls(op, xh, c, d, thr2):
    x, r1 = xh, d - op.mul(xh)
    s = op.mul_t(r1) + c - x
    p, gam = None, float(s @ s)
    for _ in range(CG_CAP):
        if not gam > thr2:
            break
        p = s if p is None else s + (gam / last) * p
        q = op.mul(p)
        a = gam / float(q @ q + p @ p)
        x, r1 = x + a * p, r1 - a * q
        s = op.mul_t(r1) + c - x
        last, gam = gam, float(s @ s)
    return x, d - r1, c - x, r1


class _Scaled:
    """f(y / D) or g(E x): the parameters as vectors, and its prox and value."""

    def __init__(self, f, size, scale):
        v = {k: torch.as_tensor(np.broadcast_to(np.asarray(f[k], dtype=np.float64), (size,)).copy()).cuda()
             for k in "abcde"}
        self.h, self.raw, self.scale = f["h"], v, scale
        self.a, self.b, self.c = v["a"] * scale, v["b"], v["c"]
        self.d, self.e = v["d"] * scale, v["e"] * scale * scale

    def prox(self, v, rho):
        vq = (rho * v - self.d) / (self.e + rho)
        r = (self.e + rho) / (self.c * self.a * self.a)
        z, t = self.a * vq - self.b, 1.0 / r
        if self.h == "square":
            u = r * z / (1.0 + r)
        elif self.h == "abs":
            u = torch.sign(z) * torch.clamp(z.abs() - t, min=0.0)
        elif self.h == "huber":
            u = torch.where(z.abs() <= 1.0 + t, r * z / (1.0 + r), z - torch.sign(z) * t)
        elif self.h == "hinge":
            u = torch.where(z > t, z - t, torch.clamp(z, max=0.0))
        elif self.h == "ind_ge0":
            u = torch.clamp(z, min=0.0)
        elif self.h == "logistic":
            lo, hi = z - t, z.clone()
            u = z - torch.sigmoid(z) * t
            for i in range(150):  # Newton inside a bracket, which every third step halves
                s = torch.sigmoid(u)
                g = s + r * (u - z)
                hi, lo = torch.where(g > 0, u, hi), torch.where(g > 0, lo, u)
                nxt = u - g / (s * (1.0 - s) + r)
                nxt = torch.where((nxt > lo) & (nxt < hi) & (i % 3 < 2), nxt, 0.5 * (lo + hi))
                ended = (hi - lo <= 1e-15 * torch.clamp(u.abs(), min=1.0)) | (g == 0)
                if bool(ended.all()):
                    break
                u = torch.where(g == 0, u, nxt)
        else:
            raise ValueError(self.h)
        return (u + self.b) / self.a

    def value(self, y):
        """Value at the original (unscaled) point; indicators are zero where a prox step leaves them."""
        v = self.raw
        u = v["a"] * y - v["b"]
        if self.h == "square":
            h = 0.5 * u * u
        elif self.h == "abs":
            h = u.abs()
        elif self.h == "huber":
            h = torch.where(u.abs() <= 1.0, 0.5 * u * u, u.abs() - 0.5)
        elif self.h == "hinge":
            h = torch.clamp(u, min=0.0)
        elif self.h == "logistic":
            h = torch.nn.functional.softplus(u, threshold=1e9)
        else:
            h = torch.zeros_like(u)
        return float((v["c"] * h + v["d"] * y + 0.5 * v["e"] * y * y).sum())


def _admm(op, D, E, Kinv, f, g, cap, x0=None):
    """Graph projection splitting with over-relaxation, residual stopping and the adaptive penalty (Algorithm 3)."""
    F, G = _Scaled(f, op.m, 1.0 / D), _Scaled(g, op.n, E)
    zero = lambda k: torch.zeros(k, dtype=torch.float64, device="cuda")  # noqa: E731
    x, y, xt, yt, rho = zero(op.n), zero(op.m), zero(op.n), zero(op.m), 1.0
    if x0 is not None:  # the missing dual by one proximal step
        x = torch.from_numpy(x0).cuda() / E
        y = op.mul(x)
        yt = F.prox(y, rho) - y
        xt = -op.mul_t(yt)
    k, lo, up = 0, 0, 0
    while True:
        ax, ay = x - xt, y - yt
        xh, yh = G.prox(ax, rho), F.prox(ay, rho)
        mu, nu = -rho * (xh - ax), -rho * (yh - ay)
        c, d = ALPHA * xh + (1.0 - ALPHA) * x + xt, ALPHA * yh + (1.0 - ALPHA) * y + yt
        eps_dual = EPS_ABS + EPS_REL * float(mu.norm())
        eps_pri = EPS_ABS + EPS_REL * float(yh.norm())
        r_dual, r_pri = float((op.mul_t(nu) + mu).norm()), float((op.mul(xh) - yh).norm())
        if Kinv is not None:
            x, y, xt, yt = _project(op, Kinv, c, d)
        else:
            x, y, xt, yt = _cgls(op, xh, c, d, (CG_TOL * eps_dual / rho) ** 2)
        done = 0 if r_pri < eps_pri and r_dual < eps_dual else None
        if done is None:
            new = rho
            if r_dual < eps_dual and TAU * k > lo:
                new, up = DELTA * rho, k
            elif r_pri < eps_pri and TAU * k > up:
                new, lo = rho / DELTA, k
            if new != rho:
                xt, yt, rho = xt * (rho / new), yt * (rho / new), new
            if k + 1 >= cap:
                done = 1
        k += 1
        if done is not None:
            break
    x, y = E * xh, yh / D
    return {"x": x, "y": y, "mu": mu / E, "nu": D * nu, "optval": F.value(y) + G.value(x), "iters": k, "status": done}


def _eps(dtype):
    return float(np.finfo(np.float64 if dtype == "float64" else np.float32).eps)


def _solved(op, f, g, case, eps, x0=None):
    D, E = _equilibrate(op, eps)
    return _admm(op, D, E, None if case["projection"] == "cgls" else _inverse(op), f, g, case["cap"], x0)


def _stacked(rs):
    out = {k: torch.cat([r[k] for r in rs]) for k in ("x", "y", "mu", "nu")}
    for k in ("optval", "iters", "status"):
        out[k] = np.array([r[k] for r in rs])
    return out


def exact(case, seed):
    kind, m, n = case["kind"], case["m"], case["n"]
    if kind in ("batch", "serve"):
        rs = []
        for i, (problem, pm, pn) in enumerate(_shapes(case)):
            A, f, g, _ = _dense(problem, pm, pn, "float32", 1000 * seed + i)
            rs.append(_solved(_DenseOp(A), f, g, case, _eps("float32")))
        return _stacked(rs)
    if case["problem"] == "sparse":
        rows, cols, vals, f, g = _sparse(case, seed)
        return _solved(_SparseOp(rows, cols, vals, m, n), f, g, case, _eps("float32"))
    A, f, g, x0 = _dense(case["problem"], m, n, case["dtype"], seed)
    op = _DenseOp(A)
    if kind == "path":
        lams = _lambdas(case, A, f)
        D, E = _equilibrate(op, _eps(case["dtype"]))
        Kinv = _inverse(op)
        return _stacked([_admm(op, D, E, Kinv, f, h, case["cap"]) for h in lams])
    if kind == "project":
        _equilibrate(op, _eps(case["dtype"]))
        c, d = _vectors(case, seed)
        x, y, _, _ = _project(op, _inverse(op), c.double(), d.double())
        return {"x": x, "y": y}
    return _solved(op, f, g, case, _eps(case["dtype"]), x0 if case["warm"] else None)
