"""The framework's measured work: what its users run, at the sizes of its own workloads.

Every case is a call sequence of the Python entry points on data that is resident on the
GPU: whole solves or runs of time steps (state loaded, then stepped in place), a grouped
run of several problems, and a single exponential action. ``listed`` gives the fixed
cases, ``draw`` more of the same ranges.

A case is a dict of plain values:
  kind    "steps" (one problem stepped), "batch" (``count`` problems stepped together),
          "expv" (one exponential action) or "phi1v" (one phi1 action)
  field   the problem: "smooth" (Dirichlet, a = 1 + amp tanh(s)), "aniso" (Dirichlet,
          strongly varying a), "paper3d" (Sec. 5.2 of the paper: mixed boundary data,
          advection in the extracted operator), "paper2d" (Sec. 5.1: periodic, Fourier)
  n1, n2, n3 (0 in 2D), scheme, prec, q (quadrature nodes of the ERK schemes, 0: exact
  phi), tau, steps, lam
"""
import math

import numpy as np
import torch

import paper_2303_15861_amd as mm

LOGISTIC = (0.0, 1.0, -1.0, 0.0)   # u (1 - u)
CUBIC = (0.0, 0.0, 1.0, -1.0)      # u^2 (1 - u)


def _case(name, kind, field, n, scheme, steps, tau, prec="fp64", q=0, lam=1.0, count=1):
    n = tuple(n) + (0,) * (3 - len(n))
    c = dict(kind=kind, field=field, n1=n[0], n2=n[1], n3=n[2], scheme=scheme, steps=steps, tau=tau, prec=prec, q=q,
             lam=lam, count=count)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one exponential action on a small grid: the smallest call, launch latency
        _case("expv 31^3", "expv", "smooth", (31, 31, 31), "l2b", 0, 1e-3),
        # a whole solve of the small 2D workload (Lawson-Euler, 100 steps)
        _case("le 63^2 solve", "steps", "smooth", (63, 63), "le", 100, 1e-3),
        # the largest 2D grid of the served request stream
        _case("l2b 511^2", "steps", "smooth", (511, 511), "l2b", 20, 1e-3),
        # the paper's periodic 2D problem at its timing size
        _case("sl2 periodic 256^2", "steps", "paper2d", (256, 256), "sl2", 8, 4.0 / 256, lam=0.57),
        # the paper's 3D problem (mixed boundary data) at its timing size
        _case("sl2 mixed 60^3", "steps", "paper3d", (60, 60, 60), "sl2", 16, 0.25 / 256, lam=0.53),
        # requests of one class advanced together, as the server does
        _case("batch of 8 l2b 63^3", "batch", "smooth", (63, 63, 63), "l2b", 10, 1e-3, count=8),
        # the medium 3D workloads
        _case("l2b 127^3", "steps", "smooth", (127, 127, 127), "l2b", 10, 5e-4),
        _case("etd2rk q4 127^3", "steps", "smooth", (127, 127, 127), "etd2rk", 4, 5e-4, q=4),
        # a grid of unequal odd and even axes
        _case("l2b 130x129x127", "steps", "smooth", (130, 129, 127), "l2b", 10, 5e-4),
        # the headline workload, FP64 and in the exact-slice precision that meets 1e-9
        _case("l2b 255^3", "steps", "smooth", (255, 255, 255), "l2b", 4, 1e-3),
        _case("l2b sliced5 255^3", "steps", "smooth", (255, 255, 255), "l2b", 4, 1e-3, prec="sliced5"),
        # the largest workload: anisotropic coefficient, ERK with quadrature
        _case("etd2rk q6 383^3", "steps", "aniso", (383, 383, 383), "etd2rk", 1, 2e-3, q=6),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    what = rng.choice(["l2b3d", "l2b3d", "ragged3d", "ragged3d", "erk3d", "erk3d", "2d", "paper3d", "paper2d", "sliced",
                       "batch", "action"])
    tau = 0.1 / rng.randint(50, 250)
    if what == "l2b3d":      # cubes of any size, the workloads' range
        n = _log_int(rng, 31, 256)
        return _case("", "steps", "smooth", (n,) * 3, rng.choice(["l2b", "l2b", "le"]), 4 if n > 160 else 10, tau)
    if what == "ragged3d":   # unequal axes
        n = tuple(_log_int(rng, 24, 256) for _ in range(3))
        return _case("", "steps", "smooth", n, rng.choice(["l2b", "l2b", "le"]), 4 if max(n) > 160 else 10, tau)
    if what == "erk3d":
        n = tuple(_log_int(rng, 48, 256) for _ in range(3)) if rng.random() < 0.5 else (_log_int(rng, 48, 256),) * 3
        return _case("", "steps", rng.choice(["smooth", "aniso"]), n, "etd2rk", 2, tau, q=rng.choice([0, 3, 4, 6]))
    if what == "2d":
        n = tuple(_log_int(rng, 33, 511) for _ in range(2)) if rng.random() < 0.5 else (_log_int(rng, 33, 511),) * 2
        return _case("", "steps", "smooth", n, rng.choice(["l2b", "l2b", "le"]), 20, tau)
    if what == "paper3d":
        N = rng.randint(16, 80)
        return _case("", "steps", "paper3d", (N,) * 3, rng.choice(["sl2", "sl2", "l2a", "sle"]), 16, 0.25 / 256,
                     lam=round(rng.uniform(0.51, 1.0), 3))
    if what == "paper2d":
        N = rng.randint(64, 256)
        return _case("", "steps", "paper2d", (N, N), rng.choice(["sl2", "sl2", "l2a", "l2b"]), 8, 4.0 / 256,
                     lam=round(rng.uniform(0.51, 1.0), 3))
    if what == "sliced":
        n = rng.randint(129, 256)
        return _case("", "steps", "smooth", (n,) * 3, "l2b", 4, tau, prec="sliced%d" % rng.randint(4, 6))
    if what == "batch":
        n = _log_int(rng, 31, 96)
        return _case("", "batch", "smooth", (n,) * 3, "l2b", 10, tau, count=rng.randint(2, 8))
    n = tuple(_log_int(rng, 17, 256) for _ in range(3))
    if rng.random() < 0.5:
        return _case("", "expv", "smooth", n, "l2b", 0, tau)
    return _case("", "phi1v", "smooth", n, "etd2rk", 0, tau, q=rng.choice([0, 4]))


# ------------------------------------------------------------------ inputs, from the seed alone

def _device():
    return "cuda:0" if torch.cuda.is_available() else "cpu"


def _sine_series(gen, n, kmax, nodes):
    """Sine series with coefficients N(0,1)/|k|^2 on the unknowns (or all nodes), shape (.., n2, n1)."""
    d, dev = len(n), _device()
    c = torch.randn(tuple(reversed(kmax)), generator=gen, dtype=torch.float64)
    k2 = sum(torch.arange(1, km + 1, dtype=torch.float64).reshape([-1 if i == j else 1 for j in range(d)]) ** 2
             for i, km in enumerate(reversed(kmax)))
    v = (c / k2).to(dev)
    for ax in range(d):                      # array axis ax is grid axis d - 1 - ax
        m, km = n[d - 1 - ax], kmax[d - 1 - ax]
        i = torch.arange(0, m + 2, device=dev) if nodes else torch.arange(1, m + 1, device=dev)
        k = torch.arange(1, km + 1, device=dev)
        basis = torch.sin(math.pi / (m + 1) * (i[:, None] * k[None, :]).double())
        shape = list(v.shape)
        v = basis @ v.movedim(ax, 0).reshape(km, -1)
        v = v.reshape([len(i)] + shape[:ax] + shape[ax + 1:]).movedim(0, ax)
    return v.contiguous()


class _Problem:
    """Coefficient, initial data and constants of one problem on the GPU."""

    def __init__(self, case, seed):
        self.n = tuple(case[k] for k in ("n1", "n2", "n3") if case[k])
        self.d = d = len(self.n)
        self.tau, self.lam, self.form, self.velocity, self.length = case["tau"], case["lam"], "flux", None, None
        self.bc, self.beta_bar = (mm.MM_BC_DIRICHLET,) * d, (0.0,) * d
        gen = torch.Generator().manual_seed(int(seed))
        dev = _device()
        if case["field"] in ("smooth", "aniso"):
            if case["field"] == "aniso":
                s = _sine_series(gen, self.n, (8, 2, 2)[:d], True)
                self.a = 0.01 + 0.995 * (1.0 + torch.tanh(3.0 * s))
            else:
                self.a = 1.0 + (0.5 if d == 2 else 0.9) * torch.tanh(_sine_series(gen, self.n, (4,) * d, True))
            u = _sine_series(gen, self.n, (8,) * d, False)
            self.u0 = u / u.abs().max()
            self.beta = (0.5, 0.5) if d == 2 else (10.0,) * d
            self.r = LOGISTIC if d == 2 else CUBIC
        elif case["field"] == "paper3d":
            N = self.n[0]
            x = torch.arange(1, N + 1, device=dev, dtype=torch.float64) / N
            xa = torch.arange(0, N + 2, device=dev, dtype=torch.float64) / N
            xa[N + 1] = xa[N - 1]
            g = torch.exp(-((xa - 0.5) ** 2))
            self.a = 0.1 * g[:, None, None] * g[None, :, None] * g[None, None, :]
            f = x * (1.0 - x) ** 2
            p = 1.0 + 0.1 * _sine_series(gen, self.n, (3, 3, 3), False)    # the printed u0, perturbed
            self.u0 = (27.0 / 4.0) ** 3 * f[:, None, None] * f[None, :, None] * f[None, None, :] * p
            self.beta = self.beta_bar = (-0.01,) * 3
            self.r, self.form, self.bc = (0.0, 1.0, 0.0, 1.0), "nondiv", (mm.MM_BC_NEUMANN,) * 3
        else:
            N, L = self.n[0], 6.0 * math.pi
            x = -3.0 * math.pi + L / N * torch.arange(N, device=dev, dtype=torch.float64)
            X2, X1 = torch.meshgrid(x, x, indexing="ij")
            self.a = torch.stack([0.5 + (X1.sin() * X2.sin()) ** 2 / 6.0, 0.5 + (X1.cos() * X2.cos()) ** 2 / 6.0])
            self.velocity = torch.stack([X1.sin() ** 2 / 5.0, X2.sin() ** 2 / 5.0])
            p = 0.2 * torch.randn(2, generator=gen, dtype=torch.float64)   # the printed u0, shifted
            self.u0 = torch.exp(-((X1 - p[0].item()) ** 2 + (X2 - p[1].item()) ** 2))
            self.beta = self.beta_bar = (0.1, 0.1)
            self.r, self.bc, self.length = (0.0, 0.25, -0.25, 0.0), (mm.MM_BC_PERIODIC,) * 2, (L, L)
        self.a, self.u0 = self.a.contiguous(), self.u0.contiguous()


_CTX = []


def _context():
    if not _CTX:
        _CTX.append(mm.Context(0))
    return _CTX[0]


def prepare(case, seed):
    ctx, parts = _context(), []
    for i in range(case["count"]):
        p = _Problem(case, seed + 1009 * i)
        op = mm.mumode_setup(ctx, p.d, p.n, p.a, p.beta, p.r, p.tau, case["scheme"], case["prec"], case["q"], p.lam,
                             p.beta_bar, p.bc, p.form, p.length, p.velocity)
        parts.append((op, p.u0, torch.empty_like(p.u0)))
    return {"case": case, "parts": parts}


def run(state):
    case, parts = state["case"], state["parts"]
    op, u0, u = parts[0]
    if case["kind"] == "expv":
        mm.mumode_expv(op, u0, u)
        return u
    if case["kind"] == "phi1v":
        mm.mumode_phi1v(op, u0, u)
        return u
    for _, start, v in parts:      # the initial data is loaded, then stepped in place
        v.copy_(start)
    if case["kind"] == "batch":
        mm.lawson_step_batch([p[0] for p in parts], [p[2] for p in parts], case["steps"])
        return [p[2] for p in parts]
    mm.step(op, u, case["steps"])
    return u


def work(case):
    """Initial data and coefficient read once, the result written once; per mode product the
    multiply-adds of a dense factor (on Dirichlet axes of half of it: the factors are
    centrosymmetric); the ERK stages as diagonal functions in the eigenbasis."""
    n = [case[k] for k in ("n1", "n2", "n3") if case[k]]
    dof = float(np.prod(n))
    fields = {"paper2d": 5}.get(case["field"], 1)        # a (and the velocity) next to u
    flops_action = dof * sum(2.0 * m for m in n) * (1.0 if case["field"].startswith("paper") else 0.5)
    actions = {"le": 1, "sle": 1, "l2b": 2, "l2a": 3, "sl2": 3, "etd2rk": 5}[case["scheme"]]
    times = case["steps"]
    if case["kind"] in ("expv", "phi1v"):
        actions, times, fields = (1 if case["kind"] == "expv" else 2), 1, 0
    if case["field"] == "paper2d":
        actions += 2.0                                   # the derivatives of the Fourier remainder
    return {"bytes": 8.0 * case["count"] * dof * (2 + (fields if fields != 5 else 4)),
            "flops": case["count"] * times * (flops_action * actions + 40.0 * dof)}


# ------------------------------------------------------------------ the same in plain torch
# Values are carried as unevaluated pairs hi + lo of 64-bit numbers, so that the result is
# the exact one to well below the rounding of any 64-bit evaluation.

def _two_sum(a, b):
    s = a + b
    t = s - a
    return s, (a - (s - t)) + (b - t)


def _top(x):
    """The leading 21 bits of every value against the largest one."""
    m = float(x.abs().max()) if x.numel() else 0.0
    if m == 0.0 or not math.isfinite(m):
        return x
    c = math.ldexp(1.5, math.frexp(m)[1] + 31)
    return (x + c) - c


def _mode(M, v, ax):
    """M (a longdouble matrix) along array axis ax of the pair v."""
    h = torch.from_numpy(M.astype(np.float64)).to(v[0].device)
    l = torch.from_numpy((M - M.astype(np.float64).astype(np.longdouble)).astype(np.float64)).to(v[0].device)
    mh = _top(h)
    ml = (h - mh) + l
    hi, lo = (t.movedim(ax, 0) for t in v)
    shape = hi.shape
    hi, lo = hi.reshape(shape[0], -1), lo.reshape(shape[0], -1)
    xh = _top(hi)
    xl = (hi - xh) + lo
    y = _two_sum(mh @ xh, ml @ hi + mh @ xl)            # (the first product is exact)
    return tuple(t.reshape(shape).movedim(0, ax).contiguous() for t in y)


def _add(v, w, c=1.0):
    """v + c w (c a 64-bit number)."""
    p = c * w[0]
    split = 134217729.0
    ch = c * split - (c * split - c)
    wh = w[0] * split - (w[0] * split - w[0])
    e = ((ch * wh - p) + ch * (w[0] - wh) + (c - ch) * wh) + (c - ch) * (w[0] - wh)
    s, t = _two_sum(v[0], p)
    return _two_sum(s, t + (v[1] + (e + c * w[1])))


class _Exact:
    def __init__(self, case, p):
        self.p, self.d = p, p.d
        self.periodic = p.length is not None
        L = np.longdouble
        self.pi = L("3.14159265358979323846264338327950288")
        self.h = [float(p.length[m]) / n if self.periodic else 1.0 / n if p.bc[m] == mm.MM_BC_NEUMANN else 1.0 / (n + 1)
                  for m, n in enumerate(p.n)]
        self.amax = ([float(p.a[m].max()) for m in range(self.d)] if self.periodic else [float(p.a.max())] * self.d)
        self.cache = {}

    def axis(self, m):
        return self.d - 1 - m

    def circulant(self, m, sym):
        n, L = self.p.n[m], np.longdouble
        k = np.arange(n)
        ks = np.where(k <= (n - 1) // 2, k, k - n).astype(L)
        nyq = (k == n // 2) & (n % 2 == 0)
        re, im = sym(ks * 2 * self.pi / L(self.p.length[m]), nyq)
        t = 2 * self.pi * (np.outer(k, k) % n).astype(L) / n
        col = (np.cos(t) @ re - np.sin(t) @ im) / n
        return col[(k[:, None] - k[None, :]) % n]

    def factor(self, c, m):
        """exp(c tau A_m) in extended precision."""
        key = (c, self.p.n[m], self.amax[m], self.p.bc[m], self.p.beta_bar[m])
        if key in self.cache:
            return self.cache[key]
        p, n, L = self.p, self.p.n[m], np.longdouble
        la, bb, ct = L(p.lam) * L(self.amax[m]), L(p.beta_bar[m]), L(c) * L(p.tau)
        if self.periodic:
            def sym(k, nyq):
                mag, ph = np.exp(-ct * la * k * k), np.where(nyq, L(0), ct * bb * k)
                return mag * np.cos(ph), mag * np.sin(ph)
            E = self.circulant(m, sym)
        elif p.bc[m] == mm.MM_BC_DIRICHLET and p.beta_bar[m] == 0.0:
            j = np.arange(1, n + 1)
            S = np.sqrt(L(2) / (n + 1)) * np.sin(self.pi * (np.outer(j, j) % (2 * n + 2)).astype(L) / (n + 1))
            ev = -4 * la * L(n + 1) ** 2 * np.sin(self.pi * j.astype(L) / (2 * n + 2)) ** 2
            E = (S * np.exp(ct * ev)) @ S
        else:
            h = L(1) / (n if p.bc[m] == mm.MM_BC_NEUMANN else n + 1)
            dif, adv = la / (h * h), bb / (2 * h)
            A = np.diag(np.full(n, -2 * dif)) + np.diag(np.full(n - 1, dif - adv), -1) + np.diag(np.full(n - 1, dif + adv), 1)
            if p.bc[m] == mm.MM_BC_NEUMANN and n >= 2:
                A[n - 1, n - 2] = 2 * dif
            A = A * ct
            s = max(0, int(math.ceil(math.log2(max(1e-30, float(np.abs(A).sum(1).max()))))) + 3)
            A, E, T = A / L(2) ** s, np.eye(n, dtype=L), np.eye(n, dtype=L)
            for i in range(1, 19):
                T = (T @ A) / i
                E = E + T
            for _ in range(s):
                E = E @ E
        self.cache[key] = E
        return E

    def act(self, c, v):
        for m in range(self.d):
            v = _mode(self.factor(c, m), v, self.axis(m))
        return v

    def shifted(self, u, m):
        """Neighbours u+ and u- along grid axis m (zero Dirichlet ghosts, mirror at a Neumann end)."""
        ax = self.axis(m)
        up, um = torch.zeros_like(u), torch.zeros_like(u)
        k = u.shape[ax]
        up.narrow(ax, 0, k - 1).copy_(u.narrow(ax, 1, k - 1))
        um.narrow(ax, 1, k - 1).copy_(u.narrow(ax, 0, k - 1))
        if self.p.bc[m] == mm.MM_BC_NEUMANN:
            up.narrow(ax, k - 1, 1).copy_(um.narrow(ax, k - 1, 1))
        return up, um

    def linear(self, u, full):
        """The linear part of g (full: of F) on one component of a pair, finite differences."""
        p, out = self.p, torch.zeros_like(u)
        a = p.a[tuple(slice(1, -1) for _ in range(self.d))]
        for m in range(self.d):
            ax, ih2 = self.axis(m), 1.0 / (self.h[m] * self.h[m])
            la = 0.0 if full else p.lam * self.amax[m]
            up, um = self.shifted(u, m)
            if p.form == "nondiv":
                out += (a - la) * ((up - u) - (u - um)) * ih2
            else:
                sl = [slice(1, -1)] * self.d
                sl[ax] = slice(2, None)
                ap = p.a[tuple(sl)]
                sl[ax] = slice(0, -2)
                am = p.a[tuple(sl)]
                out += ((0.5 * (a + ap) - la) * (up - u) - (0.5 * (a + am) - la) * (u - um)) * ih2
            b = p.beta[m] - (0.0 if full else p.beta_bar[m])
            out += b / (2.0 * self.h[m]) * (up - um)
        return out

    def rhs(self, v, full=False):
        """g(v), or F(v) = A v + g(v)."""
        p = self.p
        hi, lo = v
        r0, r1, r2, r3 = p.r
        react = r0 + hi * (r1 + hi * (r2 + hi * r3)) + lo * (r1 + hi * (2 * r2 + hi * 3 * r3))
        if not self.periodic:
            return _two_sum(self.linear(hi, full), self.linear(lo, full) + react)
        out = (react, torch.zeros_like(react))
        L = np.longdouble
        for m in range(self.d):
            ax, la = self.axis(m), p.lam * self.amax[m]
            if ("D", m) not in self.cache:
                self.cache["D", m] = self.circulant(m, lambda k, q: (0 * k, np.where(q, L(0), k)))
                self.cache["A", m] = self.circulant(m, lambda k, q: (-L(p.lam) * L(self.amax[m]) * k * k,
                                                                     np.where(q, L(0), L(p.beta_bar[m]) * k)))
            D = self.cache["D", m]
            t = _mode(D, v, ax)
            ca, cb = p.a[m] - la, p.velocity[m] - p.beta_bar[m]
            flux = _add(_two_sum(ca * t[0], ca * t[1]), _two_sum(cb * hi, cb * lo))
            out = _add(out, _mode(D, flux, ax))
            if full:
                out = _add(out, _mode(self.cache["A", m], v, ax))
        return out

    def phi(self, q, v):
        """The quadrature of phi1(tau A) v, or phi1 itself (q = 0) in the sine basis."""
        if q:
            x, w = np.polynomial.legendre.leggauss(q)
            out = (torch.zeros_like(v[0]), torch.zeros_like(v[0]))
            for xj, wj in zip(x, w):
                out = _add(out, self.act(0.5 * (xj + 1.0), v), 0.5 * wj)
            return out
        return self.diagonal(v, lambda z: torch.where(z == 0, torch.ones_like(z), torch.expm1(z) / z))

    def diagonal(self, v, f):
        L, ev = np.longdouble, []
        for m, n in enumerate(self.p.n):
            j = np.arange(1, n + 1)
            if ("S", n) not in self.cache:
                self.cache["S", n] = np.sqrt(L(2) / (n + 1)) * np.sin(
                    self.pi * (np.outer(j, j) % (2 * n + 2)).astype(L) / (n + 1))
            e = -4 * L(self.p.lam) * L(self.amax[m]) * L(n + 1) ** 2 * np.sin(self.pi * j.astype(L) / (2 * n + 2)) ** 2
            shape = [1] * self.d
            shape[self.axis(m)] = n
            ev.append(torch.from_numpy((e * L(self.p.tau)).astype(np.float64)).to(v[0].device).reshape(shape))
            v = _mode(self.cache["S", n], v, self.axis(m))
        s = f(sum(ev))
        v = _two_sum(s * v[0], s * v[1])
        for m, n in enumerate(self.p.n):
            v = _mode(self.cache["S", n], v, self.axis(m))
        return v

    def step(self, scheme, q, u):
        tau = self.p.tau
        if scheme == "le":
            return self.act(1.0, _add(u, self.rhs(u), tau))
        if scheme == "sle":
            return _add(u, self.act(1.0, self.rhs(u, True)), tau)
        if scheme == "l2b":
            g = self.rhs(u)
            U = self.act(1.0, _add(u, g, tau))
            return _add(self.act(1.0, _add(u, g, 0.5 * tau)), self.rhs(U), 0.5 * tau)
        if scheme == "l2a":
            U = self.act(0.5, _add(u, self.rhs(u), 0.5 * tau))
            return _add(self.act(1.0, u), self.act(0.5, self.rhs(U)), tau)
        if scheme == "sl2":
            al, F, g = 0.327, self.rhs(u, True), self.rhs(u)
            U = _add(u, self.act(al, F), al * tau)
            D = _add(self.rhs(U), g, -1.0)
            return _add(_add(u, self.act(0.5, F), tau), self.act(1.0, D), 0.5 * tau / al)
        g = self.rhs(u)                                              # etd2rk
        U = _add(self.act(1.0, u), self.phi(q, g), tau)
        return _add(U, self.phi(q, _add(self.rhs(U), g, -1.0)), 0.5 * tau)


def exact(case, seed):
    out = []
    for i in range(case["count"]):
        p = _Problem(case, seed + 1009 * i)
        e, u = _Exact(case, p), (p.u0, torch.zeros_like(p.u0))
        if case["kind"] == "expv":
            u = e.act(1.0, u)
        elif case["kind"] == "phi1v":
            u = e.phi(case["q"], u)
        else:
            for _ in range(case["steps"]):
                u = e.step(case["scheme"], case["q"], u)
        out.append(u[0] + u[1])
    return out if case["kind"] == "batch" else out[0]
