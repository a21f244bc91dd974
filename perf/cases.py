"""Performance cases of the propagator library: what its users run, through
the public entry points of ``paper_1204_5434_amd.binding``.

Four calls carry the work of a polymer field-theory program:

* ``evaluate``: propagators, densities, Q and H of given fields (SCFT mixing
  schemes, free-energy scans, the paper's benchmark);
* ``step``: one field step in place (deterministic relaxation, complex
  Langevin with noise, explicit or semi-implicit);
* ``gradient``: dH/dw and dH/dL by the reverse mode;
* ``batch``: one field step of many independent replicas.

Each runs in complex-double or complex-float propagators.  Results of a
complex-float context carry single precision, so their program keeps them as
complex64; H and dH/dL, differences of nearly cancelling extensive terms, are
kept by the double-precision programs only (the float ones log Q).

``exact`` computes the same results with plain torch in 64 bits: every
diffusion is a dense real matrix per axis, built from the Fourier, cosine or
sine modes of Eq. (5).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1204_5434_amd import binding as B

DEV = "cuda"
AXES = (8, 12, 16, 20, 24, 32, 40, 48, 64, 80, 96, 128, 192, 256)


def _case(call, n, L, ns, f, prec, **kw):
    c = dict(call=call, nx=n[0], ny=n[1], nz=n[2], lx=float(L[0]), ly=float(L[1]), lz=float(L[2]), ns=ns,
             f=float(f), chin=14.0, c=1.0, prec=prec, scheme="rqm4", model="diblock", b=1.0, walls="ppp",
             storage=0, update="explicit", noise=False, dt=0.01, sr=0.1, si=0.02, cosine=0.0, replicas=1)
    c.update(kw)
    return c


def listed():
    def named(name, c):
        return dict(c, name=name)

    return [
        # deterministic SCFT relaxation of a small unit cell: launches and latency
        named("scft16_f64", _case("step", (16,) * 3, (4.0,) * 3, 50, 0.5, "f64", chin=15.0, dt=0.05, si=0.0)),
        # one replica of a parameter study run by itself
        named("replica32_f32", _case("step", (32,) * 3, (4.0,) * 3, 60, 0.4, "f32", chin=20.0, c=50.0, noise=True)),
        # complex-Langevin production step of a unit cell
        named("langevin64_f64", _case("step", (64,) * 3, (6.0,) * 3, 100, 0.4, "f64", chin=20.0, c=50.0, noise=True,
                                      sr=0.2, si=0.05)),
        # the same with float propagators and the semi-implicit update
        named("langevin64_f32_sis", _case("step", (64,) * 3, (6.0,) * 3, 100, 0.4, "f32", chin=20.0, c=50.0,
                                          noise=True, sr=0.2, si=0.05, update="semi")),
        # lamellar evaluation at the paper's largest grid (the library's benchmark), both precisions
        named("lam128_f64", _case("evaluate", (128,) * 3, (10.89,) * 3, 100, 0.5, "f64")),
        named("lam128_f32", _case("evaluate", (128,) * 3, (10.89,) * 3, 100, 0.5, "f32")),
        # homopolymer solution (one sweep) on the benchmark grid
        named("edwards128_f32", _case("evaluate", (128,) * 3, (10.89,) * 3, 100, 0.5, "f32", model="edwards")),
        # film between reflecting walls, uneven axes, a block junction inside a contour step
        named("film_f64", _case("evaluate", (80, 96, 40), (7.0, 8.2, 3.4), 75, 0.37, "f64", chin=18.0, walls="ppr")),
        # uneven periodic cell (hexagonal cylinders), float propagators, second-order steps
        named("cell_f32_split2", _case("evaluate", (48, 80, 192), (4.0, 6.9, 15.0), 90, 0.33, "f32", scheme="split2",
                                       chin=19.0)),
        # variable-cell gradient: dH/dw and the box derivative
        named("gradient96_f64", _case("gradient", (96,) * 3, (5.5,) * 3, 128, 0.3, "f64", chin=18.0, sr=0.05, si=0.0,
                                      cosine=1.0)),
        # 256 uneven replicas (24-48 points a side, 40-80 contour steps) advanced together
        named("batch256_f32", _case("batch", (24, 24, 48), (0.125,) * 3, 40, 0.3, "f32", c=50.0, noise=True,
                                    replicas=256)),
        # large single-device run
        named("large256_f32", _case("evaluate", (256,) * 3, (16.0,) * 3, 200, 0.35, "f32", chin=22.0, c=100.0, sr=0.2,
                                    si=0.05)),
    ]


def _near(rng, e):
    """A supported axis length near e (within a factor of about 1.5)."""
    return rng.choice([a for a in AXES if e / 1.5 <= a <= e * 1.5] or [min(AXES, key=lambda a: abs(a - e))])


def draw(rng):
    call = rng.choices(("evaluate", "step", "gradient", "batch"), (45, 30, 12, 13))[0]
    prec = rng.choice(("f64", "f32"))
    if call == "batch":
        reps = int(round(math.exp(rng.uniform(math.log(8), math.log(256)))))
        return _case("batch", (24, 24, 48), (0.125,) * 3, rng.randint(12, 60), rng.choice((0.25, 0.3, 0.4)), prec,
                     c=50.0, noise=rng.random() < 0.7, replicas=reps if prec == "f32" else max(8, reps // 4),
                     update=rng.choice(("explicit", "semi")))
    edge = math.exp(rng.uniform(math.log(10), math.log(100 if call == "gradient" else 150)))
    if rng.random() < 0.5:
        n = (min((a for a in AXES if a <= 128), key=lambda a: abs(math.log(a / edge))),) * 3
    else:
        n = tuple(_near(rng, edge) for _ in range(3))
        while n[0] * n[1] * n[2] > 128 ** 3:
            n = tuple(_near(rng, 0.8 * a) for a in n)
    dx = rng.uniform(0.07, 0.125)
    L = tuple(round(a * dx * rng.uniform(0.9, 1.1), 3) for a in n)
    ns = int(round(math.exp(rng.uniform(math.log(16), math.log(128)))))
    model = "edwards" if call in ("evaluate", "step") and rng.random() < 0.2 else "diblock"
    walls = ["p", "p", "p"]
    if call != "step" and rng.random() < 0.3:
        walls[rng.randrange(3)] = rng.choice(("r", "a"))
    return _case(call, n, L, ns, rng.choice((0.5, round(rng.uniform(0.2, 0.6), 3))), prec,
                 chin=round(rng.uniform(10.0, 25.0), 2), c=float(rng.choice((1, 10, 50))),
                 scheme="split2" if rng.random() < 0.2 else "rqm4", model=model, b=round(rng.uniform(0.5, 4.0), 2),
                 walls="".join(walls),
                 storage=1 if call == "evaluate" and model == "diblock" and rng.random() < 0.12 else 0,
                 update=rng.choice(("explicit", "semi")) if call == "step" else "explicit",
                 noise=call == "step" and rng.random() < 0.6, dt=round(rng.uniform(0.005, 0.05), 4),
                 sr=round(rng.uniform(0.05, 0.3), 3), si=round(rng.uniform(0.01, 0.06), 3))


# ------------------------------------------------------------------ inputs --

def _replicas(case):
    """The parameter sets of the case: one, or the uneven replicas of a batch."""
    if case["call"] != "batch":
        return [case]
    rng = np.random.default_rng(case["replicas"] + case["ns"])
    out = []
    for _ in range(case["replicas"]):
        n = int(rng.choice([24, 32, 40, 48]))
        ns = int(rng.integers(case["ns"], 2 * case["ns"] + 1))
        out.append(dict(case, call="step", nx=n, ny=n, nz=n, lx=0.125 * n, ly=0.125 * n, lz=0.125 * n, ns=ns,
                        chin=float(rng.uniform(12.0, 25.0)), f=float(rng.uniform(case["f"], case["f"] + 0.2))))
    return out


def _shape(case):
    return case["nx"], case["ny"], case["nz"]


def _volume(case):
    return case["lx"] * case["ly"] * case["lz"]


def _params(case):
    bc = tuple({"p": B.PFT_PERIODIC, "r": B.PFT_REFLECTING, "a": B.PFT_ABSORBING}[w] for w in case["walls"])
    return B.Params(*_shape(case), case["lx"], case["ly"], case["lz"], case["ns"], case["f"], case["chin"], case["c"],
                    B.PFT_C128 if case["prec"] == "f64" else B.PFT_C64,
                    B.PFT_RQM4 if case["scheme"] == "rqm4" else B.PFT_SPLIT2,
                    B.PFT_EDWARDS if case["model"] == "edwards" else B.PFT_DIBLOCK,
                    case["b"] if case["model"] == "edwards" else 0.0, case["storage"], bc)


def _fields(case, seed):
    """w_plus and w_minus of every replica, each one flat tensor: randomly
    seeded complex fields (a lamellar profile added to w_minus if asked)."""
    reps = _replicas(case)
    sizes = [math.prod(_shape(r)) for r in reps]
    g = torch.Generator(device=DEV).manual_seed(seed)
    real = case["si"] == 0.0
    out = []
    for k in range(2):
        w = torch.zeros(sum(sizes), dtype=torch.complex128, device=DEV)
        v = torch.view_as_real(w)
        if real:  # fields of a real saddle point: i w_plus and w_minus real
            v[:, 1 - k] = case["sr"] * torch.randn(w.numel(), generator=g, dtype=torch.float64, device=DEV)
        else:
            v[:, 0] = case["sr"] * torch.randn(w.numel(), generator=g, dtype=torch.float64, device=DEV)
            v[:, 1] = case["si"] * torch.randn(w.numel(), generator=g, dtype=torch.float64, device=DEV)
        out.append(w)
    if case["cosine"]:
        x = torch.arange(case["nx"], dtype=torch.float64, device=DEV) / case["nx"]
        out[1].view(_shape(case)).add_((case["cosine"] * torch.cos(2 * math.pi * x)).view(-1, 1, 1))
    return out[0], out[1], sizes


def _views(flat, case):
    parts, at = [], 0
    for r in _replicas(case):
        m = math.prod(_shape(r))
        parts.append(flat[at:at + m].view(_shape(r)))
        at += m
    return parts


def _steps(case, seed, number):
    return B.pft_step(case["dt"], 1.0, 1.0, seed, 0, number, int(case["noise"]), int(case["update"] == "semi"))


def prepare(case, seed):
    wp, wm, _ = _fields(case, seed)
    s = dict(case=case, seed=seed, number=0, wp=wp, wm=wm)
    if case["call"] == "batch":
        s["handle"] = B.Batch([_params(r) for r in _replicas(case)])
        s["fields"] = (_views(wp, case), _views(wm, case))
        s["log"] = torch.zeros((1, case["replicas"], 2), dtype=torch.complex128, device=DEV)
        return s
    s["handle"] = B.Context(_params(case))
    shape = _shape(case)
    s["fields"] = (wp.view(shape), None if case["model"] == "edwards" else wm.view(shape))
    s["out"] = [torch.zeros(shape, dtype=torch.complex128, device=DEV) for _ in range(2)]
    s["scal"] = [torch.zeros(1, dtype=torch.complex128, device=DEV) for _ in range(2)]
    s["dL"] = torch.zeros(3, dtype=torch.complex128, device=DEV)
    return s


# -------------------------------------------------------------------- runs --

def run(s):
    case, h = s["case"], s["handle"]
    wp, wm = s["fields"]
    f64 = case["prec"] == "f64"

    def keep(t):
        return t if f64 else t.to(torch.complex64)

    if case["call"] == "evaluate":
        o = h.evaluate(wp, wm)
        r = {"phiA": keep(o["phiA"]), "phiB": keep(o["phiB"]), "Q": keep(o["Q"])}
        if f64:
            r["H"] = o["H"]
        return r
    if case["call"] == "step":
        (pa, pb), (Q, H) = s["out"], s["scal"]
        h.pft_cl_step(wp, wm, _steps(case, s["seed"], s["number"]), pa, pb, Q, H)
        s["number"] += 1
        r = {"w_plus": keep(wp), "phiA": keep(pa), "phiB": keep(pb), "Q": keep(Q)}
        if wm is not None:
            r["w_minus"] = keep(wm)
        if f64:
            r["H"] = H
        return r
    if case["call"] == "gradient":
        (gp, gm), (_, H) = s["out"], s["scal"]
        if f64:
            h.pft_adjoint(wp, wm, gp, gm, s["dL"], H)
            return {"dwp": gp, "dwm": gm, "dL": s["dL"], "H": H}
        h.pft_adjoint(wp, wm, gp, gm)
        return {"dwp": keep(gp), "dwm": keep(gm)}
    h.pft_batch_cl_steps(wp, wm, _steps(case, s["seed"], s["number"]), 1, s["log"])
    s["number"] += 1
    return {"w_plus": keep(s["wp"]), "w_minus": keep(s["wm"]), "Q": keep(s["log"][:, :, 0])}


def work(case):
    """The least a pass does: fields read and results written (complex
    double), q written at every contour node and read back once (the contour
    sums pair its nodes with q-dagger's in reverse order), and the line
    transforms of every contour step (5 N log2 N a transform, two a diffusion)."""
    total = {"bytes": 0.0, "flops": 0.0}
    for r in _replicas(case):
        n = _shape(r)
        M, K = math.prod(n), r["ns"]
        c = 16 if r["prec"] == "f64" else 8
        sweeps = 1 if r["model"] == "edwards" else 2
        arrays = 3 if r["scheme"] == "rqm4" else 1
        if r["call"] == "gradient":
            total["bytes"] += M * (64.0 + 2 * c * K)
            sweeps = 4  # forward and adjoint vectors and, for the box, one more transform pair each
        else:
            total["bytes"] += M * ((64.0 if r["call"] == "evaluate" else 128.0) + 2 * c * (K + 1))
        total["flops"] += sweeps * K * M * (arrays * 10 * sum(math.log2(a) for a in n) + 24 * arrays)
    return total


# ------------------------------------------------------------------- exact --
# Complex fields as real tensors (2, nx, ny, nz); diffusions as real matrices.

def _mul(a, b):
    return torch.stack((a[0] * b[0] - a[1] * b[1], a[0] * b[1] + a[1] * b[0]))


def _modes(n, wall, dev):
    """Orthonormal real modes (n, n) of one axis and their k L."""
    x = torch.arange(n, dtype=torch.float64, device=dev)
    if wall == "p":
        cols, k = [torch.full((n,), 1.0, dtype=torch.float64, device=dev)], [0.0]
        for m in range(1, (n + 1) // 2):
            ph = 2 * math.pi * ((m * x) % n) / n
            cols += [torch.cos(ph), torch.sin(ph)]
            k += [2 * math.pi * m] * 2
        cols.append(torch.cos(math.pi * x))  # n is even
        k.append(math.pi * n)
    else:
        ms = range(n) if wall == "r" else range(1, n + 1)
        fn = torch.cos if wall == "r" else torch.sin
        cols = [fn(math.pi * (((2 * x + 1) * m) % (4 * n)) / (2 * n)) for m in ms]
        k = [math.pi * m for m in ms]
    V = torch.stack(cols, 1)
    return V / V.norm(dim=0, keepdim=True), torch.tensor(k, dtype=torch.float64, device=dev)


class _Exact:
    def __init__(self, case, dev, L=None):
        self.case, self.dev, self.n = case, dev, _shape(case)
        self.M = math.prod(self.n)
        self.L = torch.tensor([case["lx"], case["ly"], case["lz"]], dtype=torch.float64, device=dev) if L is None else L
        self.modes = [_modes(n, w, dev) for n, w in zip(self.n, case["walls"])]
        self.edwards = case["model"] == "edwards"
        ns, f = case["ns"], case["f"]
        ds, fn = 1.0 / ns, case["f"] * ns
        if self.edwards:
            self.plan = [(ds, 0)] * ns
        elif abs(fn - round(fn)) <= 1e-9:
            self.plan = [(ds, 0 if j < round(fn) else 1) for j in range(ns)]
        else:
            a = math.floor(fn)
            self.plan = [(ds, 0)] * a + [(f - a * ds, 0), ((a + 1) * ds - f, 1)] + [(ds, 1)] * (ns - a - 1)
        self.K = len(self.plan)
        self.mats = {}

    def matrices(self, h):
        if h not in self.mats:
            out = []
            for a, (V, k) in enumerate(self.modes):
                out.append((V * torch.exp(-(k / self.L[a]) ** 2 * h)) @ V.T)
            self.mats[h] = out
        return self.mats[h]

    def diffuse(self, u, h):
        nx, ny, nz = self.n
        Dx, Dy, Dz = self.matrices(h)
        u = (u.reshape(-1, nz) @ Dz).view(2 * nx, ny, nz)
        u = torch.matmul(Dy, u)
        return torch.matmul(Dx, u.reshape(2, nx, ny * nz)).view(2, nx, ny, nz)

    def tables(self, wp, wm):
        """exp(-w h/4) per (h, block); w_A = i w+ - w-, w_B = i w+ + w-."""
        w = {0: torch.stack((-wp[1] - wm[0], wp[0] - wm[1])), 1: torch.stack((-wp[1] + wm[0], wp[0] + wm[1]))}
        self.E = {}
        for h, blk in set(self.plan):
            m = torch.exp(-w[blk][0] * h / 4)
            a = -w[blk][1] * h / 4
            self.E[(h, blk)] = torch.stack((m * torch.cos(a), m * torch.sin(a)))

    def step(self, q, j):
        h, blk = self.plan[j]
        e4 = self.E[(h, blk)]
        e2 = _mul(e4, e4)
        full = _mul(e2, self.diffuse(_mul(e2, q), h))
        if self.case["scheme"] == "split2":
            return full
        half = _mul(e4, self.diffuse(_mul(e2, self.diffuse(_mul(e4, q), h / 2)), h / 2))
        return (4 * half - full) / 3

    def one(self):
        q = torch.zeros((2, *self.n), dtype=torch.float64, device=self.dev)
        q[0] = 1.0
        return q

    def evaluate(self, wp, wm):
        self.tables(wp, wm)
        K = self.K
        q = torch.empty((K + 1, 2, *self.n), dtype=torch.float64, device=self.dev)
        q[0] = self.one()
        for j in range(K):
            q[j + 1] = self.step(q[j], j)
        Q = q[K].double().view(2, -1).mean(1)
        tau = [[0.0] * (K + 1), [0.0] * (K + 1)]
        for j, (h, blk) in enumerate(self.plan):
            tau[blk][j] += h / 2
            tau[blk][j + 1] += h / 2
        phi = [torch.zeros_like(wp), torch.zeros_like(wp)]
        qd = self.one()
        for i in range(K + 1):  # node i of q-dagger pairs with node K - i of q
            j = K - i
            p = _mul(q[j], qd)
            for b in range(2):
                if tau[b][j]:
                    phi[b] += tau[b][j] * p
            if i < K:
                qd = self.step(qd, j - 1)
        d = Q[0] ** 2 + Q[1] ** 2
        inv = torch.stack((Q[0] / d, -Q[1] / d)).view(2, 1, 1, 1)
        phi = [_mul(p, inv.expand_as(p)) for p in phi]
        return phi, Q, self.hamiltonian(wp, wm, Q)

    def hamiltonian(self, wp, wm, Q):
        c, V = self.case["c"], self.L.prod()
        if self.edwards:
            s = (self.case["b"] / (2 * c) * _mul(wp, wp)).view(2, -1).sum(1)
        else:
            m2 = _mul(wm, wm) / self.case["chin"]
            s = torch.stack((m2[0] + wp[1], m2[1] - wp[0])).view(2, -1).sum(1)
        logq = torch.stack((0.5 * torch.log(Q[0] ** 2 + Q[1] ** 2), torch.atan2(Q[1], Q[0])))
        return c * V / self.M * s - c * V * logq


def _normals(seed, replica, step, field, M):
    """Standard normals by Box-Muller on Philox4x64-10 words, key (seed,
    replica), counter (site / 4, field, step, 0)."""
    ctr = (field << 64) + (step << 128) - 1  # numpy increments before the first block
    bits = np.random.Philox(key=np.array([seed, replica], dtype=np.uint64), counter=ctr % (1 << 256))
    w = (bits.random_raw(4 * ((M + 3) // 4)) >> np.uint64(11)).astype(np.float64)
    u = (w + 0.5) * 2.0 ** -53
    r, t = np.sqrt(-2.0 * np.log(u[0::2])), 2 * math.pi * u[1::2]
    return np.stack((r * np.cos(t), r * np.sin(t)), 1).reshape(-1)[:M]


def _debye(x):
    s, t = torch.ones_like(x), torch.ones_like(x)
    for m in range(1, 21):
        t = t * (-x / (m + 2))
        s = s + t
    y = torch.clamp(x, min=0.5)
    return torch.where(x < 0.5, s, 2 * (torch.exp(-y) + y - 1) / (y * y))


def _filtered(ex, r, g0, a):
    """Every Fourier mode of r divided by 1 + a (g0 + Debye(|k|^2))."""
    k2 = 0
    for ax, n in enumerate(ex.n):
        m = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=ex.dev)
        k2 = k2 + ((2 * math.pi * m / ex.L[ax]) ** 2).view([-1 if b == ax else 1 for b in range(3)])
    z = torch.fft.fftn(torch.complex(r[0], r[1]))
    return torch.view_as_real(torch.fft.ifftn(z / (1 + a * (g0 + _debye(k2))))).permute(3, 0, 1, 2)


def _stepped(ex, wp, wm, phi, seed, replica):
    """The fields after one step from the densities of these fields."""
    c = ex.case
    a, M = c["dt"], ex.M
    noise = [torch.zeros(ex.n, dtype=torch.float64, device=ex.dev)] * 2
    if c["noise"]:
        s = math.sqrt(2 * a / (c["c"] * _volume(c) / M))
        noise = [s * torch.from_numpy(_normals(seed, replica, 0, f, M)).to(ex.dev).view(ex.n) for f in range(2)]
    tot = phi[0] + phi[1]
    if ex.edwards:
        F = torch.stack((c["b"] / c["c"] * wp[0] - phi[0][1], c["b"] / c["c"] * wp[1] + phi[0][0]))
    else:
        F = torch.stack((-tot[1], tot[0] - 1))
    r = a * F
    r[0] -= noise[0]
    rm = a * (2 / c["chin"] * wm + phi[1] - phi[0])
    rm[0] -= noise[1]
    if c["update"] == "semi":
        r = _filtered(ex, r, c["b"] / c["c"] if ex.edwards else 0.0, a)
        rm = rm / (1 + a * 2 / c["chin"])
    return wp - r, wm - rm


def _planes(t, shape):
    """A complex field as a real tensor (2, nx, ny, nz)."""
    return torch.view_as_real(t.view(shape)).permute(3, 0, 1, 2).contiguous()


def _cplx(t):
    return torch.complex(t[0].contiguous(), t[1].contiguous())


def _exact_gradient(case, wp, wm, dev):
    """H is holomorphic in the fields: with w = a + i b, dH/dw is
    d Re H/da - i d Re H/db."""
    L = torch.tensor([case["lx"], case["ly"], case["lz"]], dtype=torch.float64, device=dev, requires_grad=True)
    wp, wm = wp.clone().requires_grad_(), wm.clone().requires_grad_()
    ex = _Exact(case, dev, L)
    ex.tables(wp, wm)
    q = ex.one()
    for j in range(ex.K):
        q = ex.step(q, j)
    H = ex.hamiltonian(wp, wm, q.reshape(2, -1).mean(1))
    f64 = case["prec"] == "f64"
    gp, gm, lr = torch.autograd.grad(H[0], (wp, wm, L), retain_graph=f64)
    out = {"dwp": torch.complex(gp[0], -gp[1]), "dwm": torch.complex(gm[0], -gm[1])}
    if f64:
        out["dL"] = torch.complex(lr, torch.autograd.grad(H[1], L)[0])
        out["H"] = _cplx(H.detach().view(2, 1))
    return out


def exact(case, seed, dev=DEV):
    wp, wm, _ = _fields(case, seed)
    if case["call"] == "gradient":
        return _exact_gradient(case, _planes(wp.to(dev), _shape(case)), _planes(wm.to(dev), _shape(case)), dev)
    parts = []
    with torch.no_grad():
        for i, (r, a, b) in enumerate(zip(_replicas(case), _views(wp, case), _views(wm, case))):
            a, b = _planes(a.to(dev), _shape(r)), _planes(b.to(dev), _shape(r))
            if r["model"] == "edwards":
                b = torch.zeros_like(b)
            ex = _Exact(r, dev)
            phi, Q, H = ex.evaluate(a, b)
            o = {"phiA": _cplx(phi[0]), "phiB": _cplx(phi[1]), "Q": _cplx(Q.view(2, 1)), "H": _cplx(H.view(2, 1))}
            if r["call"] == "step":
                a, b = _stepped(ex, a, b, phi, seed, i)
                o["w_plus"] = _cplx(a)
                if r["model"] != "edwards":
                    o["w_minus"] = _cplx(b)
            if case["prec"] != "f64":
                del o["H"]
            parts.append(o)
    if case["call"] != "batch":
        return parts[0]
    return {"w_plus": torch.cat([p["w_plus"].view(-1) for p in parts]),
            "w_minus": torch.cat([p["w_minus"].view(-1) for p in parts]),
            "Q": torch.cat([p["Q"] for p in parts]).view(1, -1)}
