"""Performance cases of the CDUGKS step.

A case is one piece of work a program gives the library between two looks at
its results: so many time steps of one problem and its moments (``solo``), the
same for a batch of uneven problems (``batch``), requests through the solve
server (``served``), or a velocity-grid refit and the steps after it
(``refit``).  Problems come from ``workloads.py`` with a seeded smooth
disturbance, so that every seed is another state.

``exact`` steps the same problems with plain torch in FP64 on whole arrays of
a block of velocities at a time, following the scheme's equations directly
(Sec. 2 and 2.1 of the paper): ghost layers, limited slopes, face values,
inversion, fluxes, update.
"""
from __future__ import annotations

import ctypes
import math
import time

import numpy as np
import torch

from paper_2208_09132_amd import cdugks as cd
from paper_2208_09132_amd import workloads as wl

# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------


def _case(kind, flow, n, nv, storage, steps, **kw):
    c = dict(kind=kind, flow=flow, dim=len(n), storage=storage, steps=steps)
    for d in range(3):
        c["n%d" % d] = n[d] if d < len(n) else 1
        c["nv%d" % d] = nv[d] if d < len(nv) else 1
    c.update(reconstruction="slopes_of_slopes", **kw)
    return c


def listed():
    return [
        # the smallest run: the benchmark's Sod tube, a step of which is little
        # more than its launches
        dict(_case("solo", "sod", [128], [64], "f64", 64), name="sod_128x64"),
        # the paper's Sod validation set-up at its sizes: Dirichlet ends, Boole
        # weights, one velocity axis much longer than a 2-D problem's
        dict(_case("solo", "sod_validation", [1024], [1025], "f64", 32), name="sod_validation_1024x1025"),
        # the paper's sine-wave problem: few cells, a very fine velocity grid
        dict(_case("solo", "sine", [128], [16385], "f64", 16), name="sine_128x16385"),
        # an ordinary small 2-D run of an odd size
        dict(_case("solo", "kh", [41, 41], [13, 13], "f64", 50), name="kh_41x41_v13x13"),
        # the headline workload, FP64 storage
        dict(_case("solo", "kh", [256, 256], [28, 28], "f64", 8), name="kh_256x256_v28x28"),
        # the same in FP32 storage
        dict(_case("solo", "kh", [256, 256], [28, 28], "f32", 8), name="kh_256x256_v28x28_f32"),
        # a ragged 2-D vortex of the served stream's middle sizes with the far
        # velocity tails in BF16
        dict(_case("solo", "vortex", [191, 191], [21, 21], "f32_bf16tail", 10), name="vortex_191x191_v21x21_tail"),
        # the 3-D workload in its storage form
        dict(_case("solo", "shear", [64, 64, 64], [16, 16, 16], "f32", 2), name="shear_64cube_v16cube_f32"),
        # a ragged 3-D box with outflow sides in FP64
        dict(_case("solo", "box", [37, 29, 23], [11, 10, 12], "f64", 6), name="box_37x29x23_v11x10x12"),
        # uneven 1-D and 2-D problems advanced together
        dict(_case("batch", "uneven", [1], [1], "f32", 10, count=20), name="batch_20_uneven_f32"),
        # solves through the server, set-up, admission and read-out included
        dict(_case("served", "stream", [1], [1], "f32", 100, count=6), name="served_6_f32"),
        # an adaptive velocity grid: the state refit onto a finer grid, then
        # a few steps on it
        dict(_case("refit", "kh", [128, 128], [28, 28], "f64", 4, nvto=32), name="refit_128x128_v28_to_v32"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case of the same ranges.  Steps are chosen so that a small
    problem runs many and a large one few, as programs do between outputs."""
    kind = rng.choice(["solo"] * 15 + ["batch"] * 2 + ["served"] + ["refit"] * 2)
    if kind == "batch":
        return _case("batch", "uneven", [1], [1], rng.choice(["f32", "f32", "f64", "f32_bf16tail"]),
                     rng.randint(2, 10), count=rng.randint(3, 20), first=rng.randint(0, 200))
    if kind == "served":
        return _case("served", "stream", [1], [1], rng.choice(["f32", "f64"]), rng.randint(30, 100),
                     count=rng.randint(2, 5), first=rng.randint(1, 200))
    if kind == "refit":
        nv = rng.randint(14, 28)
        return _case("refit", rng.choice(["kh", "vortex"]), [_log_int(rng, 40, 200)] * 2, [nv, nv],
                     rng.choice(["f64", "f32"]), rng.randint(1, 6), nvto=rng.randint(14, 32))
    storage = rng.choice(["f64", "f64", "f32", "f32", "f32_bf16tail"])
    dim = rng.choice([1, 1, 2, 2, 2, 3, 3])
    if dim == 1:
        flow = rng.choice(["sod", "sod_validation", "sine", "fourier", "atmosphere"])
        n = [_log_int(rng, 64, 2048)]
        nv = [4 * _log_int(rng, 16, 4096 if flow == "sine" else 300) + 1 if flow in ("sod_validation", "sine")
              else _log_int(rng, 32, 1024)]
    elif dim == 2:
        flow = rng.choice(["kh", "kh", "vortex", "fourier", "atmosphere"])
        n = [_log_int(rng, 32, 320), _log_int(rng, 32, 320)]
        if flow in ("kh", "vortex"):
            n[1] = n[0]
        nv = [rng.randint(12, 32), rng.randint(12, 32)]
        if flow in ("kh", "vortex"):
            nv[1] = nv[0]
    else:
        flow = rng.choice(["shear", "box", "fourier"])
        n = [rng.randint(12, 56) for _ in range(3)]
        nv = [rng.randint(6, 16) for _ in range(3)]
        if flow == "shear":
            n, nv = [n[0]] * 3, [nv[0]] * 3
    points = int(np.prod(n)) * int(np.prod(nv))
    steps = max(2, min(rng.choice([20, 50, 64, 100]), int(1.2e9 / points)))
    c = _case("solo", flow, n, nv, storage, steps)
    if flow != "atmosphere" and rng.random() < 0.2:
        c["reconstruction"] = "single_slope"
    return c


# ---------------------------------------------------------------------------
# problems
# ---------------------------------------------------------------------------


def _disturb(p, seed, amp=0.02):
    """A smooth seeded disturbance of density and temperature."""
    rng = wl.SplitMix64(0x9E37 + 7919 * int(seed))
    x = wl.cell_centres(p["dim"], p["n"], [0.0] * p["dim"], [1.0] * p["dim"])
    p["rho"] = p["rho"] * (1.0 + amp * wl.random_fourier_field(rng, p["dim"], x))
    p["T"] = p["T"] * (1.0 + amp * wl.random_fourier_field(rng, p["dim"], x))
    return p


def _atmosphere(dim, n, nv, storage):
    """A column of gas at rest under gravity along the last axis, between
    Dirichlet sides holding its hydrostatic ends, periodic across."""
    a, RT = 0.3, 0.5
    x = wl.cell_centres(dim, n, [0.0] * dim, [1.0] * dim)
    rho = np.exp(-a * x[-1] / RT)
    rest = [0.0] * dim
    acc = [0.0] * dim
    acc[-1] = -a
    lo, hi = [1.0] + rest + [1.0], [math.exp(-a / RT)] + rest + [1.0]
    return dict(dim=dim, n=list(n), lo=[0.0] * dim, hi=[1.0] * dim, bc=["periodic"] * (dim - 1) + ["dirichlet"],
                dirichlet=[None] * (dim - 1) + [[lo, hi]], nv=list(nv), vmin=[-5.0] * dim, vmax=[5.0] * dim,
                quad="trapezoid", gamma=5.0 / 3.0, Pr=2.0 / 3.0, R=0.5, omega=0.5, relax="kn", Kn=1e-2, T_ref=1.0,
                cfl=0.5, storage=storage, rho=rho, u=np.zeros((dim, rho.size)), T=np.ones(rho.size), accel=acc)


def _problems(case, seed):
    """The problems of a case (one, or a batch's or the server's several) and
    the steps each is to run."""
    dim, st, steps = case["dim"], case["storage"], case["steps"]
    n = [case["n%d" % d] for d in range(dim)]
    nv = [case["nv%d" % d] for d in range(dim)]
    flow = case["flow"]
    if flow == "uneven":
        ps = wl.batched(count=case.get("first", 0) + case["count"], storage=st)[case.get("first", 0):]
        return [_disturb(p, 100 * seed + k) for k, p in enumerate(ps)], [steps] * len(ps)
    if flow == "stream":
        # the served stream's two flows at the smaller of its sizes
        rng = wl.SplitMix64(913 + case.get("first", 0))
        ps, ns = [], []
        for k in range(case["count"]):
            m, v = rng.integer(64, 160), rng.integer(16, 24)
            Kn = 10.0 ** rng.uniform(-4.0, 0.0)
            p = wl.vortex(m, v, Kn=Kn, storage=st) if k % 2 else wl.random_fourier(2, [m, m], [v, v], rng, Kn=Kn,
                                                                                   storage=st)
            ps.append(_disturb(p, 100 * seed + k))
            ns.append(rng.integer(max(10, steps // 2), steps))
        return ps, ns
    if flow == "sod":
        p = wl.sod(n[0], nv[0], storage=st)
    elif flow == "sod_validation":
        p = wl.sod_validation(n[0], nv[0], storage=st)
    elif flow == "sine":
        p = wl.sine_wave(n[0], nv[0], storage=st)
    elif flow == "kh":
        p = wl.kelvin_helmholtz(n[0], nv[0], seed=2208 + int(seed), storage=st)
    elif flow == "vortex":
        p = wl.vortex(n[0], nv[0], Kn=1e-2, storage=st)
    elif flow == "shear":
        p = wl.shear3d(n[0], nv[0], storage=st)
    elif flow == "atmosphere":
        p = _atmosphere(dim, n, nv, st)
    else:
        p = wl.random_fourier(dim, n, nv, wl.SplitMix64(5 + int(seed)), Kn=1e-2, storage=st)
        if flow == "box":
            p["bc"] = ["outflow", "periodic", "outflow"]
    p["reconstruction"] = case["reconstruction"]
    return [_disturb(p, seed)], [steps]


def prepare(case, seed):
    probs, steps = _problems(case, int(seed))
    kind = case["kind"]
    if kind == "served":
        srv = cd.Server(int(64e9), max_active=8, chunk_steps=50)
        return dict(kind=kind, server=srv, probs=probs, steps=steps)
    if kind == "batch":
        stream = torch.cuda.Stream()
        solvers = [cd.Solver(p, use_torch=True, stream=ctypes.c_void_p(stream.cuda_stream)) for p in probs]
        state = dict(kind=kind, stream=stream, solvers=solvers, batch=cd.Batch(solvers, chunk_steps=case["steps"]))
    else:
        solvers = [cd.Solver(probs[0], use_torch=True)]
        state = dict(kind=kind, solvers=solvers)
    state["steps"] = case["steps"]
    if kind == "refit":
        # the state to refit has left its initial equilibrium
        solvers[0].step(4)
        solvers[0].sync()
        state["to"] = dict(probs[0], nv=[case["nvto"]] * case["dim"])
        return state
    state["moments"] = [(torch.empty(s.N, dtype=torch.float64, device="cuda"),
                         torch.empty((s.D, s.N), dtype=torch.float64, device="cuda"),
                         torch.empty(s.N, dtype=torch.float64, device="cuda")) for s in solvers]
    torch.cuda.synchronize()
    return state


def run(state):
    kind = state["kind"]
    if kind == "served":
        srv = state["server"]
        tickets = [srv.submit(p, n) for p, n in zip(state["probs"], state["steps"])]
        out = [None] * len(tickets)
        while any(r is None for r in out):
            for k, t in enumerate(tickets):
                if out[k] is None:
                    r = srv.poll(t)
                    out[k] = None if r is None else r[:3]
            time.sleep(0.0005)
        return out
    if kind == "refit":
        s = state["solvers"][0].regrid(state["to"])
        s.step(state["steps"])
        out = s.moments()
        s.close()
        return out
    if kind == "batch":
        state["batch"].step(state["steps"])
    else:
        state["solvers"][0].step(state["steps"])
    for s, (rho, u, T) in zip(state["solvers"], state["moments"]):
        s.moments_device(rho.data_ptr(), u.data_ptr(), T.data_ptr())
    return state["moments"]


# ---------------------------------------------------------------------------
# the least work of a pass
# ---------------------------------------------------------------------------


def work(case):
    """Bytes: per step, g and b of every (cell, velocity) read once and
    written once, and the moments written at the end.  Operations per (cell,
    velocity) and step: the limited slopes and slopes of slopes (5 each), D
    face values of two fields, 2D+3 velocity sums per face, one equilibrium
    and inversion per face and two per cell."""
    probs, steps = _problems(case, 1)
    nbytes = flops = 0.0
    for p, s in zip(probs, steps):
        D, N, V = p["dim"], int(np.prod(p["n"])), int(np.prod(p["nv"]))
        es = 8 if p["storage"] == "f64" else 4
        lim = 2 * D * 5 + (0 if p.get("reconstruction") == "single_slope" else 2 * D * D * 5)
        per = lim + 2 * D * (2 + 4 * D) + 2 * D * (2 * D + 3) + 14 + 20 * D + 40
        if case["kind"] == "refit":
            Vn = case["nvto"] ** D
            nbytes += 2 * es * N * (V + Vn) + 4 * es * N * Vn * s
            flops += N * Vn * (20.0 * (1 + 2 ** D) + per * s)
        else:
            nbytes += 4 * es * N * V * s
            flops += float(per) * N * V * s
        nbytes += 8 * N * (D + 2)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# the same steps in FP64 with plain torch
# ---------------------------------------------------------------------------


class _Plain:
    """One problem's state: W [D+2][cells], g and b [V][cells], the cells as
    axes (z, y, x)."""

    def __init__(self, p, dev):
        self.p, self.dev, self.D = p, dev, p["dim"]
        D = self.D
        self.n = [int(p["n"][d]) for d in range(D)]
        self.shape = self.n[::-1]
        self.R, self.gamma, self.Pr = p.get("R", 0.5), p.get("gamma", 5.0 / 3.0), p.get("Pr", 2.0 / 3.0)
        self.cint = 3.0 - D + (5.0 - 3.0 * self.gamma) / (self.gamma - 1.0)
        self.omega = p.get("omega", 0.5)
        self.acc = [float(a) for a in (p.get("accel") or [0.0] * D)]
        if p.get("relax", "kn") == "kn":
            L = p.get("L_ref") or p["hi"][0] - p["lo"][0]
            rho_ref = p.get("rho_ref") or float(np.mean(p["rho"]))
            self.T_ref = p.get("T_ref") or 1.0
            self.mu = 5.0 / 16.0 * p["Kn"] * L * rho_ref * math.sqrt(2.0 * math.pi * self.R * self.T_ref)
        else:
            self.mu, self.T_ref = p["mu_ref"], p.get("T_ref") or 1.0
        t = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float64), device=dev)
        rho, u, T = t(p["rho"]).reshape(self.shape), t(p["u"]).reshape([D] + self.shape), t(p["T"]).reshape(self.shape)
        E = self.R * T / (self.gamma - 1.0) + 0.5 * (u * u).sum(0)
        self.W = torch.cat([rho[None], rho * u, (rho * E)[None]])
        self.grid(p)
        c = self.prim(self.W)
        self.g, self.b = self.empty(), self.empty()
        for s in self.blocks():
            self.g[s], self.b[s] = self.equilibrium(c, s)

    def empty(self):
        return torch.empty([self.V] + self.shape, dtype=torch.float64, device=self.dev)

    def grid(self, p):
        """Velocity nodes and weights, and the static CFL step."""
        D = self.D
        nodes, wts = [], []
        for d in range(D):
            m = int(p["nv"][d])
            h = (p["vmax"][d] - p["vmin"][d]) / (m - 1)
            nodes.append(p["vmin"][d] + h * np.arange(m))
            w = np.zeros(m)
            if p.get("quad", "trapezoid") == "boole":
                for k in range(0, m - 4, 4):
                    w[k:k + 5] += np.array([7.0, 32.0, 12.0, 32.0, 7.0]) * 2.0 * h / 45.0
            else:
                w[:] = h
                w[0] = w[-1] = 0.5 * h
            wts.append(w)
        self.axes = [torch.as_tensor(x, device=self.dev) for x in nodes]
        mesh = np.meshgrid(*nodes[::-1], indexing="ij")[::-1]
        wm = np.meshgrid(*wts[::-1], indexing="ij")
        col = lambda a: torch.as_tensor(np.ascontiguousarray(a).reshape([-1] + [1] * D), device=self.dev)
        self.xi = [col(m) for m in mesh]
        self.w = col(np.prod(wm, axis=0))
        self.hx2 = 0.5 * sum(x * x for x in self.xi)
        self.V = int(np.prod([len(x) for x in nodes]))
        self.dx = [(p["hi"][d] - p["lo"][d]) / self.n[d] for d in range(D)]
        xm = math.sqrt(sum(max(p["vmin"][d] ** 2, p["vmax"][d] ** 2) for d in range(D)))
        self.dt = p.get("dt") or p.get("cfl", 0.5) * min(self.dx) / (2.0 * xm)

    def blocks(self):
        size = max(1, int(3e7) // int(np.prod(self.n)))
        return [slice(a, min(self.V, a + size)) for a in range(0, self.V, size)]

    def prim(self, W):
        """Primitives at cells or faces from (rho, rho u, rho E)."""
        rho, u = W[0], W[1:1 + self.D] / W[0]
        T = (self.gamma - 1.0) / self.R * (W[-1] / rho - 0.5 * (u * u).sum(0))
        RT = self.R * T
        tau = self.mu * (T / self.T_ref) ** self.omega / (rho * RT)
        return dict(rho=rho, u=u, RT=RT, ig=1.0 / tau, ib=self.Pr / tau, ibg=(self.Pr - 1.0) / tau,
                    hu2=0.5 * (u * u).sum(0))

    def equilibrium(self, c, s):
        c2 = sum((self.xi[d][s] - c["u"][d]) ** 2 for d in range(self.D))
        g = c["rho"] * (2.0 * math.pi * c["RT"]) ** (-0.5 * self.D) * torch.exp(-0.5 * c2 / c["RT"])
        return g, (self.hx2[s] + 0.5 * self.cint * c["RT"]) * g

    def source(self, c, s, g, geq, beq):
        """S_g and S_b at one time (eqs. gsource, bsource)."""
        Z = sum(self.xi[d][s] * c["u"][d] for d in range(self.D)) - c["hu2"]
        Sb = Z * (g - geq) * c["ibg"]
        if not any(self.acc):
            return None, Sb
        ax = sum(self.acc[d] * self.xi[d][s] for d in range(self.D))
        f = (ax - sum(self.acc[d] * c["u"][d] for d in range(self.D))) / c["RT"]
        return f * geq, Sb + ax * (g - geq) + f * beq

    def pad(self, q, s, field):
        """Three ghost layers on every axis."""
        for d in range(self.D):
            n, bc, ax = self.n[d], self.p["bc"][d], -1 - d
            j = torch.arange(-3, n + 3, device=self.dev)
            q = q.index_select(q.dim() + ax, j % n if bc == "periodic" else j.clamp(0, n - 1))
            if bc == "dirichlet":
                for side in range(2):
                    st = [float(v) for v in self.p["dirichlet"][d][side]]
                    one = lambda v: torch.tensor(v, dtype=torch.float64, device=self.dev).reshape([1] * self.D)
                    u = torch.stack([one(v) for v in st[1:1 + self.D]])
                    c = dict(rho=one(st[0]), u=u, RT=one(self.R * st[-1]))
                    geq, beq = self.equilibrium(c, s)
                    v = (geq, beq)[field]
                    if any(self.acc):
                        f = sum(self.acc[e] * (self.xi[e][s] - u[e]) for e in range(self.D)) / c["RT"]
                        v = v + 0.25 * self.dt * f * v
                    q.narrow(q.dim() + ax, 0 if side == 0 else n + 3, 3).copy_(v)
        return q

    @staticmethod
    def van_leer(a, b):
        p = a * b
        return torch.where(p > 0, 2.0 * p / torch.where(p > 0, a + b, torch.ones_like(p)), torch.zeros_like(p))

    def face_values(self, s, c):
        """phi_bar at the left faces (index 0..n_d along d) of both fields:
        [d][field]."""
        D, dt = self.D, self.dt
        g, b = self.g[s], self.b[s]
        geq, beq = self.equilibrium(c, s)
        Sg, Sb = self.source(c, s, g, geq, beq)
        h2 = 0.25 * dt
        q = [g + h2 * c["ig"] * (geq - g), b + h2 * (c["ib"] * (beq - b) + Sb)]
        if Sg is not None:
            q[0] = q[0] + h2 * Sg
        del geq, beq, Sg, Sb
        single = self.p.get("reconstruction") == "single_slope"
        out = [[None, None] for _ in range(D)]
        for f in range(2):
            Q = self.pad(q[f], s, f)
            # cells -2..n+1 along every axis
            cut = lambda a, ax, lo, size: a.narrow(a.dim() - 1 - ax, lo, size)
            inner = lambda a, skip=-1: self._cut_all(a, skip)
            slopes = []
            for e in range(D):
                q1 = inner(Q, e)
                m = q1.shape[q1.dim() - 1 - e] - 2
                mid = cut(q1, e, 1, m)
                slopes.append(self.van_leer(mid - cut(q1, e, 0, m), cut(q1, e, 2, m) - mid))
            Qi = inner(Q)
            del Q
            for d in range(D):
                # upwind cells -1..n along d (offset 1 in the -2..n+1 box),
                # the domain's own cells across
                def at(a, shift):
                    for e in range(D):
                        a = cut(a, e, 1 + shift, self.n[d] + 2) if e == d else cut(a, e, 2, self.n[e])
                    return a
                a0, bsl = [at(a, 0) for a in slopes], []
                for e in range(D):
                    bsl.append(None if single else self.van_leer(a0[e] - at(slopes[e], -1), at(slopes[e], 1) - a0[e]))
                sides = []
                for sg in (1.0, -1.0):
                    v = at(Qi, 0) + 0.5 * sg * a0[d]
                    for e in range(D):
                        lam = 0.5 * dt * self.xi[e][s] / self.dx[e]
                        v = v - lam * (a0[e] if single else a0[e] + 0.5 * sg * bsl[e])
                    # from the left: upwind cells -1..n-1; from the right: 0..n
                    sides.append(cut(v, d, 0 if sg > 0 else 1, self.n[d] + 1))
                x = self.xi[d][s]
                out[d][f] = torch.where(x > 0, sides[0], torch.where(x < 0, sides[1], 0.5 * (sides[0] + sides[1])))
        return out

    def _cut_all(self, a, skip):
        """The -2..n+1 box of a padded field; along `skip` the whole -3..n+2."""
        for e in range(self.D):
            if e != skip:
                a = a.narrow(a.dim() - 1 - e, 1, self.n[e] + 4)
        return a

    def at_face(self, d, s, cf, vg, vb):
        """g and b at the face from phi_bar (eq. phibar inverted)."""
        h2 = 0.25 * self.dt
        geq, beq = self.equilibrium(cf, s)
        Z = sum(self.xi[e][s] * cf["u"][e] for e in range(self.D)) - cf["hu2"]
        sg = sb = 0.0
        ax = 0.0
        if any(self.acc):
            ax = sum(self.acc[e] * self.xi[e][s] for e in range(self.D))
            f = (ax - sum(self.acc[e] * cf["u"][e] for e in range(self.D))) / cf["RT"]
            sg, sb = f * geq, f * beq
        g = (vg + h2 * (cf["ig"] * geq + sg)) / (1.0 + h2 * cf["ig"])
        b = (vb + h2 * (cf["ib"] * beq + (Z * cf["ibg"] + ax) * (g - geq) + sb)) / (1.0 + h2 * cf["ib"])
        return g, b

    def step(self):
        D, dt, w = self.D, self.dt, self.w
        c0 = self.prim(self.W)
        bl = self.blocks()
        total = lambda a: a.sum(0)
        # face W from the velocity sums of phi_bar
        Wf = [0.0] * D
        keep = []
        keep_all = self.V * int(np.prod(self.n)) * 16 * D < 6e9
        for s in bl:
            fv = self.face_values(s, c0)
            for d in range(D):
                vg = w[s] * fv[d][0]
                Wf[d] = Wf[d] + torch.stack([total(vg)] + [total(self.xi[e][s] * vg) for e in range(D)] +
                                            [total(w[s] * fv[d][1])])
            keep.append(fv if keep_all else None)
        cf = []
        for d in range(D):
            if any(self.acc):
                rho, mom = Wf[d][0].clone(), Wf[d][1:1 + D].clone()
                for e in range(D):
                    mom[e] += 0.25 * dt * rho * self.acc[e]
                E = Wf[d][-1] + 0.25 * dt * sum(mom[e] * self.acc[e] for e in range(D))
                Wf[d] = torch.cat([rho[None], mom, E[None]])
            cf.append(self.prim(Wf[d]))
        # fluxes of W and of every velocity
        W1 = self.W.clone()
        for k, s in enumerate(bl):
            fv = keep[k] or self.face_values(s, c0)
            for d in range(D):
                gf, bf = self.at_face(d, s, cf[d], fv[d][0], fv[d][1])
                wx = w[s] * self.xi[d][s]
                G = torch.stack([total(wx * gf)] + [total(wx * self.xi[e][s] * gf) for e in range(D)] +
                                [total(wx * bf)])
                ax = G.dim() - 1 - d
                W1 -= dt / self.dx[d] * (G.narrow(ax, 1, self.n[d]) - G.narrow(ax, 0, self.n[d]))
        if any(self.acc):
            for e in range(D):
                W1[1 + e] += dt * self.W[0] * self.acc[e]
                W1[-1] += dt * self.W[1 + e] * self.acc[e]
        c1 = self.prim(W1)
        for k, s in enumerate(bl):
            fv = keep[k] or self.face_values(s, c0)
            keep[k] = None
            g, b = self.g[s], self.b[s]
            Fg = Fb = 0.0
            for d in range(D):
                gf, bf = self.at_face(d, s, cf[d], fv[d][0], fv[d][1])
                ax = gf.dim() - 1 - d
                sx = self.xi[d][s] / self.dx[d]
                Fg = Fg + sx * (gf.narrow(ax, 1, self.n[d]) - gf.narrow(ax, 0, self.n[d]))
                Fb = Fb + sx * (bf.narrow(ax, 1, self.n[d]) - bf.narrow(ax, 0, self.n[d]))
            geq, beq = self.equilibrium(c0, s)
            Sg, Sb = self.source(c0, s, g, geq, beq)
            ng = g + dt * (0.5 * c0["ig"] * (geq - g) - Fg)
            nb = b + dt * (0.5 * c0["ib"] * (beq - b) - Fb + Sb)
            if Sg is not None:
                ng = ng + dt * Sg
            geq, beq = self.equilibrium(c1, s)
            self.g[s] = (ng + 0.5 * dt * c1["ig"] * geq) / (1.0 + 0.5 * dt * c1["ig"])
            self.b[s] = (nb + 0.5 * dt * c1["ib"] * beq) / (1.0 + 0.5 * dt * c1["ib"])
        self.W = W1

    def refit(self, p):
        """The state on p's velocity grid: W kept, phi = phi_eq plus the old
        grid's departure interpolated linearly along each axis, zero outside
        the old box."""
        c = self.prim(self.W)
        dep = []
        geq, beq = self.equilibrium(c, slice(None))
        for old, eq in ((self.g, geq), (self.b, beq)):
            dep.append(old - eq)
        nvo, axo = [len(a) for a in self.axes], self.axes
        self.grid(p)
        for f in range(2):
            q = dep[f].reshape(nvo[::-1] + [-1])
            for d in range(self.D):
                x, a = self.axes[d], axo[d]
                h = (a[1] - a[0]).item()
                m = torch.clamp(torch.floor((x - a[0]) / h).long(), 0, len(a) - 2)
                t = (x - a[m]) / h
                M = torch.zeros((len(x), len(a)), dtype=torch.float64, device=self.dev)
                r = torch.arange(len(x), device=self.dev)
                M[r, m], M[r, m + 1] = 1.0 - t, t
                M[(x < a[0]) | (x > a[-1])] = 0.0
                k = self.D - 1 - d
                q = torch.movedim(torch.tensordot(M, q, dims=([1], [k])), 0, k)
            dep[f] = q.reshape([self.V] + self.shape)
        geq, beq = self.equilibrium(c, slice(None))
        self.g, self.b = geq + dep[0], beq + dep[1]

    def moments(self):
        c = self.prim(self.W)
        return c["rho"].reshape(-1), c["u"].reshape(self.D, -1), (c["RT"] / self.R).reshape(-1)


def exact(case, seed):
    """What run() returns for these inputs, in FP64 with plain torch; None
    where no GPU is there and the case is not a small one."""
    probs, steps = _problems(case, int(seed))
    gpu = torch.cuda.is_available()
    size = sum(float(np.prod(p["n"])) * float(np.prod(p["nv"])) * s for p, s in zip(probs, steps))
    if not gpu and size > 2e8:
        return None
    out = []
    for p, s in zip(probs, steps):
        x = _Plain(p, "cuda" if gpu else "cpu")
        if case["kind"] == "refit":
            for _ in range(4):
                x.step()
            x.refit(dict(p, nv=[case["nvto"]] * case["dim"]))
        for _ in range(s):
            x.step()
        out.append(x.moments())
    return out[0] if case["kind"] == "refit" else out
