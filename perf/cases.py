"""The sweeps that the speed of this package is judged by.

A case is one design evaluation as an optimisation program makes it: the LKS
forward sweep of a design, its objective, and (except in a line search) the
ALKS adjoint sweep with the sensitivity. The contexts, workspaces and launch
shapes are set up once per problem, as such a program keeps them over its
thousands of design updates; the step counts are shorter than a converged
run's, which repeats the same launches.

Fields and sensitivities of an FP32 context are handed on in FP32, the
precision they were computed in; those of FP64 and mixed contexts in FP64
(mixed: the sensitivity in FP32, like the adjoint sweep it comes from).

`exact` restates the scheme in plain FP64 torch operations.
"""
import functools
import math
import random

import numpy as np
import torch

from paper_2411_03090_amd import autograd as A
from paper_2411_03090_amd import lks as L
from paper_2411_03090_amd import workloads as W

DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _steady(name, nx, ny, prec, n_fwd, n_adj, tune=False, through="calls", Re=100.0):
    return dict(name=name, kind="steady", nx=nx, ny=ny, prec=prec, n_fwd=n_fwd, n_adj=n_adj,
                tune=tune, through=through, Re=Re)


def listed():
    return [
        # the smallest problem of the workloads (64 x 64, Re = 10), through autograd as a
        # torch optimiser drives it: bound by the length of a step, not by its work
        _steady("steady64_fp64_autograd", 64, 64, "fp64", 2000, 2000, through="autograd", Re=10.0),
        # the paper's heat exchanger (Sec. 3.3), 201 x 201, thermal with a heat source
        dict(name="exchanger201_fp32", kind="exchanger", n=201, prec="fp32", n_fwd=1500,
             n_adj=1500, tune=True),
        # the paper's transient heat sink (Sec. 3.4), 141 x 161, Boussinesq force, exact mode,
        # every level kept
        dict(name="sink141x161_fp32", kind="sink", nx=141, ny=161, prec="fp32", n_steps=800,
             mode="exact", keep=1.0, tune=False),
        # a small ragged unsteady channel in FP64, replaying from checkpoints
        dict(name="thermal203x117_fp64", kind="thermal", nx=203, ny=117, prec="fp64",
             n_steps=400, mode="paper", keep=0.3, tune=False),
        # the benchmark's 512 x 512 design in its headline precision
        _steady("steady512_mixed", 512, 512, "mixed", 800, 800, tune=True),
        # a line search: the objective of a trial design without its gradient, odd sizes
        _steady("linesearch509x263_fp64", 509, 263, "fp64", 1000, 0),
        # the benchmark's unsteady thermal channel, 1024 x 512, checkpointed
        dict(name="thermal1024x512_fp32", kind="thermal", nx=1024, ny=512, prec="fp32",
             n_steps=300, mode="paper", keep=0.25, tune=True),
        # many designs of uneven size in one run (graph replay), steady
        dict(name="batch32_fp32", kind="batch", n=32, lo=128, hi=512, prec="fp32", n_fwd=100,
             n_adj=100, unsteady=False, keep=1.0),
        # ... and unsteady thermal ones, checkpointed
        dict(name="ubatch16_fp32", kind="batch", n=16, lo=128, hi=512, prec="fp32", n_fwd=60,
             n_adj=60, unsteady=True, keep=0.3),
        # a large steady grid
        _steady("steady2048_fp32", 2048, 2048, "fp32", 120, 120, tune=True),
        # a small D3Q19 duct with odd sides in FP64, every level kept
        dict(name="duct97x61x53_fp64", kind="duct", nx=97, ny=61, nz=53, prec="fp64",
             n_steps=60, mode="paper", keep=1.0),
        # the benchmark's D3Q19 duct past a heated block, checkpointed
        dict(name="duct256x128x128_fp32", kind="duct", nx=256, ny=128, nz=128, prec="fp32",
             n_steps=30, mode="paper", keep=0.35),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["steady", "steady", "steady", "exchanger", "sink", "thermal", "thermal",
                       "batch", "duct", "duct"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    tune = rng.random() < 0.5
    # steps: about as much work for each size, within a pass of some tens of milliseconds
    if kind == "steady":
        nx, ny = _log_int(rng, 24, 2048), _log_int(rng, 24, 2048)
        n = max(40, min(1200, int(4e8 / (nx * ny))))
        return dict(kind=kind, nx=nx, ny=ny, prec=rng.choice(["fp32", "fp64", "mixed"]), n_fwd=n,
                    n_adj=rng.choice([0, n, n + 1]), tune=tune,
                    through=rng.choice(["calls", "autograd"]), Re=rng.choice([10.0, 100.0]))
    if kind == "exchanger":
        n = _log_int(rng, 48, 800)
        s = max(40, min(900, int(2e8 / (n * n))))
        return dict(kind=kind, n=n, prec=rng.choice(["fp32", "fp64", "mixed"]), n_fwd=s,
                    n_adj=s + rng.choice([0, 1]), tune=tune)
    if kind in ("sink", "thermal"):
        lo, hi = (48, 400) if kind == "sink" else (48, 1024)
        nx, ny = _log_int(rng, lo, hi), _log_int(rng, lo, hi)
        n = max(40, min(600, int(1.2e8 / (nx * ny))))
        return dict(kind=kind, nx=nx, ny=ny, prec=prec, n_steps=n,
                    mode=rng.choice(["paper", "exact"]) if kind == "thermal" else "exact",
                    keep=rng.choice([1.0, 0.3, 0.15]), tune=tune)
    if kind == "batch":
        lo = _log_int(rng, 32, 128)
        uns = rng.random() < 0.5
        s = rng.randint(30, 60) if uns else rng.randint(60, 120)
        return dict(kind=kind, n=rng.randint(2, 16), lo=lo, hi=min(512, 4 * lo), prec=prec,
                    n_fwd=s, n_adj=s, unsteady=uns, keep=rng.choice([1.0, 0.3]))
    nx, ny, nz = _log_int(rng, 20, 256), _log_int(rng, 16, 128), _log_int(rng, 16, 128)
    n = max(12, min(60, int(6e7 / (nx * ny * nz))))
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, prec=prec, n_steps=n,
                mode=rng.choice(["paper", "exact"]), keep=rng.choice([1.0, 0.35]))


# ---------------------------------------------------------------------------
# problems
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=4)
def _problem(key):
    """Geometry, boundary values and parameters (the design comes from the seed)."""
    c = dict(key)
    kind = c["kind"]
    if kind == "steady":
        return W.steady_channel_uniform(c["nx"], c["ny"], Re=c["Re"], seed=0, n_fwd=c["n_fwd"],
                                        n_adj=max(c["n_adj"], 1))
    if kind == "exchanger":
        return W.heat_exchanger(n=c["n"], seed=0, n_fwd=c["n_fwd"], n_adj=c["n_adj"])
    if kind == "sink":
        wl = W.heat_sink(nx=c["nx"], ny=c["ny"], seed=0, n_steps=c["n_steps"])
    elif kind == "thermal":
        wl = _thermal(c["nx"], c["ny"], 200.0, c["n_steps"])
    else:
        # the heated block starts next to the inlet and the enthalpy-flux plane crosses it,
        # where both the flow and the heat of a short horizon reach
        nx = c["nx"]
        wl = W.heated_block_duct(nx=nx, ny=c["ny"], nz=c["nz"], seed=0, n_steps=c["n_steps"],
                                 block=((3 / nx, max(7, nx // 8) / nx), (0.0, 0.25),
                                        (0.375, 0.625)), probe_col=5)
    wl.adjoint_mode = c["mode"]
    return wl


def _thermal(nx, ny, Re, n):
    """The oscillating thermal channel, its enthalpy-flux column moved from the outlet to
    where the flow of a short horizon reaches."""
    wl = W.unsteady_thermal_channel(nx, ny, Re=Re, seed=0, n_steps=n, period=n / 2.0)
    wl.mask &= np.uint8(255 - W.TAG_PROBE)
    wl.mask[1:-1, min(nx - 2, max(2, n // 8))] |= W.TAG_PROBE
    return wl


def _wl(case):
    return _problem(tuple(sorted((k, v) for k, v in case.items() if k != "name")))


def _batch_problems(case):
    """Uneven designs: the edge lengths span lo..hi, the Reynolds numbers 10..200."""
    out = []
    for d in range(case["n"]):
        rng = random.Random(1000 * case["n"] + d)
        edge = _log_int(rng, case["lo"], case["hi"])
        Re = rng.uniform(10.0, 200.0)
        if case["unsteady"]:
            out.append(_thermal(edge, edge, Re, case["n_fwd"]))
        else:
            out.append(W.steady_channel_uniform(edge, edge, Re=Re, seed=0, n_fwd=case["n_fwd"],
                                                n_adj=case["n_adj"]))
    return out


def _shape(wl):
    nz = getattr(wl, "nz", 1)
    return (nz, wl.ny, wl.nx) if hasattr(wl, "periodic_axes") else (wl.ny, wl.nx)


def _design(wl, seed):
    """clip(0.5 + 0.5 z) of a smooth random field z (features of about 8 nodes); boundary
    nodes are fluid, the held solid keeps gamma = 0."""
    shape = _shape(wl)
    gen = torch.Generator().manual_seed(int(seed))
    if wl.n_nodes <= 64 * 64:  # the small problem's design is independent noise
        g = torch.rand(shape, generator=gen, dtype=torch.float64).to(DEV)
    else:
        coarse = torch.randn([1, 1] + [max(2, s // 8) for s in shape], generator=gen,
                             dtype=torch.float64).to(DEV)
        mode = "trilinear" if len(shape) == 3 else "bilinear"
        z = torch.nn.functional.interpolate(coarse, size=shape, mode=mode, align_corners=True)
        g = (0.5 + 0.7 * z[0, 0]).clamp(0.0, 1.0)
    per = getattr(wl, "periodic_axes", 0)
    for d in range(len(shape)):
        if not (per >> d) & 1:
            dim = len(shape) - 1 - d
            g.select(dim, 0).fill_(1.0)
            g.select(dim, shape[dim] - 1).fill_(1.0)
    if len(shape) == 3:
        g[torch.from_numpy((wl.mask & W.TAG_SOLID) != 0).to(DEV)] = 0.0
    return g.contiguous()


def _budget(wl, prec, n, keep):
    """Device bytes for a `keep` share of the trajectory besides the working arrays."""
    if keep >= 1.0:
        return 0
    r = 8 if prec == "fp64" else 4
    nf = 4 if len(_shape(wl)) == 2 else 5
    return int(wl.n_nodes * r * (nf * keep * (n + 1) + 60)) + (1 << 20)


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    if case["kind"] == "batch":
        s.wls = _batch_problems(case)
        budget = 0
        if case["keep"] < 1.0:
            budget = sum(_budget(w, case["prec"], case["n_fwd"], case["keep"]) for w in s.wls) \
                + 8 * case["n"] * max(w.n_nodes for w in s.wls) * 2
        s.batch = L.Batch(s.wls, precision=case["prec"], mem_budget=budget)
        s.gammas = [_design(w, 977 * seed + d).reshape(-1) for d, w in enumerate(s.wls)]
        s.outs = [torch.empty_like(g) for g in s.gammas]
        return s
    s.wl = wl = _wl(case)
    n = case.get("n_steps", case.get("n_fwd"))
    budget = _budget(wl, case["prec"], n, case["keep"]) if "keep" in case else 0
    s.ctx = L.LKS(wl, precision=case["prec"], mem_budget=budget)
    s.gamma = _design(wl, seed).reshape(-1)
    if case.get("tune"):
        s.ctx.autotune(s.gamma, 50)
    if case.get("through") == "autograd":
        s.gamma.requires_grad_(case["n_adj"] > 0)
    s.dJ = torch.empty_like(s.gamma, requires_grad=False)
    thermal = ["T"] if wl.thermal else []
    s.forward_fields = ["drho", "ux", "uy"] + (["uz"] if len(_shape(wl)) == 3 else []) + thermal
    s.adjoint_fields = ["adj_rho", "adj_vx", "adj_vy"] \
        + (["adj_vz"] if len(_shape(wl)) == 3 else []) + (["adj_theta"] if wl.thermal else [])
    s.fields = {f: torch.empty(wl.n_nodes, dtype=torch.float64, device=DEV)
                for f in s.forward_fields + s.adjoint_fields}
    return s


def run(s):
    case = s.case
    if case["kind"] == "batch":
        J = s.batch.run(s.gammas, s.outs, case["n_fwd"], case["n_adj"])
        cast = (lambda t: t.float()) if case["prec"] == "fp32" else (lambda t: t)
        # at most 64 outputs: the gradients of up to 32 designs, the objectives in one
        return {"J": torch.tensor(J, dtype=torch.float32 if case["prec"] == "fp32"
                                  else torch.float64),
                "dJ": [cast(t) for t in s.outs]}
    ctx, wl = s.ctx, s.wl
    steps = case.get("n_steps", case.get("n_fwd"))
    n_adj = case.get("n_adj", steps)
    out = {}
    if case.get("through") == "autograd":
        s.gamma.grad = None
        J = A.objective(s.gamma, ctx, n_adj if n_adj > 0 else None)
        if n_adj > 0:
            J.backward()
            out["dJ"] = s.gamma.grad
    else:
        ctx.forward(s.gamma, steps)
        J = ctx.objective()
        if n_adj > 0:
            ctx.backward(1.0, s.dJ, n_adj)
            out["dJ"] = s.dJ
    out["J"] = torch.as_tensor(J, dtype=torch.float32 if case["prec"] == "fp32"
                               else torch.float64)
    for f in s.forward_fields + (s.adjoint_fields if n_adj > 0 else []):
        # an unsteady sweep with replays keeps no final forward level
        if wl.mode == W.MODE_UNSTEADY and n_adj > 0 and f in s.forward_fields:
            continue
        out[f] = ctx.read(f, s.fields[f])
    if case["prec"] == "fp64":
        return out
    low = set(out) if case["prec"] == "fp32" else set(s.adjoint_fields) | {"dJ"}
    return {k: v.float() if k in low and isinstance(v, torch.Tensor) else v
            for k, v in out.items()}


# bytes and operations per node of one step, each array of a level read once and each
# written once: state in and out, the design, the frozen or stored state of the adjoint,
# the FP64 sensitivity read and written where it is accumulated. Operations of the plain
# scheme (multiplies and adds).
def _step_cost(thermal, d3, r, unsteady):
    d = 3 if d3 else 2
    nf = 1 + d + (1 if thermal else 0)
    fwd = {"bytes": r * (2 * nf + 1), "flops": (190 if thermal else 120) if not d3
           else (520 if thermal else 340)}
    adj = {"bytes": r * (2 * nf + d + (1 if thermal else 0) + 1) + (16 if unsteady else 0),
           "flops": (210 if thermal else 130) if not d3 else (480 if thermal else 300)}
    return fwd, adj


def work(case):
    if case["kind"] == "batch":
        wls, n, m, uns = _batch_problems(case), case["n_fwd"], case["n_adj"], case["unsteady"]
    else:
        wls = [_wl(case)]
        n = case.get("n_steps", case.get("n_fwd"))
        m = case.get("n_adj", n)
        uns = wls[0].mode == W.MODE_UNSTEADY
    tot = {"bytes": 0.0, "flops": 0.0}
    for wl in wls:
        d3 = len(_shape(wl)) == 3
        rf = 4 if case["prec"] == "fp32" else 8
        ra = 8 if case["prec"] == "fp64" else 4
        f, _ = _step_cost(wl.thermal, d3, rf, uns)
        _, a = _step_cost(wl.thermal, d3, ra, uns)
        for k in tot:
            tot[k] += float(wl.n_nodes) * (n * f[k] + m * a[k])
    return tot


# ---------------------------------------------------------------------------
# the scheme in plain FP64 torch
# ---------------------------------------------------------------------------
def _directions(d):
    """Discrete velocities and weights: D2Q9 or D3Q19."""
    c = [v for v in np.ndindex(*([3] * d))]
    c = np.array(c, dtype=np.int64) - 1
    n = np.abs(c).sum(1)
    c, n = c[n <= 2], n[n <= 2]
    w = {2: {0: 4 / 9, 1: 1 / 9, 2: 1 / 36}, 3: {0: 1 / 3, 1: 1 / 18, 2: 1 / 36}}[d]
    return c, np.array([w[int(k)] for k in n])


class _Exact:
    """Axis a of the lattice is tensor dimension -1 - a."""

    def __init__(self, wl, gamma):
        self.wl, self.shape = wl, _shape(wl)
        self.d = d = len(self.shape)
        self.c, self.w = _directions(d)
        self.n = [self.shape[d - 1 - a] for a in range(d)]
        per = int(getattr(wl, "periodic_axes", 7 if wl.periodic else 0))
        self.per = [bool((per >> a) & 1) for a in range(d)]
        t = lambda x: torch.as_tensor(np.asarray(x), device=DEV)  # noqa: E731
        f64 = lambda x: t(np.asarray(x, dtype=np.float64))  # noqa: E731
        self.mask = t(wl.mask.astype(np.int64)).reshape(self.shape)
        self.flow, self.therm = self.mask & 3, (self.mask >> 2) & 3
        self.ub = [f64(wl.ubar[a]).reshape(self.shape) for a in range(d)]
        self.Tb = f64(wl.Tbar).reshape(self.shape)
        self.ufac = np.asarray(wl.ufac, dtype=np.float64)
        self.exact = wl.adjoint_mode == "exact"
        # ends of the non-periodic axes
        idx = np.indices(self.shape)
        self.at_end = [np.zeros(self.shape, bool) if self.per[a] else
                       (idx[d - 1 - a] == 0) | (idx[d - 1 - a] == self.n[a] - 1) for a in range(d)]
        ne = sum(e.astype(int) for e in self.at_end)
        self.ring, self.face, edge = t(ne > 0), t(ne == 1), ne >= 2
        src = [idx[k] for k in range(d)]
        for a in range(1, d):  # edges take the node one step inwards along y (and z)
            if self.per[a]:
                continue
            k = d - 1 - a
            src[k] = np.clip(src[k], 1, self.n[a] - 2)
        flat = np.ravel_multi_index(src, self.shape)
        self.edge_dst = t(np.flatnonzero(edge.reshape(-1)))
        self.edge_src = t(flat.reshape(-1)[edge.reshape(-1)])
        # coefficients of the design
        self.Aco = 4.5 * (1.0 / 6.0 - wl.nu)
        Kf = wl.nu / wl.Pr if wl.thermal else 0.0
        dK_ = Kf * (wl.Ks_over_Kf if wl.thermal else 1.0) - Kf
        g = gamma.reshape(self.shape)
        inner = ~self.ring
        z = torch.zeros(self.shape, dtype=torch.float64, device=DEV)
        qa, qk = wl.q_alpha, wl.q_K
        self.alpha = torch.where(inner, wl.alpha_max * qa * (1 - g) / (qa + g), z)
        self.B = torch.where(inner, 3 * (1 / 6 - Kf - dK_ * qk * (1 - g) / (qk + g)),
                             z + 3 * (1 / 6 - Kf))
        design = inner & ((self.mask & 128) == 0) if d == 3 else inner
        self.dalpha = torch.where(design, -wl.alpha_max * qa * (1 + qa) / (qa + g) ** 2, z)
        self.dB = torch.where(design, 3 * dK_ * qk * (1 + qk) / (qk + g) ** 2, z)
        self.beta = self.dbeta = None
        if wl.beta_max > 0:
            qb = wl.q_beta
            self.beta = torch.where(inner, wl.beta_max * qb * (1 - g) / (qb + g), z)
            self.dbeta = torch.where(inner, -wl.beta_max * qb * (1 + qb) / (qb + g) ** 2, z)
        self.gb = list(wl.gbeta)[:2] + [0.0]
        self.heated = max(int(((self.mask & W.TAG_PROBE) != 0).sum()), 1)
        self.faces = [(a, s) for a in range(d) if not self.per[a] for s in (-1, 1)]
        self.fill = {(a, s): self._fill(a, s) for a, s in self.faces}

    # -- differences -----------------------------------------------------
    def dif(self, f, a):
        dim = -1 - a
        o = 0.5 * (torch.roll(f, -1, dim) - torch.roll(f, 1, dim))
        if not self.per[a]:
            n = self.n[a]
            at = lambda i: f.select(dim, i)  # noqa: E731
            o.select(dim, 0).copy_(0.5 * (-3 * at(0) + 4 * at(1) - at(2)))
            o.select(dim, n - 1).copy_(0.5 * (3 * at(n - 1) - 4 * at(n - 2) + at(n - 3)))
        return o

    def shift(self, f, c):
        """f(x - c)"""
        s = [(int(v), -1 - a) for a, v in enumerate(c) if v]
        return torch.roll(f, [v for v, _ in s], [k for _, k in s]) if s else f

    def slab(self, f, a, s):
        return f.select(-1 - a, 0 if s < 0 else self.n[a] - 1)

    def copy_edges(self, f):
        v = f.reshape(-1)
        v[self.edge_dst] = v[self.edge_src]

    # -- forward -----------------------------------------------------------
    def init(self):
        z = torch.zeros(self.shape, dtype=torch.float64, device=DEV)
        vel = self.face & (self.flow == 1)
        u = [torch.where(vel, b * self.ufac[0], z) for b in self.ub]
        T = None
        if self.wl.thermal:
            T = torch.where(self.therm == 1, self.Tb, z)
            self.copy_edges(T)
        return z.clone(), u, T

    def step(self, st, level):
        d_, u, T = st
        fac = float(self.ufac[min(level, len(self.ufac) - 1)])
        D = range(self.d)
        G = [[self.dif(u[a], b) for b in D] for a in D]
        gT = [self.dif(T, b) for b in D] if T is not None else None
        uu = sum(x * x for x in u)
        f, g = [], []
        for c, w in zip(self.c, self.w):
            cu = sum((float(c[a]) * u[a] for a in D if c[a]), torch.zeros_like(d_))
            cGc = sum((2.0 * float(c[a] * c[b]) * G[a][b] for a in D for b in D if c[a] * c[b]),
                      torch.zeros_like(d_))
            v = w * (d_ - 1.5 * uu + 3 * cu + 4.5 * cu * cu + self.Aco * cGc)
            f.append(self.shift(v, c))
            if T is not None:
                cg = sum((float(c[a]) * gT[a] for a in D if c[a]), torch.zeros_like(d_))
                g.append(self.shift(w * (T * (1 + 3 * cu) + self.B * cg), c))
        dn = sum(f)
        un = [sum(float(c[a]) * x for c, x in zip(self.c, f) if c[a]) for a in D]
        Tn = None
        if T is not None:
            Tn = sum(g)
            if self.beta is not None:
                Tn = (Tn + self.beta) / (1 + self.beta)
            for a in D:
                if self.gb[a]:
                    un[a] = un[a] + self.gb[a] * (Tn - self.wl.T_ref)
        un = [x / (1 + self.alpha) for x in un]
        if Tn is not None:
            Tn = torch.where((self.therm == 1) & ~self.ring, self.Tb, Tn)
        for a, s in self.faces:
            cn = self.c[:, a] * s
            S = sum(self.slab(x, a, s) * (1.0 if k == 0 else 2.0) for k, x in zip(cn, f) if k >= 0)
            vel = self.slab(self.flow, a, s) == 1
            ubs = [self.slab(b, a, s) * fac for b in self.ub]
            unn = torch.where(vel, ubs[a] * s, S - self.wl.rho_out + 1.0)
            out = torch.where(vel, S - unn, torch.full_like(S, self.wl.rho_out - 1.0))
            self.slab(dn, a, s).copy_(out)
            for b in D:
                other = unn * s if b == a else torch.zeros_like(S)
                self.slab(un[b], a, s).copy_(torch.where(vel, ubs[b], other))
            if Tn is not None:
                Sg = sum(self.slab(x, a, s) * (1.0 if k == 0 else 2.0)
                         for k, x in zip(cn, g) if k >= 0)
                tb = self.slab(self.Tb, a, s)
                self.slab(Tn, a, s).copy_(
                    torch.where(self.slab(self.therm, a, s) == 1, tb, (Sg + tb) / (1 + unn)))
        self.copy_edges(dn)
        for x in un:
            x.reshape(-1)[self.edge_dst] = 0.0
        if Tn is not None:
            self.copy_edges(Tn)
        return dn, un, Tn

    def level_objective(self, st):
        d_, u, T = st
        m, o = self.mask, self.wl.objective
        if o == W.OBJ_PRESSURE_DROP:
            p = (1.0 + d_) / 3.0
            return p[(m & W.TAG_J_INLET) != 0].sum() - p[(m & W.TAG_J_OUTLET) != 0].sum()
        probe = (m & W.TAG_PROBE) != 0
        if o == W.OBJ_HEAT:
            return (u[0] * T)[probe].sum()
        if o == W.OBJ_HEAT_SINK:
            return T[probe].sum() / self.heated
        return (self.beta * (T - 1)).sum()

    # -- adjoint -----------------------------------------------------------
    def _fill(self, a, s):
        """The least-squares problems of the face with outward normal s e_a: rows r over
        the directions, unknown populations c.n > 0 and the multipliers."""
        c, w = self.c.astype(np.float64), self.w
        cn = c[:, a] * s
        un = np.flatnonzero(cn > 0)
        Bf = float(3 * (1 / 6 - (self.wl.nu / self.wl.Pr if self.wl.thermal else 0.0)))
        M = np.diag(cn) - 2 * self.Aco * (c @ c.T) * (w * cn)[None, :]
        Mg = np.diag(cn) - Bf * np.ones((len(w), 1)) * (w * cn)[None, :]
        tang = [c[:, b:b + 1] for b in range(self.d) if b != a]
        one = np.ones((len(w), 1))
        known = (cn <= 0).astype(np.float64)
        pv = np.linalg.pinv(np.hstack([M[:, un], c]))[:len(un)]
        pp = np.linalg.pinv(np.hstack([M[:, un], one] + tang))[:len(un)]
        pd = np.linalg.pinv(np.hstack([Mg[:, un], one]))[:len(un)]
        K0 = Mg[:, un]
        p0 = np.linalg.pinv(K0)
        proj = np.eye(len(w)) - K0 @ p0
        t = lambda x: torch.as_tensor(x, device=DEV)  # noqa: E731
        return dict(un=un, cn=t(cn), M=t(M * known), Mg=t(Mg * known), pv=t(pv), pp=t(pp),
                    pd=t(pd), p0=t(p0), va=t(proj @ cn), vb=t(proj.sum(1)))

    def adjoint_step(self, adj, st, seeds):
        """Adjoint coefficients (r, V, Theta) of level n from those of level n + 1 and the
        state of level n; returns them with the moments the sensitivity needs."""
        r0, V0, Th0 = adj
        _, u, T = st
        sdp, sh, ss, sbt = seeds
        D, th = range(self.d), T is not None
        c, w, z = self.c, self.w, torch.zeros_like(r0)
        f = [self.shift(r0 + sum((float(k[a]) * V0[a] for a in D if k[a]), z), -k) for k in c]
        f = [x.clone() for x in f]
        g = [self.shift(Th0, -k).clone() for k in c] if th else None
        probe = (self.mask & W.TAG_PROBE) != 0
        for a, s in self.faces:
            op = self.fill[(a, s)]
            sl = lambda x: self.slab(x, a, s)  # noqa: E731
            vel = sl(self.flow) == 1
            F = torch.stack([sl(x) for x in f])
            shp = F.shape[1:]
            m = sl(self.mask)
            seed = sdp * (((m & W.TAG_J_INLET) != 0).double() - ((m & W.TAG_J_OUTLET) != 0).double())
            b = (op["M"] @ F.reshape(len(w), -1)) + seed.reshape(1, -1)
            if th:
                Gs = torch.stack([sl(x) for x in g]).reshape(len(w), -1)
                bg = op["Mg"] @ Gs
                un = (sl(u[a]) * s).reshape(1, -1)
                v = op["va"][:, None] - un * op["vb"][:, None]
                kap = -(v * bg).sum(0, keepdim=True) / (v * v).sum(0, keepdim=True)
                col = op["cn"][:, None] - un
                flux = -(op["p0"] @ (bg + kap * col))
                diri = (sl(self.therm) == 1).reshape(1, -1)
                gu = torch.where(diri, -(op["pd"] @ bg), flux)
                kap = torch.where(diri, torch.zeros_like(kap), kap)
                b = b - kap * sl(T).reshape(1, -1) * op["cn"][:, None]
                for k, q in enumerate(op["un"]):
                    sl(g[q]).copy_(gu[k].reshape(shp))
                if sbt:
                    e = torch.where(sl(probe), sbt / (1 + un.reshape(shp)), torch.zeros(shp, dtype=torch.float64, device=DEV))
                    for q in range(len(w)):
                        k = int(c[q, a] * s)
                        if k >= 0:
                            sl(g[q]).sub_((1.0 if k == 0 else 2.0) * e)
            fu = torch.where(vel.reshape(1, -1), -(op["pv"] @ b), -(op["pp"] @ b))
            for k, q in enumerate(op["un"]):
                sl(f[q]).copy_(fu[k].reshape(shp))
        mom = lambda x, k: sum((float(wi * k(ci)) * y for ci, wi, y in zip(c, w, x) if k(ci)), z)  # noqa: E731
        r = mom(f, lambda k: 1)
        U = [mom(f, lambda k, a=a: k[a]) for a in D]
        S = [[mom(f, lambda k, a=a, b=b: k[a] * k[b]) for b in D] for a in D]
        Tt, q = z, [z] * self.d
        if th:
            Tt = mom(g, lambda k: 1)
            q = [mom(g, lambda k, a=a: k[a]) for a in D]
            if sh:
                Tt = Tt - torch.where(probe, sh * u[0], z)
            zero = (self.therm == 1) & (self.ring if self.d == 2 else torch.ones_like(self.ring))
            if not self.exact:
                zero = zero & ~self.ring
            Tt = torch.where(zero, z, Tt)
            q = [torch.where(zero, z, x) for x in q]
            U = [U[a] + T * q[a] for a in D]
            if sh:
                U[0] = U[0] - torch.where(probe, sh / 3.0 * T, z)
        ut = U if self.exact else [x / (1 + self.alpha) for x in U]
        inner = ~self.ring
        if th and not self.exact and any(self.gb):
            Tt = Tt + torch.where(inner, 3 * sum(self.gb[a] * ut[a] for a in D), z)
        if self.beta is not None:
            Tt = Tt - ss * self.beta
            if not self.exact:
                Tt = Tt / (1 + self.beta)
        r, Tt = r.clone(), Tt.clone()
        ut, q = [x.clone() for x in ut], [x.clone() for x in q]
        for x in [r, Tt] + ut + q + [S[a][b] for a in D for b in D]:
            self.copy_edges(x)
        V = [3 * ut[a] + 9 * sum(S[a][b] * u[b] for b in D) - 3 * r * u[a]
             - 2 * self.Aco * sum(self.dif(S[a][b], b) for b in D) for a in D]
        sens = 3 * self.dalpha * sum(u[a] * ut[a] for a in D)
        if self.exact:
            sens = self.dalpha * sum(u[a] * V[a] for a in D) / (1 + self.alpha)
            V = [x / (1 + self.alpha) for x in V]
        Th, cond = None, z
        if th:
            Th = Tt + 3 * sum(q[a] * u[a] for a in D)
            if self.exact:
                Th = Th - sum(self.dif(self.B * q[a], a) for a in D)
                if any(self.gb):
                    Th = Th + torch.where(inner, sum(self.gb[a] * V[a] for a in D), z)
                if self.beta is not None:
                    Th = Th / (1 + self.beta)
            else:
                Th = Th - self.B * sum(self.dif(q[a], a) for a in D) \
                    - sum(self.dif(self.B, a) * q[a] for a in D)
            cond = -self.dB * sum(self.dif(T, a) * q[a] for a in D)
            if self.beta is not None:
                sens = sens + self.dbeta * (T - 1) * (ss + (Th if self.exact else Tt))
        sens = torch.where(inner, sens, z)
        return (r, V, Th), sens, torch.where(inner, cond, z)

    def seeds(self, w):
        o = self.wl.objective
        return (w if o == W.OBJ_PRESSURE_DROP else 0.0, w if o == W.OBJ_HEAT else 0.0,
                w if o == W.OBJ_HEAT_EXCHANGE else 0.0,
                w / self.heated if o == W.OBJ_HEAT_SINK else 0.0)

    def evaluate(self, steps, n_adj):
        uns = self.wl.mode == W.MODE_UNSTEADY
        st = self.init()
        levels, J = [st], 0.0
        for n in range(steps):
            st = self.step(st, n + 1)
            if uns:
                J = J + self.level_objective(st) / steps
                levels.append((None, st[1], st[2]))
        if not uns:
            J = self.level_objective(st)
        out = {"J": torch.as_tensor(J, dtype=torch.float64)}
        names = ["ux", "uy", "uz"][:self.d]
        if not (uns and n_adj > 0):
            out["drho"] = st[0]
            out.update(zip(names, st[1]))
            if self.wl.thermal:
                out["T"] = st[2]
        if n_adj > 0:
            z = torch.zeros(self.shape, dtype=torch.float64, device=DEV)
            adj, dJ = (z, [z] * self.d, z), z
            for k in range(steps + 1 if uns else n_adj):
                n = steps - k
                sd = self.seeds((1.0 / steps if n >= 1 else 0.0) if uns else 1.0)
                adj, sens, cond = self.adjoint_step(adj, levels[n] if uns else st, sd)
                if uns:
                    # exact mode: alpha and beta act on the levels that the steps produce
                    dJ = dJ + cond + (sens if n >= 1 or not self.exact else 0.0)
                elif k == n_adj - 1:
                    dJ = sens + cond
            out["dJ"] = dJ
            out["adj_rho"] = adj[0]
            out.update(zip(["adj_vx", "adj_vy", "adj_vz"][:self.d], adj[1]))
            if self.wl.thermal:
                out["adj_theta"] = adj[2]
        return {k: v.reshape(-1) if isinstance(v, torch.Tensor) else v for k, v in out.items()}


def exact(case, seed):
    with torch.no_grad():
        if case["kind"] == "batch":
            wls = _batch_problems(case)
            got = [_Exact(w, _design(w, 977 * seed + d)).evaluate(case["n_fwd"], case["n_adj"])
                   for d, w in enumerate(wls)]
            return {"J": torch.tensor([r["J"] for r in got], dtype=torch.float64),
                    "dJ": [r["dJ"] for r in got]}
        wl = _wl(case)
        steps = case.get("n_steps", case.get("n_fwd"))
        return _Exact(wl, _design(wl, seed)).evaluate(steps, case.get("n_adj", steps))
