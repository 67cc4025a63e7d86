"""Performance cases: the work a program has this framework do, through the
public entry points of paper_2609_29081_amd.af, over the range of grid sizes,
boundaries, precisions and integrators that are used.

Kinds of case (key "kind"):
  pass      2D: one SSP-RK3 step as its parts, the way a program with its own
            step control calls them: af_cfl_dt and three af_rk_stage
  step      one af_step (RK3 or RK54, 1D or 2D), from a given state
  run       several steps: af_run (host decisions) or af_run_graph (device)
  batch     several instances of a parameter sweep advanced together
  learned   2D: one stage under the learned blend, and the blend itself
  features  2D: the training features of every face of a snapshot
  train     minibatch training of the blend network

exact() holds a plain float64 evaluation of the same method written with
torch operations on whole arrays.
"""
import math
import random

import numpy as np
import torch

from paper_2609_29081_amd import af
from paper_2609_29081_amd import workloads as W

DEV = "cuda:0"
GAMMA = 1.4
PER, OUT, NOSLIP, SYM, DIR = 0, 1, 2, 3, 4
BC = {"tube": (NOSLIP, NOSLIP, NOSLIP, SYM), "wave": (PER,) * 4, "field": (OUT,) * 4,
      "channel": (PER, PER, NOSLIP, SYM)}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the headline workload: the viscous shock tube at 1000 x 500
        dict(name="tube_fp64", kind="pass", flow="tube", n1=1000, n2=500, prec=0),
        # the same under the mixed-precision stage
        dict(name="tube_mixed", kind="pass", flow="tube", n1=1000, n2=500, prec=1),
        # the largest smooth run of the benchmark, beyond the last-level cache
        dict(name="wave_2048", kind="pass", flow="wave", n1=2048, n2=2048, prec=0),
        # a production run with the step decisions on the device
        dict(name="tube_graph", kind="run", flow="tube", n1=400, n2=200, prec=0, rk=3, steps=16,
             graph=True),
        # one synchronous step of a small grid: latency, launches, host work
        dict(name="step_small", kind="step", flow="tube", n1=64, n2=32, prec=0, rk=3),
        # a ragged grid with open sides under the fourth-order integrator
        dict(name="field_rk54", kind="step", flow="field", n1=333, n2=167, prec=0, rk=54),
        # the 1D near-vacuum problem of the paper at its resolution
        dict(name="leblanc_run", kind="run", flow="leblanc", n1=800, n2=1, prec=0, rk=3, steps=40,
             graph=False),
        # the smallest call: one step of the 1D viscous shock
        dict(name="becker_step", kind="step", flow="becker", n1=160, n2=1, prec=0, rk=54),
        # a sweep of tubes of different sizes and Reynolds numbers, together
        dict(name="sweep_batch", kind="batch", flow="tube", n1=512, n2=8, prec=1, steps=3,
             graph=True),
        # inference of the learned blend, and the stage that uses it
        dict(name="learned_stage", kind="learned", flow="tube", n1=1000, n2=500, prec=0),
        # training data of one snapshot
        dict(name="features", kind="features", flow="tube", n1=500, n2=250, prec=0),
        # training as the benchmark does it: minibatches of 1024 rows
        dict(name="train_1024", kind="train", rows=16384, batch=1024, steps=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["pass", "pass", "step", "run", "run1", "step1", "batch", "learned",
                       "features", "train"])
    if kind == "train":
        batch = _log_int(rng, 65, 4096)
        return dict(kind="train", rows=batch * rng.randint(2, 16) + rng.randint(0, 63),
                    batch=batch, steps=rng.randint(8, 64))
    if kind == "run1":
        return dict(kind="run", flow=rng.choice(["leblanc", "becker", "line"]),
                    n1=_log_int(rng, 40, 4000), n2=1, prec=0, rk=rng.choice([3, 54]),
                    steps=rng.randint(10, 40), graph=False)
    if kind == "step1":
        return dict(kind="step", flow=rng.choice(["leblanc", "becker", "line"]),
                    n1=_log_int(rng, 40, 8000), n2=1, prec=0, rk=rng.choice([3, 54]))
    flow = rng.choice(["tube", "wave", "field", "channel"])
    n1 = _log_int(rng, 48, 1400)
    n2 = max(24, min(1400, int(n1 * rng.uniform(0.35, 1.1))))
    prec = rng.choice([0, 0, 1])
    if kind == "pass":
        return dict(kind="pass", flow=flow, n1=n1, n2=n2, prec=prec)
    if kind == "step":
        return dict(kind="step", flow=flow, n1=n1, n2=n2, prec=prec, rk=rng.choice([3, 3, 54]))
    if kind == "run":
        n1 = min(n1, _log_int(rng, 48, 400))
        n2 = max(24, min(n2, n1))
        return dict(kind="run", flow=flow, n1=n1, n2=n2, prec=prec, rk=3,
                    steps=rng.randint(4, 12), graph=rng.choice([True, False]))
    if kind == "batch":
        return dict(kind="batch", flow="tube", n1=_log_int(rng, 96, 512), n2=rng.randint(2, 10),
                    prec=prec, steps=rng.randint(1, 3), graph=rng.choice([True, False]))
    return dict(kind=kind, flow=flow, n1=n1, n2=n2, prec=0)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _grid(c, n1=None, n2=None):
    n1, n2 = n1 or c["n1"], n2 or c["n2"]
    flow = c["flow"]
    if flow == "leblanc":
        return W.Grid(dim=1, n1=n1, x0=-0.5, x1=0.5, bc=(OUT,) * 4)
    if flow == "becker":
        return W.Grid(dim=1, n1=n1, x0=-1.0, x1=1.5, bc=(DIR,) * 4)
    if flow == "line":
        return W.Grid(dim=1, n1=n1, bc=(PER,) * 4)
    if flow == "tube":
        return W.Grid(dim=2, n1=n1, n2=n2, x0=0.0, x1=1.0, y0=0.0, y1=0.5, bc=BC[flow])
    return W.Grid(dim=2, n1=n1, n2=n2, x0=0.0, x1=1.0, y0=0.0, y1=n2 / n1, bc=BC[flow])


def _flow(c, g, rng):
    """(primitive fields of (x, y) as torch, physics keywords); values as a
    run holds them a while after its start: fronts a few cells wide, walls at
    rest, modes of a few wavelengths"""
    two_pi = 2.0 * math.pi
    flow = c["flow"]
    Lx, Ly = g.x1 - g.x0, (g.y1 - g.y0)
    amp = [rng.uniform(0.5, 1.0) for _ in range(6)]
    ph = [rng.uniform(0.0, 1.0) for _ in range(12)]

    if flow == "leblanc":
        xs, w = -0.2 + rng.uniform(-0.05, 0.05), 2.0 * g.dx
        pl = 6.666667e-2 * rng.uniform(0.8, 1.2)

        def f(x, y):
            s = 0.5 * (1.0 - torch.tanh((x - xs) / w))
            return (torch.exp(math.log(1e-2) * (1 - s)), torch.zeros_like(x),
                    torch.exp(math.log(pl) * s + math.log(6.666667e-11) * (1 - s)))
        return f, dict(mu=0.0, Pr=0.72, cfl_c=0.3, cfl_v=0.1)
    if flow == "becker":
        # a front between the end states of a shock of Mach number M, in the
        # width of the viscous profile
        M, mu = rng.uniform(2.0, 4.0), 1e-2
        wr = ((GAMMA - 1.0) + 2.0 / M ** 2) / (GAMMA + 1.0)
        w0 = math.sqrt(wr)
        delta = max(4.0 * mu, 2.0 * g.dx)

        def f(x, y):
            s = 0.5 * (1.0 - torch.tanh(x / delta))
            w = wr + (1.0 - wr) * s
            e = ((GAMMA + 1.0) / (GAMMA - 1.0) * w0 * w0 - w * w) / (2.0 * GAMMA)
            return (1.0 / w, 0.2 + w, (GAMMA - 1.0) * e / w)

        def cons(w):
            e = ((GAMMA + 1.0) / (GAMMA - 1.0) * w0 * w0 - w * w) / (2.0 * GAMMA)
            u = 0.2 + w
            return [1.0 / w, u / w, e / w + 0.5 * u * u / w]
        return f, dict(mu=mu, Pr=0.75, cfl_c=0.3, cfl_v=0.1, bcstate=[cons(1.0), cons(wr)])
    if flow == "line":
        def f(x, y):
            return (1.0 + 0.2 * amp[0] * torch.sin(two_pi * (x + ph[0])),
                    1.0 + 0.2 * amp[1] * torch.sin(two_pi * (2 * x + ph[1])),
                    1.0 + 0.2 * amp[2] * torch.sin(two_pi * (x + ph[2])))
        return f, dict(mu=1e-3, Pr=0.72, cfl_c=0.3, cfl_v=0.1)
    if flow == "tube":
        ratio, xs, w = rng.uniform(50.0, 200.0), 0.5 + rng.uniform(-0.1, 0.1), 4.0 * g.dx
        re = rng.uniform(200.0, 1000.0)

        def f(x, y):
            s = 0.5 * (1.0 - torch.tanh((x - xs) / w))
            r = 1.2 * torch.exp(math.log(ratio) * s)
            bump = torch.sin(math.pi * x) * torch.sin(math.pi * y)  # 0 at the walls
            u = 0.4 * amp[0] * bump * torch.cos(two_pi * (x + ph[0]))
            v = 0.2 * amp[1] * torch.sin(math.pi * x) * torch.sin(two_pi * y) \
                * torch.sin(two_pi * (2 * x + ph[1]))
            p = r / GAMMA * (1.0 + 0.1 * amp[2] * torch.cos(two_pi * (x + ph[2]))
                             * torch.cos(two_pi * y))
            return (r, u, v, p)
        return f, dict(mu=1.0 / re, Pr=0.73, cfl_c=0.2, cfl_v=0.05)

    # "wave" (periodic), "field" (open sides), "channel" (periodic along x
    # between a wall and a symmetry line)
    mom_y = flow == "channel"

    def f(x, y):
        xx, yy = (x - g.x0) / Lx, (y - g.y0) / Ly
        env = torch.sin(0.5 * math.pi * yy) if mom_y else torch.ones_like(xx)
        envv = torch.sin(math.pi * yy) if mom_y else torch.ones_like(xx)
        r = 1.0 + 0.2 * amp[0] * torch.sin(two_pi * (xx + ph[0])) * torch.cos(two_pi * (yy + ph[1]))
        u = env * (1.0 + 0.3 * amp[1] * torch.sin(two_pi * (2 * xx + ph[2]))
                   * torch.cos(two_pi * (yy + ph[3])))
        v = envv * (0.8 + 0.3 * amp[2] * torch.cos(two_pi * (xx + ph[4]))
                    * torch.sin(two_pi * (2 * yy + ph[5])))
        p = 1.0 + 0.1 * amp[3] * torch.cos(two_pi * (xx + ph[6])) * torch.cos(two_pi * (yy + ph[7]))
        return (r, u, v, p)
    return f, dict(mu=1e-3, Pr=0.72, cfl_c=0.2, cfl_v=0.05)


def _cons(P):
    if len(P) == 3:
        r, u, p = P
        return torch.stack([r, r * u, p / (GAMMA - 1.0) + 0.5 * r * u * u])
    r, u, v, p = P
    return torch.stack([r, r * u, r * v, p / (GAMMA - 1.0) + 0.5 * r * (u * u + v * v)])


def _state(g, f):
    """cell averages by Gauss-Legendre quadrature, point values sampled: a
    flat float64 state on the GPU"""
    gx, gw = np.polynomial.legendre.leggauss(3)
    gx, gw = 0.5 * (gx + 1.0), 0.5 * gw
    ar = lambda n: torch.arange(n, dtype=torch.float64, device=DEV)  # noqa: E731
    xc, xp = g.x0 + ar(g.n1) * g.dx, g.x0 + ar(g.n1x) * g.dx
    if g.dim == 1:
        avg = sum(w * _cons(f(xc + q * g.dx, None)) for q, w in zip(gx, gw))
        return torch.cat([avg.reshape(-1), _cons(f(xp, None)).reshape(-1)])
    yc, yp = g.y0 + ar(g.n2) * g.dy, g.y0 + ar(g.n2y) * g.dy

    def at(xs, ys):
        Y, X = torch.meshgrid(ys, xs, indexing="ij")
        return _cons(f(X, Y))
    avg = None
    for a, wa in zip(gx, gw):
        for b, wb in zip(gx, gw):
            t = float(wa * wb) * at(xc + a * g.dx, yc + b * g.dy)
            avg = t if avg is None else avg + t
    parts = [avg, at(xp, yc + 0.5 * g.dy), at(xc + 0.5 * g.dx, yp), at(xp, yp)]
    return torch.cat([p.reshape(-1) for p in parts])


def _input(c, seed, n1=None, n2=None):
    g = _grid(c, n1, n2)
    f, kw = _flow(c, g, random.Random(seed))
    return g, _state(g, f), kw


def _net(seed):
    """parameters of a 40-64-64-1 network: Glorot-uniform weights, small
    hidden biases, output bias near the untouched flux's 1"""
    r = np.random.default_rng(seed)

    def gl(o, i):
        a = math.sqrt(6.0 / (i + o))
        return r.uniform(-a, a, size=(o, i)).ravel()
    p = np.concatenate([gl(64, 40), 0.05 * r.standard_normal(64), gl(64, 64),
                        0.05 * r.standard_normal(64), 0.5 * gl(1, 64), np.array([0.6])])
    return torch.from_numpy(p.astype(np.float32)).to(DEV)


def _sweep(c, seed):
    """the instances of a batch: tubes of widths up to n1, half as high"""
    out = []
    for k in range(c["n2"]):
        n1 = max(32, int(c["n1"] * (1.0 - 0.75 * k / max(1, c["n2"]))))
        out.append(_input(c, seed * 1000 + k, n1, max(16, n1 // 2)))
    return out


def _rows(c, seed):
    """training rows: features of a size that faces have, targets mostly 1"""
    r = torch.Generator(device=DEV).manual_seed(seed)
    n = c["rows"]
    X = 0.4 * torch.randn((n, 40), generator=r, device=DEV)
    y = torch.clamp(1.2 - torch.rand(n, generator=r, device=DEV) ** 2
                    - 0.3 * X[:, 3].abs(), 0.0, 1.0)
    return X.contiguous(), y.contiguous()


def _solver(c, g, kw, **more):
    kw = dict(kw, gamma=GAMMA, **more)
    return af.Solver(g, precision=c.get("prec", 0), rk=c.get("rk", 3), device=DEV, **kw)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c, "kind": kind}
    if kind == "train":
        s["X"], s["y"] = _rows(c, seed)
        s["p0"] = _net(seed)
        s["p"], s["m"], s["v"] = (torch.empty_like(s["p0"]) for _ in range(3))
        return s
    if kind == "batch":
        inst = _sweep(c, seed)
        s["solvers"] = [_solver(c, g, kw) for g, _, kw in inst]
        s["U0"] = [U for _, U, _ in inst]
        s["U"] = [torch.empty_like(U) for U in s["U0"]]
        s["batch"] = af.Batch(s["solvers"])
        return s
    g, U0, kw = _input(c, seed)
    more = {"limiter": af.LIM_ALL | af.LIM_LEARNED} if kind == "learned" else {}
    s["S"] = _solver(c, g, kw, **more)
    s["U0"] = U0
    if kind == "learned":
        s["S"].af_set_blend_net(_net(seed + 1))
        s["A"] = torch.empty_like(U0)
    elif kind == "pass":
        s["A"], s["B"], s["C"] = (torch.empty_like(U0) for _ in range(3))
    elif kind in ("step", "run"):
        s["U"] = torch.empty_like(U0)
    return s


def run(s):
    c, kind = s["case"], s["kind"]
    if kind == "pass":
        S, U0, A, B, C = s["S"], s["U0"], s["A"], s["B"], s["C"]
        dt = S.af_cfl_dt(U0)
        S.af_rk_stage(0, U0, U0, A, dt_dev=dt)
        S.af_rk_stage(1, U0, A, B, dt_dev=dt)
        S.af_rk_stage(2, U0, B, C, dt_dev=dt)
        return {"U": C, "dt": dt}
    if kind == "step":
        s["U"].copy_(s["U0"])
        st, dt, h = s["S"].af_step(s["U"])
        return {"U": s["U"], "status": st, "dt": dt, "halvings": h}
    if kind == "run":
        s["U"].copy_(s["U0"])
        if c["graph"]:
            st, n, t, att = s["S"].af_run_graph(s["U"], 0.0, 1e30, c["steps"])
        else:
            st, n, t = s["S"].af_run(s["U"], 0.0, 1e30, c["steps"])
            att = n
        return {"U": s["U"], "status": st, "steps": n, "t": t, "attempts": att}
    if kind == "batch":
        for U, U0 in zip(s["U"], s["U0"]):
            U.copy_(U0)
        st, n, t, att = s["batch"].af_batch_run(s["U"], 0.0, 1e30, c["steps"],
                                                use_graph=c["graph"])
        return {"U": s["U"], "status": st, "steps": n, "t": t, "attempts": att}
    if kind == "learned":
        S = s["S"]
        theta = S.af_blend_infer(s["U0"])
        dt = S.af_cfl_dt(s["U0"])
        S.af_rk_stage(0, s["U0"], s["U0"], s["A"], dt_dev=dt)
        return {"theta": theta, "U": s["A"], "dt": dt}
    if kind == "features":
        return s["S"].af_blend_features(s["U0"])
    # train: from the initial parameters
    s["p"].copy_(s["p0"])
    s["m"].zero_()
    s["v"].zero_()
    loss = af.mlp_train(s["X"], s["y"], s["p"], s["m"], s["v"], 0, c["steps"], c["batch"], 1e-3)
    return {"p": s["p"], "m": s["m"], "v": s["v"], "loss": loss}


def work(case):
    """bytes: a stage reads U^k (and U^n after the first) and writes U^(k+1);
    flops: the operator count of the method per cell and stage"""
    c, kind = case, case["kind"]
    if kind == "train":
        n = min(c["batch"], c["rows"]) * c["steps"]
        return {"bytes": 4.0 * 41 * n, "flops": 6.0 * (40 * 64 + 64 * 64 + 64) * n}
    if kind == "batch":
        gs = []
        for k in range(c["n2"]):
            n1 = max(32, int(c["n1"] * (1.0 - 0.75 * k / max(1, c["n2"]))))
            gs.append(_grid(c, n1, max(16, n1 // 2)))
        return {"bytes": sum(64.0 * g.state_len for g in gs) * c["steps"],
                "flops": sum(9000.0 * g.n1 * g.n2 for g in gs) * c["steps"]}
    g = _grid(c)
    cells, nb = g.n1 * g.n2, 8.0 * g.state_len
    faces = g.n2 * (g.n1 + 1) + (g.n2 + 1) * g.n1
    if kind == "features":
        return {"bytes": 32.0 * cells + 160.0 * faces, "flops": 200.0 * faces}
    if kind == "learned":
        return {"bytes": 2 * nb + 32.0 * cells + 8.0 * faces,
                "flops": 3000.0 * cells + 2 * 13440.0 * faces}
    per = 3000.0 if g.dim == 2 else 600.0
    stages, states = (3, 8) if c.get("rk", 3) == 3 else (5, 20)
    n = c.get("steps", 1)
    return {"bytes": nb * states * n, "flops": per * stages * cells * n}


# ---------------------------------------------------------------------------
# the method in float64 on whole arrays
# ---------------------------------------------------------------------------
EPS = 1e-13


def _image(n, lo, hi, m=4):
    """interior site and crossed wall kind (-1: none) of every lattice
    coordinate -m .. 2n+m of an axis"""
    idx, kind = [], []
    for X in range(-m, 2 * n + m + 1):
        k = -1
        if lo == PER:
            Xi = X % (2 * n)
        elif X < 0:
            Xi, k = ((X & 1), -1) if lo == OUT else (-X, lo)
        elif X > 2 * n:
            Xi, k = ((2 * n - ((X - 2 * n) & 1)), -1) if hi == OUT else (4 * n - X, hi)
        else:
            Xi = X
        idx.append(Xi)
        kind.append(k)
    return idx, kind


def _theta_lin(zl, zh, eps):
    return torch.where(zh < eps, (zl - eps) / torch.where(zh < eps, zl - zh, torch.ones_like(zl)),
                       torch.ones_like(zl))


def _press(U):
    m2 = U[1] * U[1] if U.shape[0] == 3 else U[1] * U[1] + U[2] * U[2]
    return (GAMMA - 1.0) * (U[-1] - 0.5 * m2 / U[0])


def _theta_pair(UL, UH):
    pL = _press(UL)
    bad = bool((~(UL[0] > 0.0)).any() or (~(pL > 0.0)).any())
    e = torch.clamp(UL[0], max=EPS)
    tr = _theta_lin(UL[0], UH[0], e)
    T = UL + tr * (UH - UL)
    tp = _theta_lin(pL, _press(T), torch.clamp(pL, max=EPS))
    return torch.where(UL[0] > 0.0, tr * tp, torch.zeros_like(tr)), bad


def _dc(z, ax, h):
    """fourth-order central difference on the half lattice, zero in the
    two outer lines"""
    o = torch.zeros_like(z)
    n = z.shape[ax]
    s = lambda a: z.narrow(ax, 2 + a, n - 4)  # noqa: E731
    o.narrow(ax, 2, n - 4).copy_(((s(-2) - s(2)) + 8.0 * (s(1) - s(-1))) / (6.0 * h))
    return o


def _five(z, ax):
    n = z.shape[ax]
    return [z.narrow(ax, 2 + a, n - 4) for a in (-2, -1, 0, 1, 2)]


def _bcol(z):
    return -(z[0] + z[4]) / 12.0 + 4.0 / 3.0 * (z[1] + z[3]) - 2.5 * z[2]


BMAT = [[-1 / 8, 1 / 6, -1 / 24, 0, 0], [1 / 6, 1 / 2, -5 / 6, 1 / 6, 0],
        [-1 / 8, 1 / 2, -3 / 4, 1 / 2, -1 / 8], [0, 1 / 6, -5 / 6, 1 / 2, 1 / 6],
        [0, 0, -1 / 24, 1 / 6, -1 / 8]]


def _bquad(z):
    out = 0.0
    for m in range(5):
        for n in range(5):
            if BMAT[m][n]:
                out = out + BMAT[m][n] * z[m] * z[n]
    return out


def _bvisc(p, T, q, t2):
    return (torch.sqrt(q * q + 2.0 * T / (GAMMA - 1.0) * t2) + q.abs()) * (0.5 * (GAMMA - 1.0)) / p


class _Ref2:
    """one limited forward-Euler step of the 2D method"""

    def __init__(self, g, kw):
        self.g, self.mu = g, kw["mu"]
        self.kap = GAMMA * kw["mu"] / ((GAMMA - 1.0) * kw["Pr"])
        self.cfl = (kw["cfl_c"], kw["cfl_v"], max(4.0 * self.mu / 3.0, GAMMA * self.mu / kw["Pr"]))
        xi, kx = _image(g.n1, g.bc[0], g.bc[1])
        yi, ky = _image(g.n2, g.bc[2], g.bc[3])
        t = lambda v: torch.tensor(v, device=DEV)  # noqa: E731
        self.xi, self.yi = t(xi), t(yi)
        wall = (NOSLIP, SYM)
        sg = lambda b: torch.where(t(b), -1.0, 1.0).double()  # noqa: E731
        self.fx = (sg([k in wall for k in kx])[None, :], sg([k == NOSLIP for k in ky])[:, None])
        self.fy = (sg([k == NOSLIP for k in kx])[None, :], sg([k in wall for k in ky])[:, None])

    def parts(self, U):
        out, off = [], 0
        for _, r, c in self.g.blocks():
            out.append(U[off:off + 4 * r * c].reshape(4, r, c))
            off += 4 * r * c
        return out

    def extend(self, I):
        E = I.index_select(1, self.yi).index_select(2, self.xi)
        E[1] *= self.fx[0]
        E[1] *= self.fx[1]
        E[2] *= self.fy[0]
        E[2] *= self.fy[1]
        return E

    def lattice(self, U):
        g = self.g
        avg, xe, ye, co = self.parts(U)
        H = 2 * g.n2 + (1 if g.n2y > g.n2 else 0)
        w = 2 * g.n1 + (1 if g.n1x > g.n1 else 0)
        I = torch.empty((4, H, w), dtype=torch.float64, device=DEV)
        I[:, 1::2, 1::2], I[:, 1::2, 0::2], I[:, 0::2, 1::2], I[:, 0::2, 0::2] = avg, xe, ye, co
        lo = self.extend(I)
        a = lambda dy, dx: lo[:, 5 + dy:5 + dy + 2 * g.n2 - 1:2, 5 + dx:5 + dx + 2 * g.n1 - 1:2]  # noqa
        e = a(0, -1) + a(0, 1) + a(-1, 0) + a(1, 0)
        c = a(-1, -1) + a(-1, 1) + a(1, -1) + a(1, 1)
        V = (36.0 * avg - 4.0 * e - c) / 16.0
        th, _ = _theta_pair(avg, V)
        I[:, 1::2, 1::2] = torch.where(th < 1.0, avg + th * (V - avg), V)
        return lo, self.extend(I)

    @staticmethod
    def prims(V):
        p = _press(V)
        T = p / V[0]
        return V[1] / V[0], V[2] / V[0], p, T, torch.sqrt(GAMMA * T)

    def stress(self, ux, vx, uy, vy):
        return (self.mu * (4 / 3 * ux - 2 / 3 * vy), self.mu * (uy + vx),
                self.mu * (4 / 3 * vy - 2 / 3 * ux))

    def total(self, d, V, u, v, p, gr):
        ux, vx, Tx, uy, vy, Ty = gr
        xx, xy, yy = self.stress(ux, vx, uy, vy)
        ud = u if d == 0 else v
        a, b, Td = (xx, xy, Tx) if d == 0 else (xy, yy, Ty)
        zero = torch.zeros_like(p)
        return torch.stack([V[1 + d], V[1] * ud + (p if d == 0 else zero) - a,
                            V[2] * ud + (p if d == 1 else zero) - b,
                            (V[3] + p) * ud - (u * a + v * b + self.kap * Td)])

    def bvisc(self, d, p, T, gr):
        ux, vx, Tx, uy, vy, Ty = gr
        xx, xy, yy = self.stress(ux, vx, uy, vy)
        q = self.kap * (Tx if d == 0 else Ty)
        return _bvisc(p, T, q, xx * xx + xy * xy if d == 0 else xy * xy + yy * yy)

    def dt(self, U):
        g = self.g
        avg = self.parts(U)[0]
        u, v, p, T, c = self.prims(avg)
        a = max(float((u.abs() + c).max()) / (self.cfl[0] * g.dx),
                float((v.abs() + c).max()) / (self.cfl[0] * g.dy))
        return 1.0 / (a + float((self.cfl[2] / (self.cfl[1] * min(g.dx, g.dy) ** 2)
                                 / avg[0]).max()))

    def euler(self, U, dt, theta=None):
        """(the step's result before the wall projection is part of it, flag)"""
        g = self.g
        h = (g.dx, g.dy)
        lo, L = self.lattice(U)
        flag = False
        u, v, p, T, c = self.prims(L)
        gr = [_dc(z, 1, g.dx) for z in (u, v, T)] + [_dc(z, 0, g.dy) for z in (u, v, T)]
        # cell averages: low-order data on the cells -1 .. n
        CA = lo[:, 1::2, 1::2]
        cu, cv, cp, cT, cc = self.prims(CA)
        mid = lambda z: z[..., 1:-1, 1:-1]  # noqa: E731
        dx_ = lambda z: (z[1:-1, 2:] - z[1:-1, :-2]) / (2.0 * g.dx)  # noqa: E731
        dy_ = lambda z: (z[2:, 1:-1] - z[:-2, 1:-1]) / (2.0 * g.dy)  # noqa: E731
        cg = [dx_(cu), dx_(cv), dx_(cT), dy_(cu), dy_(cv), dy_(cT)]
        CU, pu, pv, pp, pT, pc = mid(CA), mid(cu), mid(cv), mid(cp), mid(cT), mid(cc)
        jx = (cp[1:-1, 2:] - 2 * pp + cp[1:-1, :-2]).abs() / (cp[1:-1, 2:] + 2 * pp
                                                              + cp[1:-1, :-2]).abs()
        jy = (cp[2:, 1:-1] - 2 * pp + cp[:-2, 1:-1]).abs() / (cp[2:, 1:-1] + 2 * pp
                                                              + cp[:-2, 1:-1]).abs()
        phi1 = torch.maximum(jx, jy)
        div, curl = cg[0] + cg[4], cg[1] - cg[3]
        phi2 = torch.clamp(-div / torch.sqrt(div * div + curl * curl + 1e-13), min=0.0)
        limited = []
        nfx = g.n2 * (g.n1 + 1)
        for d in range(2):
            F = self.total(d, L, u, v, p, gr)
            if d == 0:
                s = lambda o: F[:, 5 + o:5 + o + 2 * g.n2 - 1:2, 4:4 + 2 * g.n1 + 1:2]  # noqa
                A_, B_ = (slice(1, -1), slice(0, -1)), (slice(1, -1), slice(1, None))
            else:
                s = lambda o: F[:, 4:4 + 2 * g.n2 + 1:2, 5 + o:5 + o + 2 * g.n1 - 1:2]  # noqa
                A_, B_ = (slice(0, -1), slice(1, -1)), (slice(1, None), slice(1, -1))
            FH = (s(-1) + 4.0 * s(0) + s(1)) / 6.0
            Fc = self.total(d, CU, pu, pv, pp, cg)
            rs = (pu if d == 0 else pv).abs() + pc
            bd = self.bvisc(d, pp, pT, cg)
            mxm = lambda z: torch.maximum(z[A_], z[B_])  # noqa: E731
            lam = mxm(rs) + mxm(bd)
            Ua, Ub, Fa, Fb = (z[(slice(None),) + w] for z, w in ((CU, A_), (CU, B_), (Fc, A_),
                                                                 (Fc, B_)))
            FL = 0.5 * (Fa + Fb) - 0.5 * lam * (Ub - Ua)
            if theta is None:
                ts = torch.exp(-mxm(phi1) * mxm(phi2))
            elif d == 0:
                ts = theta[:nfx].reshape(g.n2, g.n1 + 1)
                if g.n1x == g.n1:
                    ts = torch.cat([ts[:, :-1], ts[:, :1]], 1)
            else:
                ts = theta[nfx:].reshape(g.n2 + 1, g.n1)
                if g.n2y == g.n2:
                    ts = torch.cat([ts[:-1], ts[:1]], 0)
            Fs = FL + ts * (FH - FL)
            m4 = 4.0 * dt / h[d]
            ULp, UHp = Ua - m4 * (FL - Fa), Ua - m4 * (Fs - Fa)
            ULm, UHm = Ub - m4 * (Fb - FL), Ub - m4 * (Fb - Fs)
            pLp, pLm = _press(ULp), _press(ULm)
            ok = (ULp[0] > 0) & (ULm[0] > 0)
            flag |= bool((~(ok & (pLp > 0) & (pLm > 0))).any())
            tr = torch.minimum(_theta_lin(ULp[0], UHp[0], torch.clamp(ULp[0], max=EPS)),
                               _theta_lin(ULm[0], UHm[0], torch.clamp(ULm[0], max=EPS)))
            tp = torch.minimum(
                _theta_lin(pLp, _press(ULp + tr * (UHp - ULp)), torch.clamp(pLp, max=EPS)),
                _theta_lin(pLm, _press(ULm + tr * (UHm - ULm)), torch.clamp(pLm, max=EPS)))
            th = ts * torch.where(ok, tr * tp, torch.zeros_like(tr))
            limited.append(FL + th * (FH - FL))
            del F, FH, Fs, ULp, UHp, ULm, UHm
        avg = self.parts(U)[0]
        new_avg = (avg - dt / g.dx * (limited[0][:, :, 1:] - limited[0][:, :, :-1])
                   - dt / g.dy * (limited[1][:, 1:] - limited[1][:, :-1]))
        del limited
        # points: residual on the whole lattice but its outer two lines
        R = torch.zeros_like(L)
        for d in range(2):
            ax = 1 - d  # axis of a plane
            hd = h[d]
            ud, uo = (u, v) if d == 0 else (v, u)
            zero = 0.0
            f = [L[1 + d], L[1] * ud + (p if d == 0 else zero), L[2] * ud + (p if d == 1 else zero),
                 (L[3] + p) * ud]
            al = _five(ud.abs() + c, ax)
            alpha = al[0]
            for z in al[1:]:
                alpha = torch.maximum(alpha, z)
            va, vb, Tt = _five(ud, ax), _five(uo, ax), _five(T, ax)
            n = L.shape[1 + ax]
            for k in range(4):
                w = _five(L[k], ax)
                ff = _five(f[k], ax)
                r = -(((ff[0] - ff[4]) + 8.0 * (ff[3] - ff[1]))
                      + alpha * ((w[0] + w[4]) - 4.0 * (w[1] + w[3]) + 6.0 * w[2])) / (6.0 * hd)
                R[k].narrow(ax, 2, n - 4).add_(r)
            s4, m43 = 4.0 / (hd * hd), 4.0 / 3.0 * self.mu
            ga, gb = (gr[3], gr[4]) if d == 0 else (gr[1], gr[0])
            mix = [-2 / 3 * self.mu * gb, self.mu * ga, self.mu * (uo * ga - 2 / 3 * ud * gb)]
            comp = (1 + d, 2 - d, 3)
            add = [s4 * m43 * _bcol(va), s4 * self.mu * _bcol(vb),
                   s4 * (m43 * _bquad(va) + self.mu * _bquad(vb) + self.kap * _bcol(Tt))]
            for k in range(3):
                R[comp[k]].narrow(ax, 2, n - 4).add_(add[k])
                R[comp[k]].add_(_dc(mix[k], ax, hd))
            del f, al, va, vb, Tt, mix, add
        del gr, u, v, p, T, c
        # points: low-order value on the lattice of points and averages
        lu, lv, lp, lT, lc = self.prims(lo)

        def cd(z, ax, hh):
            o = torch.zeros_like(z)
            n = z.shape[ax]
            o.narrow(ax, 1, n - 2).copy_((z.narrow(ax, 2, n - 2) - z.narrow(ax, 0, n - 2)) / hh)
            return o
        lg = [cd(z, 1, g.dx) for z in (lu, lv, lT)] + [cd(z, 0, g.dy) for z in (lu, lv, lT)]
        UL = lo.clone()
        for d in range(2):
            ax = 1 - d
            F = self.total(d, lo, lu, lv, lp, lg)
            b = self.bvisc(d, lp, lT, lg)
            rs = (lu if d == 0 else lv).abs() + lc
            n = lo.shape[1 + ax]
            a1 = lambda z, o: z.narrow(z.dim() - 2 + ax, o, n - 1)  # noqa: E731
            lam = torch.maximum(a1(rs, 0), a1(rs, 1)) + torch.maximum(a1(b, 0), a1(b, 1))
            Fi = 0.5 * (a1(F, 0) + a1(F, 1)) - 0.5 * lam * (a1(lo, 1) - a1(lo, 0))
            UL.narrow(1 + ax, 1, n - 2).sub_(
                2.0 * dt / h[d] * (Fi.narrow(1 + ax, 1, n - 2) - Fi.narrow(1 + ax, 0, n - 2)))
            del F, b, Fi
        out = [new_avg]
        for (_, r, cn), oy, ox in zip(g.blocks()[1:], (5, 4, 4), (4, 5, 4)):
            pick = lambda z: z[:, oy:oy + 2 * r - 1:2, ox:ox + 2 * cn - 1:2]  # noqa: E731
            U0 = pick(L)
            UH, low = U0 + dt * pick(R), pick(UL)
            th, bad = _theta_pair(low, UH)
            flag |= bad
            V = torch.where(th == 1.0, UH, low + th * (UH - low))
            self.walls(V, oy == 4, ox == 4)
            out.append(V)
        return torch.cat([z.reshape(-1) for z in out]), flag

    def walls(self, V, on_y, on_x):
        g = self.g

        def proj(P, kind, ax):
            if kind == NOSLIP:
                P[3] -= (P[1] * P[1] + P[2] * P[2]) / (2.0 * P[0])
                P[1] = 0.0
                P[2] = 0.0
            elif kind == SYM:
                P[3] -= P[1 + ax] * P[1 + ax] / (2.0 * P[0])
                P[1 + ax] = 0.0
        if on_x and g.bc[0] != PER:
            proj(V[:, :, 0], g.bc[0], 0)
            proj(V[:, :, -1], g.bc[1], 0)
        if on_y and g.bc[2] != PER:
            proj(V[:, 0], g.bc[2], 1)
            proj(V[:, -1], g.bc[3], 1)


class _Ref1:
    """one limited forward-Euler step of the 1D method"""

    def __init__(self, g, kw):
        self.g, self.mu = g, kw["mu"]
        self.kap = GAMMA * kw["mu"] / ((GAMMA - 1.0) * kw["Pr"])
        self.cfl = (kw["cfl_c"], kw["cfl_v"], max(4.0 * self.mu / 3.0, GAMMA * self.mu / kw["Pr"]))
        self.xi = torch.tensor(_image(g.n1, g.bc[0] if g.bc[0] != DIR else OUT,
                                      g.bc[1] if g.bc[1] != DIR else OUT)[0], device=DEV)
        self.side = None
        if g.bc[0] == DIR:
            self.side = torch.tensor(kw["bcstate"], dtype=torch.float64, device=DEV)

    def parts(self, U):
        g = self.g
        return U[:3 * g.n1].reshape(3, g.n1), U[3 * g.n1:].reshape(3, g.n1x)

    def extend(self, I):
        E = I.index_select(1, self.xi)
        if self.side is not None:
            E[:, :4] = self.side[0][:, None]
            E[:, -4:] = self.side[1][:, None]
        return E

    @staticmethod
    def prims(V):
        p = _press(V)
        return V[1] / V[0], p, p / V[0], torch.sqrt(GAMMA * p / V[0])

    def total(self, V, u, p, ux, Tx):
        tau = 4.0 / 3.0 * self.mu * ux
        return torch.stack([V[1], V[1] * u + p - tau, (V[2] + p) * u - (u * tau + self.kap * Tx)])

    def bvisc(self, p, T, ux, Tx):
        return _bvisc(p, T, self.kap * Tx, (self.mu * 4.0 / 3.0 * ux) ** 2)

    def dt(self, U):
        g = self.g
        avg = self.parts(U)[0]
        u, p, T, c = self.prims(avg)
        return 1.0 / (float((u.abs() + c).max()) / (self.cfl[0] * g.dx)
                      + float((self.cfl[2] / (self.cfl[1] * g.dx ** 2) / avg[0]).max()))

    def euler(self, U, dt, theta=None):
        g, dx = self.g, self.g.dx
        avg, pts = self.parts(U)
        I = torch.empty((3, g.n1 + g.n1x), dtype=torch.float64, device=DEV)
        I[:, 1::2], I[:, 0::2] = avg, pts
        lo = self.extend(I)
        nb = lambda o: lo[:, 5 + o:5 + o + 2 * g.n1 - 1:2]  # noqa: E731
        V = (6.0 * avg - (nb(-1) + nb(1))) / 4.0
        th, _ = _theta_pair(avg, V)
        I[:, 1::2] = torch.where(th < 1.0, avg + th * (V - avg), V)
        L = self.extend(I)
        u, p, T, c = self.prims(L)
        ux, Tx = _dc(u, 0, dx), _dc(T, 0, dx)
        FH = self.total(L, u, p, ux, Tx)[:, 4:4 + 2 * g.n1 + 1:2]
        CA = lo[:, 1::2]
        cu, cp, cT, cc = self.prims(CA)
        m = lambda z: z[..., 1:-1]  # noqa: E731
        cd = lambda z: (z[2:] - z[:-2]) / (2.0 * dx)  # noqa: E731
        gu, gT = cd(cu), cd(cT)
        Fc = self.total(m(CA), m(cu), m(cp), gu, gT)
        rs, b = m(cu).abs() + m(cc), self.bvisc(m(cp), m(cT), gu, gT)
        phi1 = (cp[2:] - 2 * cp[1:-1] + cp[:-2]).abs() / (cp[2:] + 2 * cp[1:-1] + cp[:-2]).abs()
        phi2 = torch.clamp(-gu / torch.sqrt(gu * gu + 1e-13), min=0.0)
        mxm = lambda z: torch.maximum(z[:-1], z[1:])  # noqa: E731
        lam = mxm(rs) + mxm(b)
        Ua, Ub, Fa, Fb = m(CA)[:, :-1], m(CA)[:, 1:], Fc[:, :-1], Fc[:, 1:]
        FL = 0.5 * (Fa + Fb) - 0.5 * lam * (Ub - Ua)
        ts = torch.exp(-mxm(phi1) * mxm(phi2))
        Fs = FL + ts * (FH - FL)
        m2 = 2.0 * dt / dx
        ULp, UHp = Ua - m2 * (FL - Fa), Ua - m2 * (Fs - Fa)
        ULm, UHm = Ub - m2 * (Fb - FL), Ub - m2 * (Fb - Fs)
        pLp, pLm = _press(ULp), _press(ULm)
        ok = (ULp[0] > 0) & (ULm[0] > 0)
        flag = bool((~(ok & (pLp > 0) & (pLm > 0))).any())
        tr = torch.minimum(_theta_lin(ULp[0], UHp[0], torch.clamp(ULp[0], max=EPS)),
                           _theta_lin(ULm[0], UHm[0], torch.clamp(ULm[0], max=EPS)))
        tp = torch.minimum(
            _theta_lin(pLp, _press(ULp + tr * (UHp - ULp)), torch.clamp(pLp, max=EPS)),
            _theta_lin(pLm, _press(ULm + tr * (UHm - ULm)), torch.clamp(pLm, max=EPS)))
        F = FL + ts * torch.where(ok, tr * tp, torch.zeros_like(tr)) * (FH - FL)
        new_avg = avg - dt / dx * (F[:, 1:] - F[:, :-1])
        # points
        fl = [L[1], L[1] * u + p, (L[2] + p) * u]
        al = _five(u.abs() + c, 0)
        alpha = al[0]
        for z in al[1:]:
            alpha = torch.maximum(alpha, z)
        R = torch.zeros_like(L)
        for k in range(3):
            w, ff = _five(L[k], 0), _five(fl[k], 0)
            R[k, 2:-2] = -(((ff[0] - ff[4]) + 8.0 * (ff[3] - ff[1]))
                           + alpha * ((w[0] + w[4]) - 4.0 * (w[1] + w[3]) + 6.0 * w[2])) / (6 * dx)
        s4, m43 = 4.0 / (dx * dx), 4.0 / 3.0 * self.mu
        R[1, 2:-2] += s4 * m43 * _bcol(_five(u, 0))
        R[2, 2:-2] += s4 * (m43 * _bquad(_five(u, 0)) + self.kap * _bcol(_five(T, 0)))
        lu, lp, lT, lc = self.prims(lo)
        ch = lambda z: torch.nn.functional.pad((z[2:] - z[:-2]) / dx, (1, 1))  # noqa: E731
        gu, gT = ch(lu), ch(lT)
        Ft, b, rs = self.total(lo, lu, lp, gu, gT), self.bvisc(lp, lT, gu, gT), lu.abs() + lc
        lam = mxm(rs) + mxm(b)
        Fi = 0.5 * (Ft[:, :-1] + Ft[:, 1:]) - 0.5 * lam * (lo[:, 1:] - lo[:, :-1])
        UL = lo.clone()
        UL[:, 1:-1] -= 2.0 * dt / dx * (Fi[:, 1:] - Fi[:, :-1])
        pick = lambda z: z[:, 4:4 + 2 * g.n1x - 1:2]  # noqa: E731
        low, UH = pick(UL), pick(L) + dt * pick(R)
        th, bad = _theta_pair(low, UH)
        V = torch.where(th == 1.0, UH, low + th * (UH - low))
        if self.side is not None:
            V[:, 0], V[:, -1] = self.side[0], self.side[1]
        return torch.cat([new_avg.reshape(-1), V.reshape(-1)]), flag or bad


def _ref(g, kw):
    return (_Ref1 if g.dim == 1 else _Ref2)(g, kw)


def _rk3(r, U, dt, theta=None):
    a, f0 = r.euler(U, dt)
    b, f1 = r.euler(a, dt)
    b = 0.75 * U + 0.25 * b
    c, f2 = r.euler(b, dt)
    return U / 3.0 + 2.0 / 3.0 * c, f0 or f1 or f2


def _rk54(r, U, dt):
    """SSPRK(5,4) of Spiteri and Ruuth"""
    E0, f0 = r.euler(U, 0.391752226571890 * dt)
    E1, f1 = r.euler(E0, 0.368410593050371 / 0.555629506348765 * dt)
    u2 = 0.444370493651235 * U + 0.555629506348765 * E1
    E2, f2 = r.euler(u2, 0.251891774271694 / 0.379898148511597 * dt)
    u3 = 0.620101851488403 * U + 0.379898148511597 * E2
    E3, f3 = r.euler(u3, 0.544974750228521 / 0.821920045606868 * dt)
    u4 = 0.178079954393132 * U + 0.821920045606868 * E3
    E4, f4 = r.euler(u4, 0.226007483236906 / 0.386708617503269 * dt)
    return (0.517231671970585 * u2 + 0.096059710526147 * E3 + 0.386708617503269 * E4,
            f0 or f1 or f2 or f3 or f4)


def _steps(g, U, kw, rk, n):
    r = _ref(g, kw)
    t, halvings, attempts, dt = 0.0, 0, 0, 0.0
    for _ in range(n):
        dt = r.dt(U)
        halvings = 0
        while True:
            V, flag = (_rk54 if rk == 54 else _rk3)(r, U, dt)
            attempts += 1
            if not flag:
                break
            dt, halvings = 0.5 * dt, halvings + 1
        U, t = V, t + dt
    return U, t, dt, halvings, attempts


def _features(g, kw, U):
    r = _Ref2(g, kw)
    lo, _ = r.lattice(U)
    CA = lo[:, 1::2, 1::2]
    u, v, p, _, _ = r.prims(CA)
    rho = CA[0]
    out = []
    for d in range(2):
        n, t = (u, v) if d == 0 else (v, u)

        def cell(z, s, q):  # tangential offset s-1, normal offset q-2 of every face
            a, b = (s - 1, q - 2)
            if d == 0:
                return z[2 + a:2 + a + g.n2, 2 + b:2 + b + g.n1 + 1]
            return z[2 + b:2 + b + g.n2 + 1, 2 + a:2 + a + g.n1]
        mean = lambda z: 0.5 * (cell(z, 1, 1) + cell(z, 1, 2))  # noqa: E731
        rf, pf, nf, tf = mean(rho), mean(p), mean(n), mean(t)
        cf = torch.sqrt(GAMMA * pf / rf)
        fe = []
        for s in range(3):
            for q in range(4):
                fe += [torch.log(cell(p, s, q) / pf), (cell(n, s, q) - nf) / cf,
                       (cell(t, s, q) - tf) / cf]
        fe += [torch.log(cell(rho, 1, q) / rf) for q in range(4)]
        out.append(torch.stack(fe, -1).reshape(-1, 40))
    return torch.cat(out, 0)


def _unpack(p):
    o, out = 0, []
    for shape in ((64, 40), (64,), (64, 64), (64,), (64,), (1,)):
        n = int(np.prod(shape))
        out.append(p[o:o + n].reshape(shape))
        o += n
    return out


def _train(c, seed):
    X, y = _rows(c, seed)
    X, y, p = X.double(), y.double(), _net(seed).double()
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    row, loss = 0, None
    nb = min(c["batch"], c["rows"])
    for k in range(c["steps"]):
        if row + nb > c["rows"]:
            row = 0
        x, t = X[row:row + nb], y[row:row + nb]
        row += nb
        W1, b1, W2, b2, w3, b3 = _unpack(p)
        h1 = torch.tanh(x @ W1.t() + b1)
        h2 = torch.tanh(h1 @ W2.t() + b2)
        res = h2 @ w3 + b3 - t
        loss = (res * res).mean()
        dz = 2.0 * res / nb
        a2 = dz[:, None] * w3 * (1.0 - h2 * h2)
        a1 = (a2 @ W2) * (1.0 - h1 * h1)
        g = torch.cat([(a1.t() @ x).reshape(-1), a1.sum(0), (a2.t() @ h1).reshape(-1), a2.sum(0),
                       h2.t() @ dz, dz.sum()[None]])
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - 1e-3 * (m / (1.0 - 0.9 ** (k + 1))) / (torch.sqrt(v / (1.0 - 0.999 ** (k + 1)))
                                                       + 1e-8)
    return {"p": p, "m": m, "v": v, "loss": loss.reshape(1)}


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "train":
        return _train(c, seed)
    if kind == "batch":
        got = [_steps(g, U, kw, 3, c["steps"]) for g, U, kw in _sweep(c, seed)]
        n = c["n2"]
        return {"U": [r[0] for r in got], "status": [None] * n, "steps": [None] * n,
                "t": [r[1] for r in got], "attempts": [None] * n}
    g, U, kw = _input(c, seed)
    if kind == "features":
        return _features(g, kw, U)
    if kind == "learned":
        W1, b1, W2, b2, w3, b3 = (z.double() for z in _unpack(_net(seed + 1)))
        h = torch.tanh(torch.tanh(_features(g, kw, U) @ W1.t() + b1) @ W2.t() + b2)
        theta = torch.clamp(h @ w3 + b3, 0.0, 1.0)
        r = _ref(g, kw)
        dt = r.dt(U)
        return {"theta": theta, "U": r.euler(U, dt, theta)[0],
                "dt": torch.tensor([dt], dtype=torch.float64)}
    if kind == "pass":
        r = _ref(g, kw)
        dt = r.dt(U)
        return {"U": _rk3(r, U, dt)[0], "dt": torch.tensor([dt], dtype=torch.float64)}
    V, t, dt, _, _ = _steps(g, U, kw, c["rk"], c.get("steps", 1))
    if kind == "step":
        return {"U": V, "status": None, "dt": dt, "halvings": None}
    return {"U": V, "status": None, "steps": None, "t": t, "attempts": None}
