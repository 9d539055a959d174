"""Timed cases: what a program does with this package, through its public entry points.

One case is a dict of plain values.  `kind` names the entry point:

  equilibrium  paper_1307_6720_amd.solver.solve: (11) on the base, (8) in the box, then B, p and rho
  interior     Plan.solve_interior, or solve_interior_noalloc, with Dirichlet data on every face
  serve        paper_1307_6720_amd.serve.Server over a list of requests
  general      Plan.solve_general: a lap u + b u = c in the box
  face         Plan.solve_face: the same on one face of the box
  fields       Plan.fields: B, p and rho of a given P
  diagnostics  Plan.diagnostics: residuals of the equilibrium's equations
  lines        Plan.trace_field_lines

Grids have 2^L + 1 nodes per axis.  The package computes in FP64 throughout, with FP32 V-cycles inside the FP64
refinement of the mixed precision.
"""

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1307_6720_amd import PREC_FP64, PREC_MIXED
from paper_1307_6720_amd import _lib
from paper_1307_6720_amd.serve import DeviceBackend, Request, Server
from paper_1307_6720_amd.solver import GridSpec, Plan, make_opts, solve, solve_interior_noalloc

DEVICE = "cuda:0"
PRECISION = {"fp64": PREC_FP64, "mixed": PREC_MIXED}
FACES = ("base", "top", "xlo", "xhi", "ylo", "yhi")
FACE_CODE = {"base": _lib.FACE_BASE, "top": _lib.FACE_TOP, "xlo": _lib.FACE_XLO, "xhi": _lib.FACE_XHI,
             "ylo": _lib.FACE_YLO, "yhi": _lib.FACE_YHI}
#: the serving stream's request shapes (nx, ny, nz)
SERVE_SHAPES = {"four": ((65, 65, 65), (129, 129, 129), (129, 129, 65), (257, 257, 257)),
                "small": ((33, 33, 33), (65, 65, 65), (65, 65, 33)),
                "129": ((129, 129, 129),),
                "257": ((257, 257, 257),)}


def _grid(nx, ny, nz, lx=1.0, ly=1.0, lz=1.0):
    return {"nx": nx, "ny": ny, "nz": nz, "lx": lx, "ly": ly, "lz": lz}


def listed():
    return [
        # the smallest job: a potential field on 33^3, one call after another in an interactive program or a parameter
        # scan; launches and round trips count
        {"name": "equilibrium-33-mixed", "kind": "equilibrium", **_grid(33, 33, 33), "precision": "mixed", "rtol": 1e-10,
         "alpha": 0.0, "a": 0.0, "h": 0.2, "bipoles": 2, "noise": 0.0},
        # an ordinary job to full accuracy
        {"name": "equilibrium-129-fp64", "kind": "equilibrium", **_grid(129, 129, 129), "precision": "fp64",
         "rtol": 1e-12, "alpha": 0.5, "a": 0.5, "h": 0.2, "bipoles": 6, "noise": 0.0},
        # one equilibrium of the benchmark's size at a time, the mixed path and the FP64 path
        {"name": "equilibrium-257-mixed", "kind": "equilibrium", **_grid(257, 257, 257), "precision": "mixed",
         "rtol": 1e-10, "alpha": 0.5, "a": 0.5, "h": 0.2, "bipoles": 6, "noise": 0.0},
        {"name": "equilibrium-257-fp64", "kind": "equilibrium", **_grid(257, 257, 257), "precision": "fp64",
         "rtol": 1e-10, "alpha": 1.0, "a": 0.5, "h": 0.2, "bipoles": 6, "noise": 0.0},
        # the largest single equilibrium: a noisy magnetogram of many bipoles, dz = 2 dx
        {"name": "equilibrium-513-mixed", "kind": "equilibrium", **_grid(513, 513, 257), "precision": "mixed",
         "rtol": 1e-12, "alpha": 0.8, "a": 1.0, "h": 0.1, "bipoles": 40, "noise": 0.01},
        # (8) with the caller's own data on the side and top faces, on a box with three different axes
        {"name": "interior-65x129x33-fp64", "kind": "interior", **_grid(65, 129, 33, 0.5, 1.0, 0.25),
         "entry": "plan", "precision": "fp64", "rtol": 1e-10, "alpha": 0.5, "a": 0.5, "h": 0.2},
        # throughput: the benchmark's twelve requests in flight
        {"name": "serve-257x12-mixed", "kind": "serve", "shapes": "257", "requests": 12, "precision": "mixed",
         "rtol": 1e-10},
        # throughput of a server with requests of four shapes
        {"name": "serve-four-shapes-32", "kind": "serve", "shapes": "four", "requests": 32, "precision": "mixed",
         "rtol": 1e-10},
        # the general elliptic problem in the box, and on a face (its solution is boundary data for (8))
        {"name": "general-257", "kind": "general", **_grid(257, 257, 257), "rtol": 1e-10},
        {"name": "face-129x65-xhi", "kind": "face", **_grid(65, 129, 65, 0.5, 1.0, 0.5), "face": "xhi", "rtol": 1e-10},
        # what follows a solve: the check of the equations and the field lines drawn from the base
        {"name": "diagnostics-257", "kind": "diagnostics", **_grid(257, 257, 257)},
        {"name": "lines-257", "kind": "lines", **_grid(257, 257, 257), "lines": 16384, "max_steps": 1024, "ds": 0.5},
    ]


def draw(rng):
    """One more case of the same ranges; rng is a random.Random."""
    kind = rng.choice(("equilibrium", "equilibrium", "equilibrium", "interior", "interior", "serve", "general", "face",
                       "fields", "diagnostics", "lines"))

    def grid(lo, hi, most):
        # nodes per axis 2^lo + 1 .. 2^hi + 1 with nearly equal spacings (z up to twice finer or coarser), the longest
        # side of the base 1; at most `most` nodes
        while True:
            base = rng.randint(lo, hi)
            n = [2 ** min(hi, max(lo, base + rng.choice((-1, 0, 0, 1)))) + 1 for _ in range(3)]
            if n[0] * n[1] * n[2] <= most:
                break
        h = 1.0 / (max(n) - 1)
        return _grid(*n, h * (n[0] - 1), h * (n[1] - 1), h * (n[2] - 1) * rng.choice((0.5, 0.75, 1.0, 1.0, 1.5, 2.0)))

    model = {"alpha": round(rng.uniform(0.0, 1.0), 3), "a": round(rng.choice((0.0, rng.uniform(0.0, 1.0))), 3),
             "h": rng.choice((0.1, 0.2))}
    if kind == "equilibrium":
        return {"kind": kind, **grid(3, 9, 513 * 513 * 257), "precision": rng.choice(("mixed", "fp64")),
                "rtol": rng.choice((1e-10, 1e-11, 1e-12)), **model, "bipoles": rng.randint(2, 20),
                "noise": rng.choice((0.0, 0.0, 0.01))}
    if kind == "interior":
        entry = rng.choice(("plan", "noalloc"))
        return {"kind": kind, **grid(3, 7 if entry == "noalloc" else 8, 129 ** 3 if entry == "noalloc" else 257 ** 3),
                "entry": entry, "precision": rng.choice(("mixed", "fp64")), "rtol": rng.choice((1e-8, 1e-10, 1e-11)),
                **model}
    if kind == "serve":
        shapes = rng.choice(("four", "small", "129", "257"))
        return {"kind": kind, "shapes": shapes, "requests": rng.randint(1, 12 if shapes == "257" else 32),
                "precision": rng.choice(("mixed", "mixed", "fp64")), "rtol": rng.choice((1e-8, 1e-10))}
    if kind == "general":
        return {"kind": kind, **grid(3, 8, 257 ** 3), "rtol": rng.choice((1e-8, 1e-10, 1e-11))}
    if kind == "face":
        return {"kind": kind, **grid(3, 8, 257 ** 3), "face": rng.choice(FACES), "rtol": rng.choice((1e-8, 1e-10, 1e-11))}
    if kind == "fields":
        return {"kind": kind, **grid(3, 9, 257 * 513 * 257), **model}
    if kind == "diagnostics":
        return {"kind": kind, **grid(3, 9, 257 * 513 * 257)}
    return {"kind": kind, **grid(4, 8, 257 ** 3), "lines": int(2 ** rng.uniform(0, 14)),
            "max_steps": int(2 ** rng.uniform(4, 10)), "ds": rng.choice((0.25, 0.5, 1.0, -0.5))}


# ---- inputs -------------------------------------------------------------------------------------------------------
def _spec(case):
    return GridSpec(case["nx"], case["ny"], case["nz"], case["lx"], case["ly"], case["lz"])


def _model(nz, lz, alpha, a, h):
    """xi = a exp(-z/h), an isothermal background, mu0 = g = 1."""
    z = np.arange(nz) * (lz / (nz - 1))
    e = np.exp(-z / h)
    return SimpleNamespace(alpha=alpha, xi=a * e, dxi=-(a / h) * e, pb=np.exp(-z), rhob=np.exp(-z), mu0=1.0, g=1.0)


def _magnetogram(g, bipoles, noise, rng):
    """Gaussian bipoles with zero net flux and, with noise > 0, noise on every interior node."""
    x = np.linspace(0.0, g.lx, g.nx)
    y = np.linspace(0.0, g.ly, g.ny)
    pos, neg = np.zeros((g.ny, g.nx)), np.zeros((g.ny, g.nx))
    side = min(g.lx, g.ly)
    for _ in range(bipoles):
        w = side * rng.uniform(0.03, 0.1)
        for into in (pos, neg):
            cx, cy = g.lx * rng.uniform(0.2, 0.8), g.ly * rng.uniform(0.2, 0.8)
            into += np.outer(np.exp(-((y - cy) / w) ** 2), np.exp(-((x - cx) / w) ** 2))
    inner = (slice(1, -1), slice(1, -1))
    bz = pos - (pos[inner].sum() / max(neg[inner].sum(), 1e-300)) * neg
    if noise:
        bz[inner] += rng.normal(0.0, noise * np.abs(bz[inner]).max(), size=bz[inner].shape)
        bz[inner] -= bz[inner].mean()
    bz[0] = bz[-1] = 0.0
    bz[:, 0] = bz[:, -1] = 0.0
    return bz


def _axes(g, device):
    lin = lambda n, length: torch.arange(n, dtype=torch.float64, device=device) * (length / (n - 1))  # noqa: E731
    return lin(g.nx, g.lx), lin(g.ny, g.ly), lin(g.nz, g.lz)


def _modes(g, rng, device, count=12):
    """(potential, (dx, dy, dz of it)) of a few decaying Fourier modes: the smooth arrays that a solve returns."""
    x, y, z = _axes(g, device)
    out = [torch.zeros((g.nz, g.ny, g.nx), dtype=torch.float64, device=device) for _ in range(4)]
    for _ in range(count):
        m, n = int(rng.integers(1, 7)), int(rng.integers(1, 7))
        amp = float(rng.normal())
        kx, ky = m * math.pi / g.lx, n * math.pi / g.ly
        k = math.hypot(kx, ky)
        sx, cx, sy, cy, ez = torch.sin(kx * x), torch.cos(kx * x), torch.sin(ky * y), torch.cos(ky * y), torch.exp(-k * z)
        prod = lambda c, u, v: (c * ez)[:, None, None] * v[None, :, None] * u[None, None, :]  # noqa: E731
        out[0] += prod(amp / k, sx, sy)
        out[1] += prod(amp * kx / k, cx, sy)
        out[2] += prod(amp * ky / k, sx, cy)
        out[3] += prod(-amp, sx, sy)
    return out[0], out[1:]


def _general_arrays(shape, lengths, rng, device):
    """a = 1 + sin(x + 2y [+ 3z])/2, b = -(1 + x^2) - 5 w^2 (w the last axis), random c and boundary values of u."""
    axes = [np.linspace(0.0, length, n) for n, length in zip(shape[::-1], lengths)]
    grids = np.meshgrid(*axes[::-1], indexing="ij", sparse=True)
    a = 1.0 + 0.5 * np.sin(sum((q + 1) * w for q, w in enumerate(grids[::-1])))
    b = np.broadcast_to(-(1.0 + grids[-1] ** 2) - 5.0 * grids[0] ** 2, shape)
    c, u = rng.standard_normal(shape), rng.standard_normal(shape)
    u[tuple(slice(1, -1) for _ in shape)] = 0.0
    return [torch.from_numpy(np.array(t, order="C")).to(device) for t in (a, b, c, u)]


def _face_view(P, face):
    return {"base": P[0], "top": P[-1], "xlo": P[:, :, 0], "xhi": P[:, :, -1], "ylo": P[:, 0], "yhi": P[:, -1]}[face]


def _face_lengths(case):
    return {"base": ("lx", "ly"), "top": ("lx", "ly"), "xlo": ("ly", "lz"), "xhi": ("ly", "lz"), "ylo": ("lx", "lz"),
            "yhi": ("lx", "lz")}[case["face"]]


def _requests(case, seed):
    """Parameters and magnetograms of a serving stream: each request's shape by its number, the rest from its seed."""
    out = []
    shapes = SERVE_SHAPES[case["shapes"]]
    for i in range(case["requests"]):
        rng = np.random.default_rng((seed, i))
        g = GridSpec(*shapes[int(np.random.default_rng(i).integers(len(shapes)))])
        model = _model(g.nz, g.lz, float(rng.uniform(0.0, 1.0)), float(rng.uniform(0.0, 1.0)), 0.2)
        out.append((g, model, _magnetogram(g, int(rng.integers(4, 21)), 0.0, rng)))
    return out


def _inputs(case, seed, device):
    """Every input of a pass, from the seed alone."""
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    if kind == "serve":
        return SimpleNamespace(requests=_requests(case, seed))
    g = _spec(case)
    s = SimpleNamespace(g=g)
    if "alpha" in case:
        s.model = _model(g.nz, g.lz, case["alpha"], case["a"], case["h"])
    if kind == "equilibrium":
        s.bz0 = torch.from_numpy(_magnetogram(g, case["bipoles"], case["noise"], rng)).to(device)
    elif kind == "interior":
        s.P = _modes(g, rng, device)[0] + float(rng.standard_normal())
        s.P[1:-1, 1:-1, 1:-1] = 0.0
    elif kind == "general":
        s.a, s.b, s.c, s.u = _general_arrays(g.shape, (g.lx, g.ly, g.lz), rng, device)
    elif kind == "face":
        s.P = torch.zeros(g.shape, dtype=torch.float64, device=device)
        view = _face_view(s.P, case["face"])
        s.a, s.b, s.c, u = _general_arrays(tuple(view.shape), [case[k] for k in _face_lengths(case)], rng, device)
        view.copy_(u)
    elif kind == "fields":
        s.P = _modes(g, rng, device)[0]
        s.P[-1] = 0.0
    else:
        s.B = [-t for t in _modes(g, rng, device)[1]]
        if kind == "diagnostics":
            s.model = _model(g.nz, g.lz, 0.0, 0.0, 0.2)
            q = 0.05 * s.B[2] ** 2
            z = torch.from_numpy(s.model.pb).to(device)[:, None, None]
            s.p, s.rho = z - q, z + 2.0 * q
        else:
            u = rng.uniform(0.02, 0.98, size=(case["lines"], 3)) * np.array([g.lx, g.ly, 0.0])
            s.seeds = torch.from_numpy(u).to(device)
    return s


class _Backend(DeviceBackend):
    """Keeps the six arrays of a request in one block, each at the alignment of an allocation of its own."""

    def acquire(self, key):
        res = super().acquire(key)
        n = res.P.numel()
        res.block = torch.zeros((6, -(-n // 64) * 64), dtype=torch.float64, device=self.device)
        res.P, *res.F = [t[:n].view(res.P.shape) for t in res.block]
        return res


# ---- one pass -----------------------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    s = _inputs(case, seed, DEVICE)
    s.case = case
    empty = lambda n: tuple(torch.zeros(s.g.shape, dtype=torch.float64, device=DEVICE) for _ in range(n))  # noqa: E731
    if kind == "serve":
        # a slot per request: each result stays in its resident's block until the next pass
        s.backend = _Backend(max_slots=case["requests"], device=DEVICE, precisions=PRECISION[case["precision"]])
        s.results = {}
        s.server = Server(s.backend, 200 << 30,
                          on_finish=lambda req, res: s.results.__setitem__(req.id, res.block[:, :res.P.numel()]))
    elif kind == "equilibrium":
        s.plan = Plan(s.g, PRECISION[case["precision"]], device=DEVICE)
        s.out = empty(6)
    elif kind == "interior":
        s.opts = make_opts(PRECISION[case["precision"]], case["rtol"], faces_given=True)
        if case["entry"] == "plan":
            s.plan = Plan(s.g, PRECISION[case["precision"]], device=DEVICE)
    elif kind in ("general", "face"):
        s.opts = make_opts(PREC_FP64, case["rtol"])
        s.plan = Plan(s.g, PREC_FP64 | _lib.PLAN_GENERAL, device=DEVICE)
    else:
        s.plan = Plan(s.g, PREC_FP64, device=DEVICE)
        if kind == "lines":
            n, m = case["lines"], case["max_steps"]
            s.ds = case["ds"] * s.g.lx / (s.g.nx - 1)
            s.out = (torch.zeros((m + 1, n, 3), dtype=torch.float64, device=DEVICE),
                     torch.zeros(n, dtype=torch.int32, device=DEVICE), torch.zeros(n, dtype=torch.int32, device=DEVICE))
        else:
            s.out = empty(5)
    return s


def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "equilibrium":
        r = solve(s.plan, s.bz0, s.model, PRECISION[case["precision"]], case["rtol"], out=s.out)
        return r.P, r.Bx, r.By, r.Bz, r.p, r.rho
    if kind == "interior":
        if case["entry"] == "plan":
            s.plan.solve_interior(s.model, s.P, s.opts)
        else:
            solve_interior_noalloc(s.g, s.model, s.P, s.opts)
        return s.P
    if kind == "serve":
        reqs = [Request(i, (g.nx, g.ny, g.nz), m, bz0, PRECISION[case["precision"]], case["rtol"])
                for i, (g, m, bz0) in enumerate(s.requests)]
        s.server.run(reqs)
        return [s.results[i] for i in range(len(reqs))]
    if kind == "general":
        s.plan.solve_general(s.a, s.b, s.c, s.u, s.opts)
        return s.u
    if kind == "face":
        s.plan.solve_face(FACE_CODE[case["face"]], s.a, s.b, s.c, s.P, s.opts)
        return s.P
    if kind == "fields":
        return s.plan.fields(s.model, s.P, s.out)
    if kind == "diagnostics":
        return s.plan.diagnostics(s.model, *s.B, s.p, s.rho, s.out)
    return s.plan.trace_field_lines(*s.B, s.seeds, s.ds, case["max_steps"], out=s.out)


def work(case):
    """Inputs read once and outputs written once; the arithmetic of the cycles a solve takes (about one per factor of
    ten of rtol, 4 sweeps, a residual and the transfers of some 12 operations per node, over all levels)."""
    kind = case["kind"]
    if kind == "serve":
        shapes = SERVE_SHAPES[case["shapes"]]
        n = case["requests"] * sum(x * y * z for x, y, z in shapes) / len(shapes)
        base = case["requests"] * sum(x * y for x, y, _ in shapes) / len(shapes)
    else:
        n = case["nx"] * case["ny"] * case["nz"]
        base = case["nx"] * case["ny"]
    cycle = 80.0 * math.ceil(-math.log10(case["rtol"])) if "rtol" in case else 0.0
    if kind in ("equilibrium", "serve"):
        return {"bytes": 48.0 * n + 8.0 * base, "flops": n * (cycle + 60.0)}
    if kind == "interior":
        return {"bytes": 8.0 * n, "flops": n * cycle}
    if kind == "general":
        return {"bytes": 32.0 * n, "flops": n * cycle}
    if kind == "face":
        n = {"base": base, "top": base, "xlo": case["ny"] * case["nz"], "xhi": case["ny"] * case["nz"],
             "ylo": case["nx"] * case["nz"], "yhi": case["nx"] * case["nz"]}[case["face"]]
        return {"bytes": 32.0 * n, "flops": n * cycle}
    if kind == "fields":
        return {"bytes": 48.0 * n, "flops": 60.0 * n}
    if kind == "diagnostics":
        return {"bytes": 80.0 * n, "flops": 70.0 * n}
    # lines: the seeds and the points; a bundle from the base takes about a twelfth of the steps
    steps = 0.08 * case["lines"] * case["max_steps"]
    return {"bytes": 24.0 * case["lines"] + 24.0 * steps, "flops": 400.0 * steps}


# ---- the same in plain 64-bit arithmetic --------------------------------------------------------------------------
def _sine(n, h, device):
    """(orthonormal sine basis of the interior nodes, eigenvalues of minus the second difference)."""
    m = torch.arange(1, n - 1, dtype=torch.float64, device=device)
    S = math.sqrt(2.0 / (n - 1)) * torch.sin(torch.outer(m, m) % (2 * (n - 1)) * (math.pi / (n - 1)))
    return S, (4.0 / (h * h)) * torch.sin(m * (math.pi / (2 * (n - 1)))) ** 2


def _plane_sine(t, Sy, Sx):
    return torch.matmul(torch.matmul(Sy, t), Sx)


def _exact_interior(P, g, model):
    """P with its interior the exact discrete solution of (8) for the Dirichlet data on its faces."""
    dev = P.device
    dx, dy, dz = g.lx / (g.nx - 1), g.ly / (g.ny - 1), g.lz / (g.nz - 1)
    (Sx, lx), (Sy, ly) = _sine(g.nx, dx, dev), _sine(g.ny, dy, dev)
    k = 1.0 - torch.from_numpy(np.asarray(model.xi)).to(dev)[1:-1, None, None]
    P = P.clone()
    P[1:-1, 1:-1, 1:-1] = 0.0
    c = P[1:-1, 1:-1, 1:-1].clone()
    c[:, :, 0] -= (k / dx ** 2)[:, :, 0] * P[1:-1, 1:-1, 0]
    c[:, :, -1] -= (k / dx ** 2)[:, :, 0] * P[1:-1, 1:-1, -1]
    c[:, 0] -= (k / dy ** 2)[:, 0] * P[1:-1, 0, 1:-1]
    c[:, -1] -= (k / dy ** 2)[:, 0] * P[1:-1, -1, 1:-1]
    c[0] -= P[0, 1:-1, 1:-1] / dz ** 2
    c[-1] -= P[-1, 1:-1, 1:-1] / dz ** 2
    r = _plane_sine(c, Sy, Sx)
    lam = ly[:, None] + lx[None, :]
    off, d0 = 1.0 / dz ** 2, model.alpha ** 2 - 2.0 / dz ** 2
    up = torch.empty_like(r)
    for q in range(r.shape[0]):
        d = d0 - k[q] * lam
        if q:
            d = d - off * up[q - 1]
            r[q] = (r[q] - off * r[q - 1]) / d
        else:
            r[q] = r[q] / d
        up[q] = off / d
    for q in range(r.shape[0] - 2, -1, -1):
        r[q] -= up[q] * r[q + 1]
    P[1:-1, 1:-1, 1:-1] = _plane_sine(r, Sy, Sx)
    return P


def _exact_base(bz0, g):
    (Sx, lx), (Sy, ly) = _sine(g.nx, g.lx / (g.nx - 1), bz0.device), _sine(g.ny, g.ly / (g.ny - 1), bz0.device)
    P0 = torch.zeros_like(bz0)
    P0[1:-1, 1:-1] = _plane_sine(_plane_sine(bz0[1:-1, 1:-1], Sy, Sx) / (ly[:, None] + lx[None, :]), Sy, Sx)
    return P0


def _diff(t, axis, h):
    """Central difference, zero at the two ends."""
    d = torch.zeros_like(t)
    n = t.shape[axis]
    d.narrow(axis, 1, n - 2).copy_((t.narrow(axis, 2, n - 2) - t.narrow(axis, 0, n - 2)) / (2.0 * h))
    return d


def _diff_z(t, h):
    d = _diff(t, 0, h)
    d[0] = (-3.0 * t[0] + 4.0 * t[1] - t[2]) / (2.0 * h)
    return d


def _diff2(t, axis, h):
    d = torch.zeros_like(t)
    n = t.shape[axis]
    mid = t.narrow(axis, 1, n - 2)
    d.narrow(axis, 1, n - 2).copy_((t.narrow(axis, 2, n - 2) - 2.0 * mid + t.narrow(axis, 0, n - 2)) / (h * h))
    return d


def _walls(t, value):
    """Side and top faces set to `value` (a number, or one per plane)."""
    if not isinstance(value, float):
        value = value[:, None]
        t[-1] = value[-1]
    else:
        t[-1] = value
    t[:, :, 0] = t[:, :, -1] = value
    t[:, 0] = t[:, -1] = value
    return t


def _exact_fields(P, g, model):
    dx, dy, dz = g.lx / (g.nx - 1), g.ly / (g.ny - 1), g.lz / (g.nz - 1)
    tab = {k: torch.from_numpy(np.asarray(getattr(model, k))).to(P.device) for k in ("xi", "dxi", "pb", "rhob")}
    col = {k: v[:, None, None] for k, v in tab.items()}
    Pz = _diff_z(P, dz)
    Bx = _walls(model.alpha * _diff(P, 1, dy) + _diff(Pz, 2, dx), 0.0)
    By = _walls(-model.alpha * _diff(P, 2, dx) + _diff(Pz, 1, dy), 0.0)
    del Pz
    Bz = _walls(-(_diff2(P, 2, dx) + _diff2(P, 1, dy)), 0.0)
    p = _walls(col["pb"] - col["xi"] * Bz * Bz / (2.0 * model.mu0), tab["pb"])
    slope = Bx * _diff(Bz, 2, dx) + By * _diff(Bz, 1, dy) + Bz * _diff_z(Bz, dz)
    rho = col["rhob"] + (col["dxi"] * Bz * Bz / (2.0 * model.mu0) + col["xi"] * slope / model.mu0) / model.g
    return Bx, By, Bz, p, _walls(rho, tab["rhob"])


def _exact_diagnostics(g, model, Bx, By, Bz, p, rho):
    dx, dy, dz = g.lx / (g.nx - 1), g.ly / (g.ny - 1), g.lz / (g.nz - 1)
    jx = (_diff(Bz, 1, dy) - _diff_z(By, dz)) / model.mu0
    jy = (_diff_z(Bx, dz) - _diff(Bz, 2, dx)) / model.mu0
    jz = (_diff(By, 2, dx) - _diff(Bx, 1, dy)) / model.mu0
    fx = jy * Bz - jz * By - _diff(p, 2, dx)
    fy = jz * Bx - jx * Bz - _diff(p, 1, dy)
    fz = jx * By - jy * Bx - _diff_z(p, dz) - rho * model.g
    div = _diff(Bx, 2, dx) + _diff(By, 1, dy) + _diff_z(Bz, dz)
    return [_walls(t, 0.0) for t in (jx, jy, jz, torch.sqrt(fx * fx + fy * fy + fz * fz), div)]


def _exact_general(a, b, c, u, lengths):
    """u with its interior the solution of a lap u + b u = c: conjugate gradients on -lap u - (b/a) u = -c/a with the
    exact solver of -lap as preconditioner (b <= 0 < a)."""
    dev, shape = u.device, u.shape
    hs = [length / (n - 1) for n, length in zip(shape[::-1], lengths)][::-1]
    mid = tuple(slice(1, -1) for _ in shape)
    bases = [_sine(n, h, dev) for n, h in zip(shape, hs)]
    lam = sum(lv.reshape([-1 if q == k else 1 for q in range(len(shape))]) for k, (_, lv) in enumerate(bases))

    def sines(t):
        for k, (S, _) in enumerate(bases):
            t = torch.movedim(torch.tensordot(S, t, dims=([1], [k])), 0, k).contiguous()
        return t

    full = torch.zeros_like(u)

    def minus_lap(v):
        return -sum(_diff2(v, k, h) for k, h in enumerate(hs))[mid]

    beta = (b / a)[mid]
    u = u.clone()
    u[mid] = 0.0
    r = -(c / a)[mid] - minus_lap(u)
    x, p, old, best = torch.zeros_like(r), None, None, None
    for _ in range(60):
        z = sines(sines(r) / lam)
        rz = float((r * z).sum())
        if best is not None and rz <= 1e-30 * best:
            break
        best = rz if best is None else best
        p = z if p is None else z + (rz / old) * p
        full[mid] = p
        q = minus_lap(full) - beta * p
        step = rz / float((p * q).sum())
        x += step * p
        r = r - step * q
        old = rz
    u[mid] = x
    return u


def _exact_lines(g, B, seeds, ds, max_steps):
    dev = seeds.device
    n = seeds.shape[0]
    size = torch.tensor([g.lx, g.ly, g.lz], dtype=torch.float64, device=dev)
    cells = torch.tensor([g.nx - 1, g.ny - 1, g.nz - 1], dtype=torch.float64, device=dev)
    h = size / cells
    flat = torch.stack([t.reshape(-1) for t in B], 1)
    lerp = lambda u, v, w: u + w * (v - u)  # noqa: E731

    def direction(x):
        q = torch.minimum(torch.clamp(x, min=0.0), size) / h
        i = torch.minimum(torch.floor(q), cells - 1.0)
        w = q - i
        i = i.to(torch.int64)
        at = i[:, 0] + g.nx * (i[:, 1] + g.ny * i[:, 2])
        wx, wy, wz = w[:, :1], w[:, 1:2], w[:, 2:]
        rows = [lerp(flat[at + o], flat[at + o + 1], wx) for o in (0, g.nx, g.nx * g.ny, g.nx * (g.ny + 1))]
        v = lerp(lerp(rows[0], rows[1], wy), lerp(rows[2], rows[3], wy), wz)
        size_v = torch.sqrt(v[:, 0] * v[:, 0] + v[:, 1] * v[:, 1] + v[:, 2] * v[:, 2])
        return v / torch.where(size_v > 0.0, size_v, torch.ones_like(size_v))[:, None], size_v > 0.0

    pts = torch.zeros((max_steps + 1, n, 3), dtype=torch.float64, device=dev)
    pts[0] = seeds
    on = ((seeds >= 0.0) & (seeds <= size)).all(1)
    x = seeds
    for step in range(max_steps):
        if not bool(on.any()):
            break
        k1, a = direction(x)
        k2, b = direction(x + (0.5 * ds) * k1)
        k3, c = direction(x + (0.5 * ds) * k2)
        k4, d = direction(x + ds * k3)
        x = x + (ds / 6.0) * (((k1 + 2.0 * k2) + 2.0 * k3) + k4)
        on = on & a & b & c & d & ((x >= 0.0) & (x <= size)).all(1)
        pts[step + 1][on] = x[on]
    return pts


def exact(case, seed):
    device = DEVICE if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    nodes = case["nx"] * case["ny"] * case["nz"] if "nx" in case else sum(
        x * y * z for x, y, z in SERVE_SHAPES[case["shapes"]]) * case["requests"]
    if device == "cpu" and nodes > 3_000_000:
        return None
    s = _inputs(case, seed, device)

    def equilibrium(g, model, bz0):
        P = torch.zeros(g.shape, dtype=torch.float64, device=device)
        P[0] = _exact_base(bz0, g)
        P = _exact_interior(P, g, model)
        return (P,) + tuple(_exact_fields(P, g, model))

    if kind == "serve":
        return [torch.stack([t.reshape(-1) for t in equilibrium(g, m, torch.from_numpy(bz0).to(device))])
                for g, m, bz0 in s.requests]
    if kind == "equilibrium":
        return equilibrium(s.g, s.model, s.bz0)
    if kind == "interior":
        return _exact_interior(s.P, s.g, s.model)
    if kind == "general":
        return _exact_general(s.a, s.b, s.c, s.u, (s.g.lx, s.g.ly, s.g.lz))
    if kind == "face":
        view = _face_view(s.P, case["face"])
        view.copy_(_exact_general(s.a, s.b, s.c, view.clone(), [case[k] for k in _face_lengths(case)]))
        return s.P
    if kind == "fields":
        return _exact_fields(s.P, s.g, s.model)
    if kind == "diagnostics":
        return _exact_diagnostics(s.g, s.model, *s.B, s.p, s.rho)
    return _exact_lines(s.g, s.B, s.seeds, case["ds"] * s.g.lx / (s.g.nx - 1), case["max_steps"]), None, None
