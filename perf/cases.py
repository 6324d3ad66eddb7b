"""The performance cases: what a user of libelwh has it do, through the Python
binding, over the sizes that the framework serves.

Kinds of case:

  square   one 2-D Cartesian problem: a filter application, an application of
           A_h (the body of a CG iteration), or a short CG solve
  cube     the same applications on a 3-D Cartesian grid, FP64 or FP32 stepping
  sector   A_h on a mapped 2-D grid (the annular sectors of the
           iterations-against-frequency experiment)
  shell    A_h on a mapped 3-D grid (the partial toroidal shell, free radial
           faces)
  openbox  the two-field operator with every face absorbing: GMRES iterations
  batch    a ragged batch of 2-D problems solved together
  net      the warm-start network: inference, or loss and gradient

Inputs are smooth random media (log-normal, correlation length 0.1, as the
benchmark's), Gaussian sources and smooth random fields, made on the GPU from
the case's seed.  Reference values (exact) come from a discrete strain energy
differentiated by torch's autograd in float64.
"""

import math

import numpy as np
import torch

DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # the 64^2 constant-medium problem of the tests, one filter application: launches and latency
        {"name": "square64_filter", "kind": "square", "call": "filter", "nx": 64, "ny": 64, "omega": 10.0},
        # one CG iteration's A_h on a warm-start problem (256^2, omega in 20..60)
        {"name": "square256_A", "kind": "square", "call": "A", "nx": 256, "ny": 256, "omega": 40.0},
        # one CG iteration's A_h on the benchmark's workload (1024^2, ten points per shear wavelength)
        {"name": "square1024_A", "kind": "square", "call": "A", "nx": 1024, "ny": 1024, "omega": 470.0},
        # a short CG solve on a grid of odd, unequal sides: the Krylov vector work beside the steps
        {"name": "rect_cg", "kind": "square", "call": "cg", "nx": 611, "ny": 373, "omega": 120.0},
        # the layered 3-D cube, FP64, at a medium size
        {"name": "cube128_A", "kind": "cube", "prec": "f64", "nx": 128, "ny": 128, "nz": 128, "omega": 89.0},
        # the 3-D cube with FP32 stepping at 256^3, the size the benchmark quotes it at
        {"name": "cube256_f32_A", "kind": "cube", "prec": "f32", "nx": 256, "ny": 256, "nz": 256, "omega": 178.6},
        # the benchmark's mapped 2-D grid: quarter annulus, 801 x 4003 cells
        {"name": "sector_A", "kind": "sector", "nq": 801, "nr": 4003, "annulus": 1, "omega": 200.14},
        # the toroidal shell at the paper's smaller size, 400 x 120 x 40 points
        {"name": "shell_A", "kind": "shell", "nq": 399, "nr": 119, "ns": 39, "omega": 5.1234},
        # absorbing boundaries: GMRES iterations on the 1024^2 open box
        {"name": "openbox_gmres", "kind": "openbox", "nx": 1024, "ny": 1024, "omega": 470.0, "iters": 12},
        # a ragged batch: sizes 256..1024, omega 20..80, a few CG iterations of every problem
        {"name": "batch16", "kind": "batch", "nprob": 16, "nmin": 256, "nmax": 1024, "wmin": 20.0, "wmax": 80.0,
         "iters": 3},
        # inference of the warm-start network for a batch of 48 problems
        {"name": "net_forward48", "kind": "net", "call": "forward", "batch": 48, "size": 256},
        # its training batch: loss and gradient of 16 samples
        {"name": "net_grad16", "kind": "net", "call": "grad", "batch": 16, "size": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["square", "square", "square", "cube", "cube", "sector", "shell", "openbox", "batch", "net"])
    if kind == "square":
        nx, ny = _log_int(rng, 40, 1500), _log_int(rng, 40, 1500)
        n = max(nx, ny)
        return {"kind": kind, "call": rng.choice(["filter", "A", "cg"]), "nx": nx, "ny": ny,
                "omega": round(0.46 * n / rng.uniform(1.0, 6.0), 3)}
    if kind == "cube":
        nx, ny, nz = (_log_int(rng, 20, 200) for _ in range(3))
        return {"kind": kind, "prec": rng.choice(["f64", "f32"]), "nx": nx, "ny": ny, "nz": nz,
                "omega": round(0.7 * max(nx, ny, nz) / rng.uniform(1.0, 3.0), 3)}
    if kind == "sector":
        nq = _log_int(rng, 40, 800)
        return {"kind": kind, "nq": nq, "nr": int(nq * rng.uniform(2.0, 5.0)), "annulus": rng.choice([1, 2]),
                "omega": round(nq / rng.uniform(4.0, 8.0), 3)}
    if kind == "shell":
        ns = rng.randint(6, 38)
        return {"kind": kind, "nq": int(ns * rng.uniform(6.0, 10.0)), "nr": int(ns * rng.uniform(2.5, 3.5)), "ns": ns,
                "omega": round(ns / rng.uniform(5.0, 8.0), 4)}
    if kind == "openbox":
        nx, ny = _log_int(rng, 64, 1000), _log_int(rng, 64, 1000)
        return {"kind": kind, "nx": nx, "ny": ny, "omega": round(0.46 * max(nx, ny) / rng.uniform(1.0, 3.0), 3),
                "iters": rng.randint(4, 12)}
    if kind == "batch":
        nmin = _log_int(rng, 64, 400)
        return {"kind": kind, "nprob": rng.randint(2, 12), "nmin": nmin, "nmax": int(nmin * rng.uniform(1.0, 2.5)),
                "wmin": 20.0, "wmax": round(rng.uniform(30.0, 80.0), 2), "iters": rng.randint(2, 3)}
    return {"kind": kind, "call": rng.choice(["forward", "grad"]), "batch": rng.randint(1, 16),
            "size": 16 * rng.randint(4, 16)}


# ---- inputs (torch only, from the seed alone) ---------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _grf(shape, h, ell, gen):
    """Smooth Gaussian random field of correlation length ell, zero mean, unit
    deviation (periodic; h per array axis)."""
    spec = torch.fft.rfftn(torch.randn(shape, generator=gen, device=DEV, dtype=F64))
    k2 = torch.zeros((), device=DEV, dtype=F64)
    for a, n in enumerate(shape):
        freq = torch.fft.rfftfreq if a == len(shape) - 1 else torch.fft.fftfreq
        k = 2 * math.pi * freq(n, d=h[a], device=DEV, dtype=F64)
        k2 = k2 + (k * k).reshape([-1 if b == a else 1 for b in range(len(shape))])
    g = torch.fft.irfftn(spec * torch.exp(-0.25 * ell * ell * k2), s=shape)
    g = g - g.mean()
    return (g / g.std()).contiguous()


def _random_media(shape, h, gen):
    """Log-normal rho and mu, lambda / mu in [1, 3]."""
    g1, g2, g3 = (_grf(shape, h, 0.1, gen) for _ in range(3))
    rho, mu = torch.exp(0.2 * g1), torch.exp(0.2 * g2)
    return rho, mu * torch.clamp(2.0 * torch.exp(0.2 * g3), 1.0, 3.0), mu


def _gaussians(shape, h, gen, count, width):
    """Sum of `count` Gaussian sources of the given width, random directions."""
    d = len(shape)
    f = torch.zeros((d,) + tuple(shape), device=DEV, dtype=F64)
    for _ in range(count):
        at = 0.2 + 0.6 * torch.rand(d, generator=gen, device=DEV, dtype=F64)
        e = torch.randn(d, generator=gen, device=DEV, dtype=F64)
        r2 = torch.zeros((), device=DEV, dtype=F64)
        for a, n in enumerate(shape):
            x = torch.arange(n, device=DEV, dtype=F64) * h[a] - at[a] * (n - 1) * h[a]
            r2 = r2 + (x * x).reshape([-1 if b == a else 1 for b in range(d)])
        f += (e / e.norm()).reshape([-1] + [1] * d) * torch.exp(-r2 / (2 * width * width))
    return f


def _field(shape, gen):
    """A vector field as a Krylov direction is: smooth over a few nodes."""
    return torch.stack([_grf(shape, [1.0] * len(shape), 4.0, gen) for _ in range(len(shape))])


def _sector_nodes(nq, nr, annulus):
    """Annular sector: q radial (r_out - r_in = 1), r along the outer arc of length 5."""
    r_out = 10.0 / (annulus * math.pi)
    q = torch.arange(nq + 1, device=DEV, dtype=F64) / nq
    r = torch.arange(nr + 1, device=DEV, dtype=F64) / nr
    rad = (r_out - 1.0 + q)[None, :]
    th = (0.5 * math.pi * annulus * r - 0.5 * math.pi)[:, None]
    return [rad * torch.cos(th), rad * torch.sin(th)]


def _shell_nodes(nq, nr, ns):
    """Partial toroidal shell of major radius 4 and minor radius 1..2: q, r, s -> phi, theta, radius."""
    ph = (math.pi * torch.arange(nq + 1, device=DEV, dtype=F64) / nq)[None, None, :]
    th = (math.pi * torch.arange(nr + 1, device=DEV, dtype=F64) / nr)[None, :, None]
    rad = (1.0 + torch.arange(ns + 1, device=DEV, dtype=F64) / ns)[:, None, None]
    ring = 4.0 + rad * torch.cos(th)
    return [ring * torch.cos(ph), ring * torch.sin(ph), (rad * torch.sin(th)).expand(ns + 1, nr + 1, nq + 1)]


def _problem(case, seed):
    """Grid, media, forcing and a field of one single-problem case, on the GPU."""
    gen = _gen(seed)
    kind = case["kind"]
    p = {"omega": case["omega"], "nodes": None, "impedance": kind == "openbox"}
    if kind in ("square", "openbox", "cube"):
        p["n"] = (case["nx"], case["ny"]) + ((case["nz"],) if kind == "cube" else ())
        # cells are square; the longest side has length 1
        p["h"] = [1.0 / max(p["n"])] * len(p["n"])
        p["bc"] = {"square": (0, 0, 0, 1), "openbox": (2, 2, 2, 2), "cube": (0,) * 6}[kind]
    elif kind == "sector":
        p["n"], p["bc"] = (case["nq"], case["nr"]), (0, 0, 0, 0)
        p["nodes"] = _sector_nodes(case["nq"], case["nr"], case["annulus"])
    else:
        p["n"], p["bc"] = (case["nq"], case["nr"], case["ns"]), (0, 0, 0, 0, 1, 1)
        p["nodes"] = _shell_nodes(case["nq"], case["nr"], case["ns"])
    shape = tuple(k + 1 for k in reversed(p["n"]))
    p["shape"] = shape
    one = torch.ones(shape, device=DEV, dtype=F64)
    if p["nodes"] is not None:
        p["h"] = [1.0 / k for k in p["n"]]
    hs = list(reversed(p["h"]))
    if kind == "shell":
        rho, lam, mu = one, 2.0 * one, one.clone()
    elif kind == "cube":
        # three layers along z with 5% smooth perturbations
        z = (torch.arange(shape[0], device=DEV, dtype=F64) / (shape[0] - 1)).reshape(-1, 1, 1)
        cs = torch.where(z < 1 / 3, 2.0, torch.where(z < 2 / 3, 1.5, 1.0))
        rho = torch.where(z < 1 / 3, 1.5, torch.where(z < 2 / 3, 1.2, 1.0)) * one
        mu = rho * cs * cs
        rho, lam, mu = (m * (1.0 + 0.05 * torch.clamp(_grf(shape, hs, 0.1, gen), -3.0, 3.0))
                        for m in (rho, 2.0 * mu, mu))
    elif kind == "square" and case["nx"] == case["ny"] == 64:
        rho, lam, mu = one, 2.0 * one, one.clone()
    else:
        rho, lam, mu = _random_media(shape, hs if kind != "sector" else [5.0 / p["n"][1], 1.0 / p["n"][0]], gen)
    p["rho"], p["lam"], p["mu"] = rho.contiguous(), lam.contiguous(), mu.contiguous()
    width = 3.2 * max(p["h"])
    p["f"] = _gaussians(shape, hs, gen, 2, width)
    p["x"] = _field(shape, gen)
    return p


# the network: (inputs, outputs, SiLU) per 3x3 convolution, parameters in this order
_LAYERS = [(7, 32, 1), (32, 32, 1), (32, 64, 1), (64, 64, 1), (64, 96, 1), (96, 96, 1), (96, 128, 1), (128, 128, 1),
           (128, 128, 1), (128, 128, 1), (256, 128, 1), (128, 128, 1), (224, 96, 1), (96, 96, 1), (160, 64, 1),
           (64, 64, 1), (96, 32, 1), (32, 32, 1), (32, 2, 0)]


def _net_inputs(case, seed):
    gen = _gen(seed)
    B, n = case["batch"], case["size"]
    x = torch.empty((B, n, n, 7), device=DEV, dtype=torch.float32)
    for b in range(B):
        for c in range(7):
            # media logarithms, forcing components, then the two constants
            x[b, :, :, c] = (_grf((n, n), [1.0 / n] * 2, 0.1 if c < 3 else 0.02, gen) if c < 5
                             else 0.3 + 0.5 * torch.rand((), generator=gen, device=DEV, dtype=F64)).to(torch.float32)
    y = torch.randn((B, n, n, 2), generator=gen, device=DEV, dtype=torch.float32)
    w = 0.5 + torch.rand((B, n, n), generator=gen, device=DEV, dtype=torch.float32)
    theta = []
    for ci, co, _ in _LAYERS:
        theta.append(torch.randn(9 * ci * co, generator=gen, device=DEV, dtype=F64) * math.sqrt(2.0 / (9 * ci)))
        theta.append(0.05 * torch.randn(co, generator=gen, device=DEV, dtype=F64))
    return x, y, w, torch.cat(theta).to(torch.float32)


def _batch_problems(case, seed):
    gen = _gen(seed)
    rng = np.random.default_rng(7000)          # the batch's sizes belong to the case
    out = []
    for _ in range(case["nprob"]):
        n = int(rng.integers(case["nmin"], case["nmax"] + 1))
        omega = float(rng.uniform(case["wmin"], case["wmax"]))
        shape, h = (n + 1, n + 1), [1.0 / n] * 2
        rho, lam, mu = _random_media(shape, h, gen)
        out.append((n, omega, rho, lam, mu, _gaussians(shape, h, gen, 2, 3.2 / n)))
    return out


# ---- the measured calls -----------------------------------------------------------


def prepare(case, seed):
    from paper_2205_12344_amd import elwh, inputs
    kind = case["kind"]
    if kind == "net":
        x, y, w, theta = _net_inputs(case, seed)
        net = elwh.WarmStartNet(max_batch=case["batch"], H=case["size"])
        net.set_params(theta.cpu().numpy())
        return {"case": case, "net": net, "x": x, "y": y, "w": w}
    if kind == "batch":
        probs = _batch_problems(case, seed)
        cases = [inputs.Case(f"p{k}", 2, (n, n), om, rho, lam, mu, None, inputs.BC_FREE_TOP_2D)
                 for k, (n, om, rho, lam, mu, _) in enumerate(probs)]
        return {"case": case, "batch": elwh.Batch(cases), "f": [p[5] for p in probs]}
    p = _problem(case, seed)
    if kind == "sector":
        ctx = elwh.MappedContext(*p["nodes"], p["rho"], p["lam"], p["mu"], p["omega"], bc=p["bc"])
    elif kind == "shell":
        ctx = elwh.MappedContext3(*p["nodes"], p["rho"], p["lam"], p["mu"], p["omega"], bc=p["bc"])
    else:
        opts = {"prec": elwh.FP32_STEP} if case.get("prec") == "f32" else {}
        length = [k * h for k, h in zip(p["n"], p["h"])]
        ctx = elwh.Context(len(p["n"]), p["n"], p["rho"], p["lam"], p["mu"], p["omega"], p["bc"], length=length,
                           **opts)
    return {"case": case, "ctx": ctx, "x": p["x"], "f": p["f"], "out": torch.empty_like(p["x"])}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "net":
        if case["call"] == "forward":
            return state["net"].forward(state["x"])
        loss, grad = state["net"].loss_grad(state["x"], state["y"], state["w"])
        return [grad, np.float32(loss)]
    if kind == "batch":
        vs, _, _ = state["batch"].solve(state["f"], tol=0.0, maxit=case["iters"])
        return vs
    ctx = state["ctx"]
    if kind == "openbox":
        v0, v1, _ = ctx.solve2(state["f"], tol=0.0, maxit=case["iters"])
        return [v0, v1]
    call = case.get("call", "A")
    if call == "filter":
        return ctx.apply_filter(state["x"], state["f"], out=state["out"])
    if call == "cg":
        v, _ = ctx.solve(state["f"], tol=0.0, maxit=_CG_ITERS)
        return v
    return ctx.apply_A(state["x"], out=state["out"])


_CG_ITERS = 8


def _steps(omega, h, speed):
    """Estimated steps per period: the time-step rule with the radius of a uniform medium."""
    return max(3, math.ceil(2 * math.pi / omega * speed / (0.8 * h)))


def work(case):
    """Bytes: inputs and coefficients read once, outputs written once; flops of
    the stencil, leapfrog and filter sum over all steps (or of the
    convolutions)."""
    kind = case["kind"]
    if kind == "net":
        pix, macs, size = case["batch"] * case["size"] ** 2, 0, 0
        level = [0, 0, 1, 1, 2, 2, 3, 3, 4, 4, 3, 3, 2, 2, 1, 1, 0, 0, 0]
        for (ci, co, _), lev in zip(_LAYERS, level):
            macs += 9 * ci * co * pix // 4 ** lev
            size += 9 * ci * co + co
        if case["call"] == "forward":
            return {"bytes": 4 * (pix * (7 + 2) + size), "flops": 2 * macs}
        return {"bytes": 4 * (pix * (7 + 2 + 1) + 2 * size), "flops": 6 * macs}
    if kind == "batch":
        rng = np.random.default_rng(7000)
        nbytes = flops = 0
        for _ in range(case["nprob"]):
            n, om = int(rng.integers(case["nmin"], case["nmax"] + 1)), float(rng.uniform(case["wmin"], case["wmax"]))
            applies = case["iters"] + 1
            nbytes += 8 * (3 + 2 + 2) * n * n
            flops += 75 * n * n * _steps(om, 1.0 / n, 3.7) * applies
        return {"bytes": nbytes, "flops": flops}
    if kind in ("square", "openbox"):
        nodes, h = case["nx"] * case["ny"], 1.0 / max(case["nx"], case["ny"])
        nt = _steps(case["omega"], h, 2.24 if case["nx"] == case["ny"] == 64 else 3.7)
        if kind == "openbox":
            applies = case["iters"] + 2                # right-hand side, iterations, final residual
            return {"bytes": 8 * (3 + 2 + 4) * nodes, "flops": 82 * nodes * nt * applies}
        applies = _CG_ITERS + 2 if case["call"] == "cg" else 1
        fields = 6 if case["call"] == "filter" else 4
        return {"bytes": 8 * (3 + fields) * nodes, "flops": 75 * nodes * nt * applies}
    if kind == "cube":
        nodes, h = case["nx"] * case["ny"] * case["nz"], 1.0 / max(case["nx"], case["ny"], case["nz"])
        return {"bytes": 8 * (3 + 6) * nodes, "flops": 190 * nodes * _steps(case["omega"], h, 6.1)}
    if kind == "sector":
        nodes = case["nq"] * case["nr"]
        h = min(1.0 / case["nq"], 5.0 / case["nr"])
        return {"bytes": 8 * (7 + 4) * nodes, "flops": 120 * nodes * _steps(case["omega"], h, 4.7)}
    nodes, h = case["nq"] * case["nr"] * case["ns"], min(1.0 / case["ns"], math.pi / case["nr"])
    return {"bytes": 8 * (12 + 6) * nodes, "flops": 500 * nodes * _steps(case["omega"], h, 4.1)}


# ---- reference values in 64 bits -----------------------------------------------------


def _node_diff(U, dim, h):
    """Central difference along `dim`, one-sided at the ends (used on
    traction-type faces; the value on a Dirichlet face is not)."""
    n = U.shape[dim]
    inner = (U.narrow(dim, 2, n - 2) - U.narrow(dim, 0, n - 2)) / (2 * h)
    first = (U.narrow(dim, 1, 1) - U.narrow(dim, 0, 1)) / h
    last = (U.narrow(dim, n - 1, 1) - U.narrow(dim, n - 2, 1)) / h
    return torch.cat([first, inner, last], dim=dim)


class _Elastic:
    """Ltilde = -W^-1 grad E of the discrete strain energy on one grid."""

    def __init__(self, p):
        self.p, self.d = p, len(p["n"])
        d, shape = self.d, p["shape"]
        self.h, self.rho = p["h"], p["rho"]
        bc = p["bc"]
        self.free = [(bc[2 * a] != 0, bc[2 * a + 1] != 0) for a in range(d)]
        one = torch.ones(shape, device=DEV, dtype=F64)
        self.wax = []                       # trapezoid weight of each axis
        self.mask = one.clone()             # 1 on unknown nodes
        for a in range(d):
            w = torch.ones(shape[d - 1 - a], device=DEV, dtype=F64)
            m = w.clone()
            for end, free in zip((0, -1), self.free[a]):
                if free:
                    w[end] = 0.5
                else:
                    m[end] = 0.0
            sh = [-1 if k == d - 1 - a else 1 for k in range(d)]
            self.wax.append(w.reshape(sh))
            self.mask = self.mask * m.reshape(sh)
        self.wn = one.clone()
        for w in self.wax:
            self.wn = self.wn * w
        if p["nodes"] is None:
            self.J = one
            self.G = [[1.0 if c == a else 0.0 for c in range(d)] for a in range(d)]
        else:
            self._metric()
        self.lamJ, self.muJ = p["lam"] / self.J, p["mu"] / self.J
        self.GG = [[self._dot(self.G[a], self.G[b]) for b in range(d)] for a in range(d)]

    def _metric(self):
        d, X = self.d, [x.contiguous() for x in self.p["nodes"]]

        def diff(x, a):
            k, h, n = d - 1 - a, self.h[a], x.shape[d - 1 - a]
            s = lambda i: x.narrow(k, i if i >= 0 else n + i, 1)  # noqa: E731
            inner = (x.narrow(k, 2, n - 2) - x.narrow(k, 0, n - 2)) / (2 * h)
            first = (-3 * s(0) + 4 * s(1) - s(2)) / (2 * h)
            last = (3 * s(-1) - 4 * s(-2) + s(-3)) / (2 * h)
            return torch.cat([first, inner, last], dim=k)

        T = [[diff(x, a) for x in X] for a in range(d)]    # T[a][c] = d x_c / d a
        if d == 2:
            (xq, yq), (xr, yr) = T
            self.J = xq * yr - xr * yq
            self.G = [[yr, -xr], [-yq, xq]]
            return
        cross = lambda u, v: [u[1] * v[2] - u[2] * v[1], u[2] * v[0] - u[0] * v[2], u[0] * v[1] - u[1] * v[0]]  # noqa: E731
        self.G = [cross(T[1], T[2]), cross(T[2], T[0]), cross(T[0], T[1])]
        self.J = self._dot(T[0], self.G[0])

    @staticmethod
    def _dot(u, v):
        return sum(a * b for a, b in zip(u, v) if not (isinstance(a, float) and a == 0.0)
                   and not (isinstance(b, float) and b == 0.0))

    def energy(self, U):
        d, E = self.d, 0.0
        Dn = []
        for a in range(d):
            k, h = d - 1 - a, self.h[a]
            n = U.shape[k + 1]
            D = [(U[c].narrow(k, 1, n - 1) - U[c].narrow(k, 0, n - 1)) / h for c in range(d)]
            w = 0.5
            for b in range(d):
                if b != a:
                    w = w * self.wax[b]
            dd = self._dot(D, D)
            for off in (0, 1):          # the edge's block is the mean of its two nodes'
                at = lambda q: q if isinstance(q, float) else q.narrow(k, off, n - 1)  # noqa: E731,B023
                gd = self._dot([at(g) for g in self.G[a]], D)
                E = E + (0.5 * w * ((at(self.lamJ) + at(self.muJ)) * gd * gd
                                    + at(self.muJ) * at(self.GG[a][a]) * dd)).sum()
            Dn.append([_node_diff(U[c], k, h) for c in range(d)])
        wn = self.wn * self.mask
        for a in range(d):
            for b in range(a + 1, d):
                A, B, Ga, Gb = Dn[a], Dn[b], self.G[a], self.G[b]
                e = self.lamJ * self._dot(Ga, A) * self._dot(Gb, B) + self.muJ * self._dot(Gb, A) * self._dot(Ga, B)
                if self.p["nodes"] is not None:
                    e = e + self.muJ * self.GG[a][b] * self._dot(A, B)
                E = E + (wn * e).sum()
        return E

    def apply(self, u):
        """Ltilde u = W^-1 L_h u on the unknown nodes (W = J w)."""
        v = (u * self.mask).detach().requires_grad_(True)
        with torch.enable_grad():
            g, = torch.autograd.grad(self.energy(v), v)
        return -g * self.mask / (self.J * self.wn)

    def gershgorin(self):
        """max over the unknown rows of sum_j |(rho^-1 Ltilde)_ij|, from probes
        that are 1 on every third node of each axis, one component at a time."""
        d, rows = self.d, 0.0
        for comp in range(d):
            for colour in range(3 ** d):
                e = torch.zeros((d,) + self.p["shape"], device=DEV, dtype=F64)
                e[comp][tuple(slice((colour // 3 ** k) % 3, None, 3) for k in range(d))] = 1.0
                rows = rows + self.apply(e).abs()
        return float((rows / self.rho).max())


class _Filter:
    """Pi_h and A_h of one problem (one-field, or two-field with damping)."""

    def __init__(self, p):
        self.p, self.op = p, _Elastic(p)
        om = p["omega"]
        dt = 0.8 * 2.0 / math.sqrt(self.op.gershgorin())
        self.nt = max(3, math.ceil(2 * math.pi / om / dt))
        self.dt = 2 * math.pi / om / self.nt
        c = (math.sin(0.5 * om * self.dt) / (0.5 * om * self.dt)) ** 2
        self.a = c * self.dt ** 2 / p["rho"]
        self.cos = [math.cos(2 * math.pi * k / self.nt) for k in range(self.nt + 1)]
        self.w = [2.0 / self.nt * (0.5 if k in (0, self.nt) else 1.0) * (self.cos[k] - 0.25)
                  for k in range(self.nt + 1)]
        self.m = self.op.wn * self.op.J * p["rho"] * self.op.mask
        if p["impedance"]:
            B = torch.zeros((2,) + p["shape"], device=DEV, dtype=F64)
            cp, cs = torch.sqrt((p["lam"] + 2 * p["mu"]) / p["rho"]), torch.sqrt(p["mu"] / p["rho"])
            for axis in range(2):
                for end in (0, -1):
                    sl = (slice(None),) * (1 - axis) + (end,)
                    for comp in range(2):
                        B[comp][sl] += 2.0 / p["h"][axis] * (cp if comp == axis else cs)[sl]
            self.g = 0.5 * c * self.dt * B * om * self.dt / math.sin(om * self.dt)

    def pi(self, u0, f=None):
        op = self.op
        zero = torch.zeros_like(u0)
        f = zero if f is None else f * op.mask
        u0 = u0 * op.mask
        u1 = u0 + 0.5 * self.a * (op.apply(u0) - f * self.cos[0])
        acc = self.w[0] * u0 + self.w[1] * u1
        for n in range(1, self.nt):
            u0, u1 = u1, 2 * u1 - u0 + self.a * (op.apply(u1) - f * self.cos[n])
            acc += self.w[n + 1] * u1
        return acc

    def A(self, x):
        return x * self.op.mask - self.pi(x)

    def dot(self, x, y):
        return float((self.m * x * y).sum())

    def cg(self, f, iters):
        r = self.pi(torch.zeros_like(f), f)
        x, p, rr = torch.zeros_like(r), r.clone(), self.dot(r, r)
        for _ in range(iters):
            q = self.A(p)
            alpha = rr / self.dot(p, q)
            x += alpha * p
            r = r - alpha * q
            new = self.dot(r, r)
            p, rr = r + new / rr * p, new
        return x

    def pi2(self, u0, v0, f=None):
        """Two-field filter: filtered displacement and centred velocity."""
        op, g, dt = self.op, self.g, self.dt
        f = torch.zeros_like(u0) if f is None else f
        u1 = u0 + dt * (1 - g) * v0 + 0.5 * self.a * (op.apply(u0) - f * self.cos[0])
        acc, vel = self.w[0] * u0 + self.w[1] * u1, self.w[0] * v0
        for n in range(1, self.nt + 1):
            u2 = (2 * u1 - (1 - g) * u0 + self.a * (op.apply(u1) - f * self.cos[n])) / (1 + g)
            vel = vel + self.w[n] * (u2 - u0) / (2 * dt)
            if n < self.nt:
                acc = acc + self.w[n + 1] * u2
            u0, u1 = u1, u2
        return acc, vel

    def gmres2(self, f, iters):
        """One GMRES cycle from zero on z = [u0; u1 / omega] in the M inner product."""
        om = self.p["omega"]
        zero = torch.zeros_like(f)

        def A(z):
            a, b = self.pi2(z[0], om * z[1])
            return z - torch.stack([a, b / om])

        a, b = self.pi2(zero, zero, f)
        r = torch.stack([a, b / om])
        beta = math.sqrt(self.dot(r, r))
        V, H = [r / beta], np.zeros((iters + 1, iters))
        for j in range(iters):
            w = A(V[j])
            for _ in range(2):
                for i, v in enumerate(V):
                    s = self.dot(v, w)
                    H[i, j] += s
                    w = w - s * v
            H[j + 1, j] = math.sqrt(self.dot(w, w))
            V.append(w / H[j + 1, j])
        rhs = np.zeros(iters + 1)
        rhs[0] = beta
        y = np.linalg.lstsq(H, rhs, rcond=None)[0]
        z = sum(float(c) * v for c, v in zip(y, V))
        return [z[0], om * z[1]]


def _net_forward(theta, x):
    """The network in float64: each convolution as nine shifted products."""
    off = 0
    layers = []
    for ci, co, act in _LAYERS:
        W = theta[off:off + 9 * ci * co].reshape(9, ci, co)
        layers.append((W, theta[off + 9 * ci * co:off + 9 * ci * co + co], act))
        off += 9 * ci * co + co

    def conv(h, k):
        W, b, act = layers[k]
        H, Wd = h.shape[1:3]
        hp = torch.nn.functional.pad(h, (0, 0, 1, 1, 1, 1))
        z = b
        for t in range(9):
            z = z + hp[:, t // 3:t // 3 + H, t % 3:t % 3 + Wd, :].reshape(-1, h.shape[3]).matmul(W[t]).reshape(
                h.shape[0], H, Wd, -1)
        return z * torch.sigmoid(z) if act else z

    h, skips = x, []
    for lev in range(5):
        h = conv(conv(h, 2 * lev), 2 * lev + 1)
        skips.append(h)
        if lev < 4:
            h = 0.25 * (h[:, 0::2, 0::2] + h[:, 1::2, 0::2] + h[:, 0::2, 1::2] + h[:, 1::2, 1::2])
    for lev in (3, 2, 1, 0):
        h = h.repeat_interleave(2, 1).repeat_interleave(2, 2)
        h = torch.cat([h, skips[lev]], dim=3)
        k = 10 + 2 * (3 - lev)
        h = conv(conv(h, k), k + 1)
    return conv(h, 18)


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return None                      # many problems of hundreds of steps: too slow here
    if kind == "net":
        x, y, w, theta = _net_inputs(case, seed)
        theta = theta.double()
        if case["call"] == "forward":
            step = 8                     # samples are independent: bounded memory
            with torch.no_grad():
                return torch.cat([_net_forward(theta, x[k:k + step].double()) for k in range(0, x.shape[0], step)])
        theta.requires_grad_(True)
        total, B = 0.0, x.shape[0]
        for k in range(0, B, 4):
            yk, wk = y[k:k + 4].double(), w[k:k + 4].double()[..., None]
            yh = _net_forward(theta, x[k:k + 4].double())
            num, den = (wk * (yh - yk) ** 2).sum(dim=(1, 2, 3)), (wk * yk ** 2).sum(dim=(1, 2, 3))
            part = (num / den).sum() / B
            part.backward()
            total += float(part.detach())
        return [theta.grad, np.float64(total)]
    p = _problem(case, seed)
    with torch.no_grad():
        F = _Filter(p)
        if kind == "openbox":
            return F.gmres2(p["f"], case["iters"])
        call = case.get("call", "A")
        if call == "filter":
            return F.pi(p["x"], p["f"])
        if call == "cg":
            return F.cg(p["f"], _CG_ITERS)
        return F.A(p["x"])
