"""Workloads of the stencil-sweep library as a user's program runs them.

`listed()` names twelve calls through the package's public entry points, from
a launch-bound 2 MiB grid to 9600 x 9600 and 512^3; `draw()` gives further
ones of the same ranges (odd extents, both boundary rules, the three storage
types, every pattern of the paper's Tab. 1 and the order-4 star).  `prepare()`
makes what a program holds before the call, `run()` is one call, `exact()` is
its result in plain FP64 torch and `work()` the bytes and operations it cannot
do without.

A case is a dict of plain values:
  kind     "grid": Plan.run / run_flux / adjoint on one grid;
           "batch": BatchPlan.run on many uneven 2D grids;
           "varcoef": StencilFn forward and backward.
  ndim, pattern ("star" / "box"), radius, nz, ny, nx, dtype, bc, steps
  call     "run", "flux" (outflow account) or "adjoint" (transposed sweep)
  graph    replay the run's launches from a HIP graph (ST_PLAN_GRAPH)
"""
import math

import numpy as np
import torch

import paper_2303_08365_amd as st

_TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
_BYTES = {"f64": 8, "f32": 4, "bf16": 2}
_DEV = "cuda"


def _grid(name, ndim, pattern, radius, shape, dtype, bc, steps, call="run", graph=False):
    nz, ny, nx = (1,) * (3 - ndim) + tuple(shape)
    return {"name": name, "kind": "grid", "ndim": ndim, "pattern": pattern, "radius": radius, "nz": nz, "ny": ny,
            "nx": nx, "dtype": dtype, "bc": bc, "steps": steps, "call": call, "graph": graph}


def listed():
    return [
        # the small everyday call: 2 MiB, whole run in one call, launch and
        # latency bound; a stepping loop that repeats it replays a graph
        _grid("heat2d-f64-512", 2, "star", 1, (512, 512), "f64", "zero", 100, graph=True),
        # a small 3D domain with odd extents, a few steps per call (a solver
        # that looks at its field between calls)
        _grid("heat3d-f32-odd97", 3, "star", 1, (89, 97, 101), "f32", "zero", 10),
        # the library's headline: 3D heat in FP64
        _grid("heat3d-f64-512", 3, "star", 1, (512, 512, 512), "f64", "zero", 100),
        # an ordinary production domain: no extent a round number
        _grid("heat3d-f64-ragged", 3, "star", 1, (251, 319, 377), "f64", "zero", 50),
        # order-4 wave-type star, periodic box, FP32
        _grid("star25-f32-512", 3, "star", 4, (512, 512, 512), "f32", "periodic", 50),
        # smoothing with the 9-point box on a large periodic image-like grid
        _grid("box9-f32-8192", 2, "box", 1, (8192, 8192), "f32", "periodic", 200),
        # 27-point box (multigrid-smoother shape), FP64
        _grid("box27-f64-512", 3, "box", 1, (512, 512, 512), "f64", "zero", 20),
        # reverse mode through a constant-weight radius-2 star, ragged sizes
        _grid("star9-f64-adjoint", 2, "star", 2, (2999, 4099), "f64", "zero", 60, call="adjoint"),
        # long 1D rod
        _grid("heat1d-f64-1e7", 1, "star", 1, (10_000_000,), "f64", "zero", 1000),
        # bfloat16 storage with the FP64 outflow account, large and not cubic
        _grid("heat3d-bf16-flux", 3, "star", 1, (300, 420, 500), "bf16", "zero", 30, call="flux"),
        # ensemble of 64 uneven 2D grids, own coefficients, one launch per pass
        {"name": "batch64-f32", "kind": "batch", "count": 64, "lo": 256, "hi": 4096, "shape_seed": 0, "dtype": "f32",
         "bc": "zero", "steps": 200},
        # conductivity and initial-field gradients through 200 steps with
        # checkpoints every 20
        {"name": "varcoef-f32-256", "kind": "varcoef", "nz": 256, "ny": 256, "nx": 256, "dtype": "f32", "steps": 200,
         "every": 20},
    ]


# Cell updates (weighted by points) a drawn case may cost: below the headline's.
_MAX_POINT_STEPS = 512 ** 3 * 100 * 5


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extent(rng, lo, hi):
    """Log-uniform; half of them even multiples of 16 as programs like them,
    the rest as they come (mostly odd or ragged)."""
    n = _log_int(rng, lo, hi)
    return max(lo, 16 * (n // 16)) if rng.random() < 0.5 else n


def draw(rng):
    kind = rng.choice(["grid"] * 8 + ["batch", "varcoef"])
    if kind == "batch":
        lo = _log_int(rng, 64, 256)
        return {"kind": "batch", "count": _log_int(rng, 4, 64), "lo": lo, "hi": lo * rng.randint(2, 12),
                "shape_seed": rng.randrange(1000), "dtype": rng.choice(["f32", "f64"]),
                "bc": rng.choice(["zero", "periodic"]), "steps": _log_int(rng, 20, 200)}
    if kind == "varcoef":
        steps = _log_int(rng, 10, 100)
        return {"kind": "varcoef", "nz": _extent(rng, 48, 256), "ny": _extent(rng, 48, 256),
                "nx": _extent(rng, 48, 256), "dtype": rng.choice(["f32", "f32", "f64"]), "steps": steps,
                "every": rng.randint(4, 20)}
    ndim, pattern, radius = rng.choice([(2, "star", 1), (2, "star", 1), (3, "star", 1), (3, "star", 1), (3, "star", 1),
                                        (1, "star", 1), (1, "star", 2), (2, "box", 1), (2, "star", 2), (2, "box", 2),
                                        (3, "box", 1), (3, "star", 4)])
    lo, hi = {1: (10_000, 10_000_000), 2: (200, 8192), 3: (48, 512)}[ndim]
    shape = tuple(_extent(rng, lo, hi) for _ in range(ndim))
    points = 1 + 2 * ndim * radius if pattern == "star" else (2 * radius + 1) ** ndim
    room = max(2, int(_MAX_POINT_STEPS / (points * math.prod(shape))))
    steps = min(room, _log_int(rng, 4, 100) * (10 if ndim == 1 else 1))
    dtype = rng.choice(["f64", "f64", "f32", "f32", "bf16"])
    bc = rng.choice(["zero", "zero", "periodic"])
    call = rng.choice(["run"] * 6 + ["flux", "adjoint"])
    c = _grid("", ndim, pattern, radius, shape, dtype, "zero" if call == "flux" else bc, steps, call,
              call == "run" and rng.random() < 0.25)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _shape(c):
    return (c["nz"], c["ny"], c["nx"])[3 - c["ndim"]:] if c["kind"] == "grid" else (c["nz"], c["ny"], c["nx"])


def _offsets(ndim, pattern, radius):
    centre = (0,) * ndim
    if pattern == "star":
        return [centre] + [tuple(s * d if a == ax else 0 for a in range(ndim)) for ax in range(ndim)
                           for d in range(1, radius + 1) for s in (-1, 1)]
    out = [()]
    for _ in range(ndim):
        out = [o + (d,) for o in out for d in range(-radius, radius + 1)]
    return [centre] + [o for o in out if o != centre]


def _round_w(w, dtype):
    """Weights as the computation holds them, the centre closing their sum to 1."""
    w = [float(v) if dtype == "f64" else float(np.float32(v)) for v in w]
    w[0] = 1.0 - math.fsum(w[1:])
    return [v if dtype == "f64" else float(np.float32(v)) for v in w]


def _weights(c, seed):
    points = len(_offsets(c["ndim"], c["pattern"], c["radius"]))
    if c["pattern"] == "box":
        w = [1.0 / points] * points
    elif c["radius"] == 1:
        w = [0.0] + [{1: 0.25, 2: 0.2, 3: 0.15}[c["ndim"]]] * (points - 1)
    elif c["radius"] == 2:
        w = [0.0] + [0.25 / (points - 1)] * (points - 1)
    else:
        r = np.random.default_rng(seed).random(points - 1)
        w = [0.0] + list(r * (0.5 / r.sum()))
    return _round_w(w, c["dtype"])


def _gen(seed):
    return torch.Generator(device=_DEV).manual_seed(int(seed))


def _field(shape, gen):
    """U[0,1) plus the lowest sine mode, in FP64: noise over a smooth field."""
    u = torch.rand(shape, generator=gen, device=_DEV, dtype=torch.float64)
    mode = torch.ones((), device=_DEV, dtype=torch.float64)
    for n in shape:
        x = torch.arange(1, n + 1, device=_DEV, dtype=torch.float64) / (n + 1)
        mode = mode[..., None] * torch.sin(math.pi * x)
    return u.add_(mode)


def _grid_inputs(c, seed):
    return _field(_shape(c), _gen(seed)).to(_TORCH[c["dtype"]]), _weights(c, seed)


def _batch_shapes(c):
    u = np.random.default_rng(c["shape_seed"]).uniform(math.log(c["lo"]), math.log(c["hi"]), size=(c["count"], 2))
    return [(int(a), int(b)) for a, b in np.rint(np.exp(u))]


def _batch_inputs(c, seed):
    gen = _gen(seed)
    grids = [_field(s, gen).to(_TORCH[c["dtype"]]) for s in _batch_shapes(c)]
    alphas = np.random.default_rng(seed).uniform(0.05, 0.24, size=c["count"])
    return grids, [_round_w([0.0] + [a] * 4, c["dtype"]) for a in alphas]


def _varcoef_inputs(c, seed):
    gen = _gen(seed)
    shape = _shape(c)
    u0 = _field(shape, gen)
    k = torch.rand(shape, generator=gen, device=_DEV, dtype=torch.float64).add_(0.5)
    for _ in range(3):  # three 3x3x3 means: a smooth conductivity inside [0.5, 1.5]
        p = torch.nn.functional.pad(k[None, None], (1,) * 6, mode="replicate")
        k = torch.nn.functional.avg_pool3d(p, 3, stride=1)[0, 0]
    y = torch.rand(shape, generator=gen, device=_DEV, dtype=torch.float64)
    return [t.to(_TORCH[c["dtype"]]).contiguous() for t in (u0, k, y)]


_ALPHA = 0.1  # varcoef diffusion number


def prepare(case, seed):
    c = case
    if c["kind"] == "batch":
        grids, coeffs = _batch_inputs(c, seed)
        plan = st.BatchPlan(_offsets(2, "star", 1), [tuple(g.shape) for g in grids], c["dtype"], c["bc"])
        return {"case": c, "plan": plan, "grids": grids, "works": [torch.empty_like(g) for g in grids],
                "coeffs": coeffs, "steps": [c["steps"]] * len(grids)}
    if c["kind"] == "varcoef":
        u0, k, y = _varcoef_inputs(c, seed)
        return {"case": c, "u0": u0.requires_grad_(), "k": k.requires_grad_(), "y": y}
    u, w = _grid_inputs(c, seed)
    plan = st.Plan(_offsets(c["ndim"], c["pattern"], c["radius"]), _shape(c), c["dtype"], c["bc"], graph=c["graph"])
    return {"case": c, "plan": plan, "u": u, "work": torch.empty_like(u), "coeffs": w,
            "flux": torch.zeros(1, device=_DEV, dtype=torch.float64)}


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "batch":
        return s["plan"].run(s["grids"], s["works"], s["coeffs"], s["steps"])
    if c["kind"] == "varcoef":
        u = st.StencilFn.apply(s["u0"], s["k"], _ALPHA, c["steps"], c["every"])
        loss = torch.nn.functional.mse_loss(u, s["y"])
        gu, gk = torch.autograd.grad(loss, (s["u0"], s["k"]))
        return u.detach(), gu, gk
    if c["call"] == "flux":
        s["flux"].zero_()
        s["plan"].run_flux(s["u"], s["coeffs"], c["steps"], s["flux"], work=s["work"])
        return s["u"], s["flux"]
    if c["call"] == "adjoint":
        return s["plan"].adjoint(s["u"], c["steps"], s["work"], coeffs=s["coeffs"])
    return s["plan"].run(s["u"], s["coeffs"], c["steps"], work=s["work"])


# ---------------------------------------------------------------------------
# 64-bit results
# ---------------------------------------------------------------------------
class _Padded:
    """FP64 field with r ghost cells a side; zero, or refilled by wrapping."""

    def __init__(self, u, r, bc):
        self.r, self.bc, self.n = r, bc, tuple(u.shape)
        self.a = torch.zeros([n + 2 * r for n in self.n], device=u.device, dtype=torch.float64)
        self.view((0,) * u.dim()).copy_(u)

    def view(self, off):
        return self.a[tuple(slice(self.r + o, self.r + o + n) for o, n in zip(off, self.n))]

    def wrap(self):
        if self.bc != "periodic":
            return
        for ax, n in enumerate(self.n):
            for g in range(self.r):  # ghost planes one by one: extents may be below r
                self.a.select(ax, self.r - 1 - g).copy_(self.a.select(ax, self.r + (-1 - g) % n))
                self.a.select(ax, self.r + n + g).copy_(self.a.select(ax, self.r + g % n))


def _sweep64(u, offs, w, steps, bc, flux=False):
    r = max(abs(o) for off in offs for o in off)
    p = _Padded(u.double(), r, bc)
    centre = (0,) * u.dim()
    leave = torch.zeros((), device=u.device, dtype=torch.float64)
    for _ in range(steps):
        p.wrap()
        if flux:  # what cell c sends through point o beyond the edge: w * u(c) where c - o is outside
            for o, v in zip(offs[1:], w[1:]):
                for ax, d in enumerate(o):
                    if d:  # a star point has one nonzero entry
                        edge = p.view(centre)
                        leave += v * edge.narrow(ax, 0 if d > 0 else edge.shape[ax] - abs(d), abs(d)).sum()
        new = p.view(offs[0]) * w[0]
        for o, v in zip(offs[1:], w[1:]):
            new.add_(p.view(o), alpha=v)
        p.view(centre).copy_(new)
    return p.view(centre).contiguous(), leave.reshape(1)


def _vc_step(u, k, a):
    out = u.clone()
    for ax in range(3):
        n = u.shape[ax]
        f = (k.narrow(ax, 0, n - 1) + k.narrow(ax, 1, n - 1)) * (u.diff(dim=ax) * (0.5 * a))
        out.narrow(ax, 0, n - 1).add_(f)
        out.narrow(ax, 1, n - 1).sub_(f)
        for i in (0, n - 1):
            out.select(ax, i).sub_(k.select(ax, i) * u.select(ax, i) * a)
    return out


def _vc_grad_k(g, u, lam, a):
    for ax in range(3):
        n = u.shape[ax]
        d = u.diff(dim=ax) * lam.diff(dim=ax) * (-0.5 * a)
        g.narrow(ax, 0, n - 1).add_(d)
        g.narrow(ax, 1, n - 1).add_(d)
        for i in (0, n - 1):
            g.select(ax, i).sub_(u.select(ax, i) * lam.select(ax, i) * a)


def exact(case, seed):
    c = case
    if c["kind"] == "batch":
        grids, coeffs = _batch_inputs(c, seed)
        offs = _offsets(2, "star", 1)
        return [_sweep64(g, offs, w, c["steps"], c["bc"])[0] for g, w in zip(grids, coeffs)]
    if c["kind"] == "varcoef":
        u0, k, y = (t.double() for t in _varcoef_inputs(c, seed))
        states = [u0]
        for _ in range(c["steps"]):
            states.append(_vc_step(states[-1], k, _ALPHA))
        out = states.pop()
        lam, gk = (out - y) * (2.0 / y.numel()), torch.zeros_like(k)
        while states:
            _vc_grad_k(gk, states.pop(), lam, _ALPHA)
            lam = _vc_step(lam, k, _ALPHA)  # the step is symmetric
        return out, lam, gk
    u, w = _grid_inputs(c, seed)
    offs = _offsets(c["ndim"], c["pattern"], c["radius"])
    if c["call"] == "flux":
        if c["pattern"] == "star":
            return _sweep64(u, offs, w, c["steps"], c["bc"], flux=True)
        return _sweep64(u, offs, w, c["steps"], c["bc"])[0], None
    if c["call"] == "adjoint":
        offs = [tuple(-v for v in o) for o in offs]
    return _sweep64(u, offs, w, c["steps"], c["bc"])[0]


def work(case):
    c = case
    if c["kind"] == "batch":
        cells = sum(a * b for a, b in _batch_shapes(c))
        return {"bytes": 2 * cells * _BYTES[c["dtype"]], "flops": cells * c["steps"] * 9}
    cells = math.prod(_shape(c))
    if c["kind"] == "varcoef":
        # in: u0, k, y; out: the final field and two gradients.  A step: six
        # faces of a sum, a difference and a multiply-add; the adjoint step
        # that plus six products for dL/dk
        return {"bytes": 6 * cells * _BYTES[c["dtype"]], "flops": cells * c["steps"] * (24 + 24 + 24)}
    points = len(_offsets(c["ndim"], c["pattern"], c["radius"]))
    return {"bytes": 2 * cells * _BYTES[c["dtype"]], "flops": cells * c["steps"] * (2 * points - 1)}
