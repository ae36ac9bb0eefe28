"""The work that programs have this library do, as measurable cases.

A case names an operation ("op"), its direction, data type and sizes.  The listed cases cover the
single-step calls from the smallest (launch latency) to the benchmark's 512^3 arrays, and the reverse
sweeps of time loops, which is what a program that differentiates a solver spends its time in.
`draw` gives further cases of the same ranges: every stencil family, both directions, both data
types, sizes spread over their logarithm, odd extents among them.

Field values follow the library's own workloads: coefficient fields layered along the slowest axis,
adjoint seeds and states uniform in (-1, 1), for Burgers a sine plus noise.
"""
import math

import torch

import paper_1907_02818_amd as sadj

BURGERS_C, BURGERS_D = 0.1, 0.05
DTYPES = {"f64": torch.float64, "f32": torch.float32}
SINGLE_STEP = ("wave1d", "wave2d", "wave3d", "star3d", "box2d", "box3d", "burgers1d")


def listed():
    return [
        # a call so small that only launch and host time count: one step of the 1-D toy solver
        dict(name="wave1d_adjoint_4096", op="wave1d", way="adjoint", dtype="f64", n=4096),
        # one step of the 1-D nonlinear solver at the benchmark's size
        dict(name="burgers1d_adjoint_16M", op="burgers1d", way="adjoint", dtype="f64", n=1 << 24),
        # a 2-D section with odd extents, adjoints of both time levels wanted
        dict(name="wave2d_adjoint_both_odd", op="wave2d", way="adjoint", dtype="f64", ny=2050, nx=4099, both=True),
        # the headline workload: one radius-4 step of the seismic solver, 512^3
        dict(name="wave3d_r4_adjoint_512", op="wave3d", way="adjoint", dtype="f64", radius=4, nz=512, ny=512, nx=512),
        # forward step of the paper's 7-point solver, rows that are no multiple of a cache line
        dict(name="wave3d_r1_primal_500", op="wave3d", way="primal", dtype="f32", radius=1, nz=500, ny=500, nx=500),
        # a small 3-D block, as in a coarse level or an inversion's patch
        dict(name="wave3d_r4_adjoint_small", op="wave3d", way="adjoint", dtype="f64", radius=4, nz=80, ny=96, nx=112, both=True),
        # an asymmetric (upwind-biased) star and its adjoint's mirrored gather, ragged grid
        dict(name="star3d_r2_adjoint_ragged", op="star3d", way="adjoint", dtype="f32", radius=2, nz=300, ny=350, nx=404),
        # a stretch of a radius-4 time loop swept backwards with three buffers
        dict(name="wave3d_r4_sweep_256", op="sweep", dtype="f64", radius=4, nz=256, ny=256, nx=256, nsteps=20),
        # the benchmark's long radius-1 sweep with a work array
        dict(name="wave3d_r1_sweep_fused_512", op="sweep_fused", dtype="f64", radius=1, nz=512, ny=512, nx=512, nsteps=25),
        # the same on a small ragged grid in single precision
        dict(name="wave3d_r1_sweep_fused_small", op="sweep_fused", dtype="f32", radius=1, nz=96, ny=130, nx=164, nsteps=48),
        # gradient of a nonlinear time loop that keeps all its states
        dict(name="burgers_gradient_history", op="burgers_history", dtype="f64", n=1 << 20, nsteps=64),
        # gradient of a longer loop that keeps every 16th state and recomputes the others
        dict(name="burgers_gradient_ckpt", op="burgers_ckpt", dtype="f64", n=3000001, nsteps=128, every=16),
    ]


def _log_int(rng, lo, hi):
    """An integer from lo to hi, uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _extent(rng, lo, hi):
    """As _log_int; a third as drawn, a third multiples of 4, a third multiples of 32."""
    step = rng.choice((1, 4, 32))
    return max(lo, _log_int(rng, lo, hi) // step * step)


def _grid3(rng, lo, hi, cells):
    while True:
        g = dict(nz=_extent(rng, lo, hi), ny=_extent(rng, lo, hi), nx=_extent(rng, lo, hi))
        if g["nz"] * g["ny"] * g["nx"] <= cells:
            return g


def draw(rng):
    op = rng.choice(("wave1d", "burgers1d", "wave2d", "box2d", "wave3d", "wave3d", "star3d", "box3d", "sweep", "sweep", "sweep_fused",
                     "sweep_fused", "burgers_history", "burgers_history", "burgers_ckpt", "burgers_ckpt"))
    case = dict(op=op, dtype=rng.choice(("f64", "f64", "f32")))
    if op in SINGLE_STEP:
        case["way"] = rng.choice(("adjoint", "adjoint", "primal"))
    if op in ("wave1d", "wave2d", "wave3d") and case["way"] == "adjoint":
        case["both"] = rng.random() < 0.3
    if op in ("wave1d", "burgers1d"):
        case["n"] = _extent(rng, 1000, 1 << 25)
    elif op in ("wave2d", "box2d"):
        case.update(ny=_extent(rng, 64, 8192), nx=_extent(rng, 64, 8192))
    elif op in ("wave3d", "star3d", "box3d"):
        if op != "box3d":
            case["radius"] = rng.choice((1, 1, 2, 3, 4, 4))
        case.update(_grid3(rng, 32, 640, 1 << 27))
    elif op in ("sweep", "sweep_fused"):
        case["radius"] = rng.choice((1, 1, 2, 3, 4, 4)) if op == "sweep" else rng.choice((1, 1, 1, 2, 4))
        case.update(_grid3(rng, 32, 400, 1 << 24))
        case["nsteps"] = _log_int(rng, 3, 60)
    elif op == "burgers_history":
        case["n"] = _extent(rng, 1000, 1 << 22)
        case["nsteps"] = _log_int(rng, 4, max(4, min(300, (1 << 27) // case["n"])))
    else:
        case["n"] = _extent(rng, 1000, 1 << 23)
        case["nsteps"] = _log_int(rng, 10, max(10, min(400, (1 << 28) // case["n"])))
        case["every"] = _log_int(rng, 2, 40)
        size = 8 if case["dtype"] == "f64" else 4
        case["static"] = rng.random() < 0.5 and (case["every"] - 1) * case["n"] * size <= 64 << 20
    return case


def _shape(case):
    if "nz" in case:
        return (case["nz"], case["ny"], case["nx"])
    return (case["ny"], case["nx"]) if "ny" in case else (case["n"],)


def _layered(shape, lo, hi, dtype, gen):
    """A coefficient field in layers along the slowest axis (uniform noise in 1-D)."""
    if len(shape) == 1:
        return lo + (hi - lo) * torch.rand(shape, generator=gen, dtype=dtype, device="cuda")
    layers = max(2, shape[0] // 32)
    value = lo + (hi - lo) * torch.rand(layers, generator=gen, dtype=dtype, device="cuda")
    at = torch.arange(shape[0], device="cuda") * layers // shape[0]
    return value[at].reshape((-1,) + (1,) * (len(shape) - 1)).expand(shape).contiguous()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype, op = DTYPES[case["dtype"]], case["op"]
    shape = _shape(case)

    def field():
        return torch.rand(shape, generator=gen, dtype=dtype, device="cuda").mul_(2).sub_(1)

    def burgers_state():
        x = torch.arange(shape[0], device="cuda", dtype=torch.float64) * (2 * math.pi * 8 / shape[0])
        return (0.75 * torch.sin(x)).to(dtype).add_(field(), alpha=0.25)

    s = dict(case)
    if op == "burgers1d":
        s["u"] = burgers_state()
        s["r_bar" if case["way"] == "adjoint" else "r"] = field()
        if case["way"] == "adjoint":
            s["u_bar"] = field()
        return s
    if op == "burgers_history":
        s["states"] = torch.zeros((case["nsteps"] + 1, shape[0]), dtype=dtype, device="cuda")
        s["states"][0] = burgers_state()
        s["states"][:, 0], s["states"][:, -1] = s["states"][0, 0], s["states"][0, -1]
        s["seed"], s["lam"] = field(), [torch.zeros(shape, dtype=dtype, device="cuda") for _ in range(2)]
        return s
    if op == "burgers_ckpt":
        rows = case["nsteps"] // case["every"] + 1
        s["ckpt"] = torch.zeros((rows, shape[0]), dtype=dtype, device="cuda")
        s["ckpt"][0] = burgers_state()
        s["u_final"] = torch.zeros(shape, dtype=dtype, device="cuda")
        s["work"] = torch.zeros((max(2, case["every"] - 1), shape[0]), dtype=dtype, device="cuda")
        s["seed"], s["lam"] = field(), [torch.zeros(shape, dtype=dtype, device="cuda") for _ in range(2)]
        return s
    # the coefficient's upper end keeps a leapfrog time loop stable for every radius
    hi = {1: 0.25, 2: 0.2, 3: 0.1 if case.get("radius") == 4 else 0.15}[len(shape)]
    s["c"] = _layered(shape, 0.01, hi, dtype, gen)
    if op in ("sweep", "sweep_fused"):
        s["lam"] = [field(), field(), torch.zeros(shape, dtype=dtype, device="cuda")]
        if op == "sweep_fused":
            s["work"] = torch.zeros(shape, dtype=dtype, device="cuda")
        return s
    if op in ("box2d", "box3d"):
        w = torch.rand((3,) * len(shape), generator=gen, dtype=torch.float64, device="cuda")
        s["weights"] = (w - 0.5).cpu().tolist()
    if op == "star3d":
        w = torch.rand(1 + 6 * case["radius"], generator=gen, dtype=torch.float64, device="cuda")
        s["weights"] = (w - 0.5).cpu().tolist()
    if case["way"] == "primal":
        s["u"], s["r"] = field(), field()
        if op.startswith("wave"):
            s["u_prev"] = field()
    else:
        s["r_bar"], s["u_bar"] = field(), field()
        if case.get("both"):
            s["u_prev_bar"] = field()
    return s


def run(s):
    op = s["op"]
    if op in SINGLE_STEP:
        return _run_step(s, op)
    if op in ("sweep", "sweep_fused"):
        # one stretch of a long reverse sweep: the two live adjoint states carry over from the
        # stretch before, the third buffer starts from zero
        lam, n = s["lam"], s["nsteps"]
        lam[2].zero_()
        if op == "sweep":
            sadj.sadj_adjoint_wave3d_steps(s["radius"], n, s["c"], *lam)
        else:
            sadj.sadj_adjoint_wave3d_steps_fused(s["radius"], n, s["c"], *lam, s["work"])
        s["lam"] = lam = [lam[(n + k) % 3] for k in range(3)]
        return lam[0], lam[1]
    # gradient of a nonlinear time loop: forward, seed the adjoint of the last state, backward
    lam, n = s["lam"], s["nsteps"]
    if op == "burgers_history":
        sadj.sadj_primal_burgers1d_steps(BURGERS_C, BURGERS_D, n, s["states"])
        lam[0].copy_(s["seed"])
        lam[1].zero_()
        sadj.sadj_adjoint_burgers1d_steps(BURGERS_C, BURGERS_D, n, n, s["states"], *lam)
        return s["states"], lam[n % 2]
    sadj.sadj_primal_burgers1d_ckpt(BURGERS_C, BURGERS_D, n, s["every"], s["ckpt"], s["work"], s["u_final"])
    lam[0].copy_(s["seed"])
    lam[1].zero_()
    if s.get("static"):
        sadj.sadj_adjoint_burgers1d_ckpt_static(BURGERS_C, BURGERS_D, n, s["every"], s["ckpt"], *lam)
    else:
        sadj.sadj_adjoint_burgers1d_ckpt(BURGERS_C, BURGERS_D, n, s["every"], s["ckpt"], s["work"], *lam)
    return s["ckpt"], s["u_final"], lam[n % 2]


def _run_step(s, op):
    primal = s["way"] == "primal"
    if op == "burgers1d":
        if primal:
            sadj.sadj_primal_burgers1d(BURGERS_C, BURGERS_D, s["u"], s["r"])
        else:
            sadj.sadj_adjoint_burgers1d(BURGERS_C, BURGERS_D, s["u"], s["r_bar"], s["u_bar"])
    elif op.startswith("wave"):
        first = (s["radius"],) if op == "wave3d" else ()
        if primal:
            getattr(sadj, "sadj_primal_" + op)(*first, s["u"], s["u_prev"], s["c"], s["r"])
        else:
            getattr(sadj, "sadj_adjoint_" + op)(*first, s["c"], s["r_bar"], s["u_bar"], s.get("u_prev_bar"))
    else:
        first = (s["radius"], s["weights"]) if op == "star3d" else (s["weights"],)
        name = "star3d" if op == "star3d" else "box"
        if primal:
            getattr(sadj, "sadj_primal_" + name)(*first, s["u"], s["c"], s["r"])
        else:
            getattr(sadj, "sadj_adjoint_" + name)(*first, s["c"], s["r_bar"], s["u_bar"])
    if primal:
        return s["r"]
    return (s["u_bar"], s["u_prev_bar"]) if s.get("both") else s["u_bar"]


def work(case):
    """Inputs read once, outputs written once (an accumulated array is both); operations of the
    stencil formulas, recomputation of states that were not kept included."""
    cells = math.prod(_shape(case))
    size = 8 if case["dtype"] == "f64" else 4
    op = case["op"]
    if op == "burgers_history":
        # forward: one state read, nsteps written; backward: nsteps states and lam read, lam written
        words, flops = 2 * case["nsteps"] + 3, case["nsteps"] * (11 + 21)
    elif op == "burgers_ckpt":
        # forward: one state read, the checkpoints and the last state written; backward: the
        # checkpoints and lam read, lam written
        rows = case["nsteps"] // case["every"]
        words, flops = 2 * rows + 5, case["nsteps"] * (11 + 11 + 21)
    elif op in ("sweep", "sweep_fused"):
        # c and the three buffers read, two of them hold the result
        words, flops = 6, case["nsteps"] * (12 * case["radius"] + 6)
    elif op == "burgers1d":
        words, flops = (2, 11) if case["way"] == "primal" else (4, 21)
    else:
        points = {"box2d": 9, "box3d": 27}.get(op) or 1 + 2 * len(_shape(case)) * case.get("radius", 1)
        flops = 2 * points + 4
        words = 3 if case["way"] == "primal" else 4
        if op.startswith("wave"):
            words = 4 if case["way"] == "primal" else 6 if case.get("both") else 4
    return {"bytes": words * cells * size, "flops": flops * cells}


def tolerance(case):
    # about four times the error seen against 64-bit arithmetic in another order: 2e-16 and 8e-8 for
    # one step, 5e-15 and 2.5e-6 for a long time loop.  A nonlinear loop in single precision may round
    # a state to the other side of zero, where the upwind direction changes: single cells are further off.
    loop = case["op"] not in SINGLE_STEP
    if case["dtype"] == "f64":
        return {"rel": 2e-14} if loop else {"rel": 1e-15}
    if case["op"].startswith("burgers") and loop:
        return {"rel": 1e-5, "max": 0.1}
    return {"rel": 1e-5} if loop else {"rel": 4e-7}


# ------------------------------------------------------------------ the same in 64 bits, plain torch

_STAR = {1: (-2.0, 1.0), 2: (-5 / 2, 4 / 3, -1 / 12), 3: (-49 / 18, 3 / 2, -3 / 20, 1 / 90),
         4: (-205 / 72, 8 / 5, -1 / 5, 8 / 315, -1 / 560)}


def _wave_taps(ndim, radius):
    taps = [((0,) * ndim, ndim * _STAR[radius][0])]
    for d in range(ndim):
        for k in range(1, radius + 1):
            for sign in (-1, 1):
                taps.append((tuple(sign * k if a == d else 0 for a in range(ndim)), _STAR[radius][k]))
    return taps


def _star_taps(radius, w):
    """centre, then per axis x, y, z the offsets -R..-1, +1..+R; offsets in array order (z, y, x)."""
    taps, i = [((0, 0, 0), w[0])], 1
    for axis in (2, 1, 0):
        for o in list(range(-radius, 0)) + list(range(1, radius + 1)):
            taps.append((tuple(o if a == axis else 0 for a in range(3)), w[i]))
            i += 1
    return taps


def _box_taps(w, at=()):
    if not isinstance(w, list):
        return [(at, w)]
    return [t for i, x in enumerate(w) for t in _box_taps(x, at + (i - 1,))]


def _inside(shape, radius):
    return tuple(slice(radius, n - radius) for n in shape)


def _gather(u, taps, radius):
    """sum_o w_o u[i+o] for i in I."""
    out = None
    for offset, w in taps:
        v = u[tuple(slice(radius + o, n - radius + o) for o, n in zip(offset, u.shape))]
        out = v * w if out is None else out.add_(v, alpha=w)
    return out


def _scatter(out, q, taps, radius):
    """out[i+o] += w_o q[i] for i in I; q holds the cells of I only."""
    for offset, w in taps:
        out[tuple(slice(radius + o, n - radius + o) for o, n in zip(offset, out.shape))].add_(q, alpha=w)


def _burgers_primal(u):
    um, u0, up = u[:-2], u[1:-1], u[2:]
    r = u.clone()
    r[1:-1] = u0 - BURGERS_C * (u0.clamp(min=0) * (u0 - um) + u0.clamp(max=0) * (up - u0)) + BURGERS_D * (um - 2 * u0 + up)
    return r


def _burgers_adjoint(u, r_bar, u_bar):
    um, u0, up, r = u[:-2], u[1:-1], u[2:], r_bar[1:-1]
    pos, neg = u0.clamp(min=0), u0.clamp(max=0)
    u_bar[:-2] += (BURGERS_C * pos + BURGERS_D) * r
    u_bar[2:] += (-BURGERS_C * neg + BURGERS_D) * r
    slope = (u0 >= 0) * (u0 - um) + pos + (u0 <= 0) * (up - u0) - neg
    u_bar[1:-1] += (1 - 2 * BURGERS_D - BURGERS_C * slope) * r


def exact(case, seed):
    s = {k: ([x.double() for x in v] if k == "lam" else v.double() if isinstance(v, torch.Tensor) else v)
         for k, v in prepare(case, seed).items()}
    op, shape = case["op"], _shape(case)
    radius = case.get("radius", 1)
    inside = _inside(shape, radius)
    if op == "burgers1d":
        if case["way"] == "primal":
            s["r"][1:-1] = _burgers_primal(s["u"])[1:-1]
            return s["r"]
        _burgers_adjoint(s["u"], s["r_bar"], s["u_bar"])
        return s["u_bar"]
    if op in ("burgers_history", "burgers_ckpt"):
        history = op == "burgers_history"
        nsteps, rows = case["nsteps"], s["states"] if history else s["ckpt"]
        every = 1 if history else case["every"]
        u = rows[0].clone()
        for t in range(nsteps):
            u = _burgers_primal(u)
            if (t + 1) % every == 0:
                rows[(t + 1) // every] = u
        final, lam = u, s["seed"]
        for seg in range((nsteps - 1) // every, -1, -1):
            states = [rows[seg]]
            for t in range(seg * every + 1, min(nsteps, (seg + 1) * every)):
                states.append(_burgers_primal(states[-1]))
            for u in reversed(states):
                before = torch.zeros_like(lam)
                _burgers_adjoint(u, lam, before)
                lam = before
        return (rows, lam) if history else (rows, final, lam)
    if op in ("sweep", "sweep_fused"):
        taps = _wave_taps(3, radius)
        a, b, p = s["lam"]
        ci = s["c"][inside]
        for _ in range(case["nsteps"]):
            ai = a[inside]
            b[inside] += 2 * ai
            _scatter(b, ci * ai, taps, radius)
            p[inside] -= ai
            a, b, p = b, p, torch.zeros_like(a)
        return a, b
    if op.startswith("wave"):
        taps = _wave_taps(len(shape), radius)
    elif op == "star3d":
        taps = _star_taps(radius, s["weights"])
    else:
        taps = _box_taps(s["weights"])
    if case["way"] == "primal":
        value = s["c"][inside] * _gather(s["u"], taps, radius)
        if op.startswith("wave"):
            value += 2 * s["u"][inside] - s["u_prev"][inside]
        s["r"][inside] = value
        return s["r"]
    r = s["r_bar"][inside]
    _scatter(s["u_bar"], s["c"][inside] * r, taps, radius)
    if op.startswith("wave"):
        s["u_bar"][inside] += 2 * r
        if case.get("both"):
            s["u_prev_bar"][inside] -= r
            return s["u_bar"], s["u_prev_bar"]
    return s["u_bar"]
