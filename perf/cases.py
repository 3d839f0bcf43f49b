"""Timed cases of the operator pair: what a user's programs call, over the sizes they call it at.

A case names one call (its "call" key) and its sizes:

  pair       Plan.forward and Plan.adjoint on a plan the program keeps
  forward    Plan.forward alone
  adjoint    Plan.adjoint alone
  gradient   autograd.loss_and_grad: 0.5 ||H p - y||^2 and its gradient, one reconstruction iteration
  request    a served request of its own medium: the plan is built inside the call, then H and H^T
  served     four requests of uneven grids in flight at once, on an Executor or in a Group
  response   eir_apply, convolution and correlation of every trace with a transducer response

Media ("medium"): "skull", an ellipsoidal shell of 8 cells of heterogeneous solid in uniform
water; "tissue", a heterogeneous fluid; "solid", a heterogeneous solid without any fluid.
Everything is made on the GPU from the seed alone.
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_1709_02733_amd import autograd, el

DX = 1e-4                                    # m
CFL = 0.3                                    # c_max dt / dx, as every recipe of the package
MECHANISMS = [(2.0 * math.pi * 0.5e6, 0.5), (2.0 * math.pi * 2.0e6, 0.5)]


def _case(name, call, n, nsteps, npml=16, nrec=1024, medium="skull", precision="f32", relax=False, **more):
    nx, ny, nz = (n, n, n) if isinstance(n, int) else n
    return dict(name=name, call=call, nx=nx, ny=ny, nz=nz, nsteps=nsteps, npml=npml, nrec=nrec, medium=medium,
                precision=precision, relax=relax, **more)


def listed():
    return [
        # the parity configuration (64^3, 400 samples, 128 receivers), the smallest grid a
        # program steps: launches and latency count
        _case("pair_64", "pair", 64, 400, npml=8, nrec=128),
        # a served request of the smallest served size, with its own medium: plan set-up counts
        _case("request_96", "request", 96, 800, nrec=512),
        # the adjoint image of a kept plan at that size; most cells lie in absorbing layers
        _case("adjoint_96", "adjoint", 96, 800),
        # four small requests in flight on the executor, the serving loop's default mode
        _case("served_96", "served", 96, 400, nrec=512, mode="executor"),
        # one iteration of the reconstruction study (128^3, 1000 samples, 512 receivers)
        _case("gradient_128", "gradient", 128, 1000, nrec=512),
        # double precision, for programs that check or refine a result
        _case("pair_f64_128", "pair", 128, 200, precision="f64"),
        # a solid specimen on a ragged grid of odd sizes: every cell takes the elastic update
        _case("pair_solid_odd", "pair", (157, 131, 109), 250, npml=10, nrec=333, medium="solid"),
        # an acoustic problem: heterogeneous soft tissue on a ragged grid
        _case("forward_tissue_odd", "forward", (203, 187, 150), 300, npml=12, nrec=700, medium="tissue"),
        # a skull whose absorption rises with frequency
        _case("pair_relax_192", "pair", 192, 200, relax=True),
        # the largest served size, a quarter of its samples
        _case("pair_256", "pair", 256, 450),
        # the headline configuration (384^3, 1024 receivers), a twentieth of its samples
        _case("pair_384", "pair", 384, 126),
        # the measured traces of the headline configuration through a 171-tap transducer response
        _case("response_2500", "response", 384, 2500, taps=171),
    ]


_WEIGHT = dict(skull=1.0, tissue=1.0, solid=2.2)
_OPS = dict(pair=2, forward=1, adjoint=1, gradient=2, request=2, served=4)


def _cost(case):
    """Skull cell-updates in single precision that take about the case's time."""
    cells = case["nx"] * case["ny"] * case["nz"]
    return (cells * case["nsteps"] * _OPS[case["call"]] * _WEIGHT[case["medium"]]
            * (2.3 if case["precision"] == "f64" else 1.0))


def draw(rng):
    call = rng.choice(["pair", "pair", "forward", "adjoint", "gradient", "request", "served", "response"])
    if call == "response":
        case = _case("", call, 384, int(math.exp(rng.uniform(math.log(200), math.log(3000)))),
                     nrec=rng.randint(37, 1024), taps=rng.randint(20, 400))
        del case["name"]
        return case
    top = {"served": 128, "request": 256, "gradient": 192}.get(call, 384)
    base = math.exp(rng.uniform(math.log(40), math.log(top)))
    n = [max(32, min(top, int(base * rng.uniform(0.75, 1.25)))) for _ in range(3)]
    if rng.random() < 0.5:
        n = [max(32, min(top, int(base)))] * 3
    medium = rng.choice(["skull", "skull", "skull", "tissue", "solid"])
    precision = "f64" if call in ("pair", "forward", "adjoint") and rng.random() < 0.2 else "f32"
    npml = rng.choice([0, 4, 8, 10, 16, 16])
    npml = min(npml, (min(n) - 2) // 4)
    relax = medium == "skull" and call == "pair" and min(n) >= 2 * npml + 40 and rng.random() < 0.25
    case = _case("", call, tuple(n), 1, npml=npml, nrec=rng.randint(64, 1024), medium=medium, precision=precision,
                 relax=relax)
    if call == "served":
        case["mode"] = rng.choice(["executor", "group"])
    del case["name"]
    # samples: up to 1000, at most half the cost of the largest listed case
    most = 0.5 * 384 ** 3 * 126 * 2 / _cost(case)
    case["nsteps"] = int(max(8, min(1000, most) * math.exp(rng.uniform(math.log(0.15), 0.0))))
    return case


# --------------------------------------------------------------------------- inputs

def _noise(gen, shape, cells):
    """Smooth random field, one value per `cells` cells interpolated linearly, max |.| = 1."""
    coarse = [max(2, s // cells + 2) for s in shape]
    g = torch.randn([1, 1] + coarse, generator=gen, device="cuda", dtype=torch.float32)
    f = F.interpolate(g, size=list(shape), mode="trilinear", align_corners=True)[0, 0]
    return f / f.abs().max()


def _sphere(count):
    """Upper unit hemisphere, golden-angle spiral."""
    k = np.arange(count) + 0.5
    z = 1.0 - k / count
    r = np.sqrt(np.maximum(0.0, 1.0 - z * z))
    th = k * math.pi * (3.0 - math.sqrt(5.0))
    return np.stack([r * np.cos(th), r * np.sin(th), z], axis=1)


def _problem(case, seed, shape=None):
    """Cell maps, initial pressure, traces and receivers of one operation."""
    nz, ny, nx = shape or (case["nz"], case["ny"], case["nx"])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    n = np.array([nx, ny, nz], dtype=np.float64)
    c = (n - 1) / 2
    ax = [torch.arange(m, device="cuda", dtype=torch.float64) - mid for m, mid in zip((nx, ny, nz), c)]
    X, Y, Z = ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]
    semi = np.array([0.39, 0.36, 0.33]) * n * rng.uniform(0.97, 1.0, 3)
    r = torch.sqrt(X * X + Y * Y + Z * Z)
    ell = torch.sqrt((X / semi[0]) ** 2 + (Y / semi[1]) ** 2 + (Z / semi[2]) ** 2)
    r_in = r / torch.clamp(ell, min=1e-9)
    shp = (nz, ny, nx)
    g = [1.0 + 0.05 * _noise(gen, shp, 5).double() for _ in range(3)]
    water, rate = 1500.0 * rng.uniform(0.97, 1.0), rng.uniform(0.0, 2.0)
    if case["medium"] == "tissue":
        cp, cs, rho = 1500.0 * g[0], torch.zeros_like(r), 1000.0 * g[2]
        alpha = 2.0 * cp * 2.0
        shell = torch.zeros_like(r, dtype=torch.bool)
    else:
        shell = (r >= r_in) & (r < r_in + 8.0 + 2.0 * _noise(gen, shp, 24)) & (r > 0)
        if case["medium"] == "solid":
            shell = torch.ones_like(shell)
        cp = torch.where(shell, 2800.0 * g[0], water)
        cs = torch.where(shell, 1500.0 * g[1], 0.0)
        rho = torch.where(shell, 1850.0 * g[2], 1000.0)
        alpha = torch.where(shell, 2.0 * cp * 20.0, 2.0 * cp * rate)
    mu = rho * cs * cs
    lam = rho * cp * cp - 2.0 * mu
    alpha_r = None
    if case["relax"]:
        m = case["npml"] + 2
        inner = torch.zeros_like(shell)
        inner[m:nz - m, m:ny - m, m:nx - m] = True
        inner &= shell
        alpha_r = torch.where(inner, 2.0 * alpha, 0.0).float()
        alpha = torch.where(inner, 0.0, alpha)
    vessels = torch.clamp(_noise(gen, shp, 4) - 0.3, min=0.0)
    p0 = torch.where((ell < 0.9) & ~(shell if case["medium"] == "skull" else torch.zeros_like(shell)),
                     vessels.double(), 0.0).float()
    # measured traces: band-limited noise, a few samples long
    y = torch.randn((case["nsteps"] + 6, case["nrec"]), generator=gen, device="cuda", dtype=torch.float64)
    y = sum(y[q:q + case["nsteps"]] * w for q, w in enumerate((0.05, -0.2, 0.5, 1.0, 0.5, -0.2, 0.05))).contiguous()
    rec = (c + 0.47 * n * _sphere(case["nrec"])) * DX
    return dict(lam=lam.float(), mu=mu.float(), rho=rho.float(), alpha=alpha.float(), alpha_r=alpha_r, p0=p0, y=y,
                rec=rec, dt=CFL * DX / float(cp.max()), shape=shp)


def _plan(case, pr):
    nz, ny, nx = pr["shape"]
    return el.Plan(nx, ny, nz, DX, pr["dt"], case["nsteps"], case["npml"], pr["lam"], pr["mu"], pr["rho"],
                   pr["alpha"], pr["rec"], precision=case["precision"], alpha_r=pr["alpha_r"],
                   mechanisms=MECHANISMS if case["relax"] else None)


def _dtype(case):
    return torch.float64 if case["precision"] == "f64" else torch.float32


def _served_shapes(case):
    """Grids of the four requests: the case's and three a little larger or ragged."""
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    return [(nz, ny, nx), (nz + 16, ny + 16, nx + 16), (nz, ny + 9, nx + 5), (nz + 32, ny, nx + 32)]


def _taps(case, seed):
    """A 2.25 MHz sine under a Gaussian window, a little detuned by the seed."""
    n = case["taps"]
    t = np.arange(n) - (n - 1) / 2
    f = 2.0 * math.pi * 4.0 / n * (1.0 + 0.01 * (seed % 7))
    return np.sin(f * t) * np.exp(-0.5 * (t / (0.25 * n)) ** 2)


def _traces(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((case["nsteps"], case["nrec"]), generator=gen, device="cuda", dtype=torch.float64)


def prepare(case, seed):
    call = case["call"]
    if call == "response":
        return dict(call=call, h=torch.from_numpy(_taps(case, seed)).cuda(), y=_traces(case, seed))
    if call == "served":
        prs = [_problem(case, seed + 1000 * q, s) for q, s in enumerate(_served_shapes(case))]
        plans = [_plan(case, pr) for pr in prs]
        pool = el.Executor(max_slots=4) if case["mode"] == "executor" else el.Group(max_members=4)
        return dict(call=call, case=case, plans=plans, pool=pool, inputs=[(pr["p0"], pr["y"]) for pr in prs])
    pr = _problem(case, seed)
    if call == "request":
        return dict(call=call, case=case, pr=pr)
    return dict(call=call, plan=_plan(case, pr), p0=pr["p0"].to(_dtype(case)), y=pr["y"])


def run(state):
    call = state["call"]
    if call == "response":
        return [el.eir_apply(state["h"], state["y"]), el.eir_apply(state["h"], state["y"], transpose=True)]
    if call == "served":
        return _run_served(state)
    if call == "request":
        plan = _plan(state["case"], state["pr"])
        out = [plan.forward(state["pr"]["p0"]), plan.adjoint(state["pr"]["y"])]
        plan.close()
        return out
    plan = state["plan"]
    if call == "forward":
        return [plan.forward(state["p0"])]
    if call == "adjoint":
        return [plan.adjoint(state["y"])]
    if call == "gradient":
        return list(autograd.loss_and_grad(plan, state["p0"], state["y"]))
    return [plan.forward(state["p0"]), plan.adjoint(state["y"])]


def _run_served(state):
    case, pool = state["case"], state["pool"]
    outs, slots = [], []
    for q, (plan, (p0, y)) in enumerate(zip(state["plans"], state["inputs"])):
        op = el.OP_FORWARD if q % 2 == 0 else el.OP_ADJOINT
        if op == el.OP_FORWARD:
            inp, out = p0, torch.empty((plan.nsteps, plan.nrec), dtype=torch.float64, device=plan.device)
        else:
            inp, out = y, torch.empty(plan.shape, dtype=plan.dtype, device=plan.device)
        outs.append(out)
        slots.append(pool.add(plan, op, inp, out) if case["mode"] == "group" else pool.start(plan, op, inp, out))
    if case["mode"] == "group":
        pool.run(case["nsteps"])
        pool.sync(0)
        for s in slots:
            pool.poll(s)
    else:
        for s in slots:
            pool.wait(s)
    return outs


# --------------------------------------------------------------------------- necessary work

def _op_work(case, shape):
    """One operation: a time step reads the state and the medium once and writes the state once.
    Where the medium is fluid the state is the velocity and one stress (8 elements read and
    written) plus one memory variable per absorbing-layer axis, elsewhere the full state (18)
    plus six; the media are four maps, none where they are uniform (the skull's water)."""
    nz, ny, nx = shape
    es = 8 if case["precision"] == "f64" else 4
    cells = nx * ny * nz
    if case["medium"] == "skull":
        # shell of 8 cells, and two on either side where its stencils reach
        a = np.array([0.39 * nx, 0.36 * ny, 0.33 * nz]) * 0.985
        vol = lambda d: 4.0 / 3.0 * math.pi * float(np.prod(np.maximum(a + d, 0.0)))
        solid = min(1.0, (vol(10.0) - vol(-2.0)) / cells)
    else:
        solid = 1.0 if case["medium"] == "solid" else 0.0
    media_fluid = 3 if case["medium"] == "tissue" else 0
    layer = sum(2.0 * case["npml"] / m for m in (nx, ny, nz)) * cells
    per = solid * (18 + 4) + (1 - solid) * (8 + media_fluid)
    elements = cells * per + layer * (solid * 12 + (1 - solid) * 4)
    if case["relax"]:
        elements += cells * solid * 0.6 * 3 * (1 + 2 * len(MECHANISMS))
    flops = cells * (solid * 160 + (1 - solid) * 60) + layer * (solid * 24 + (1 - solid) * 8)
    steps = case["nsteps"] - 1
    return dict(bytes=steps * elements * es + cells * 5 * es + case["nsteps"] * case["nrec"] * 8.0,
                flops=steps * flops + case["nsteps"] * case["nrec"] * 16.0)


def work(case):
    if case["call"] == "response":
        n = case["nsteps"] * case["nrec"]
        return dict(bytes=2 * 16.0 * n, flops=2 * 2.0 * n * case["taps"])
    if case["call"] == "served":
        ws = [_op_work(case, s) for s in _served_shapes(case)]
    else:
        ws = [_op_work(case, (case["nz"], case["ny"], case["nx"]))] * _OPS[case["call"]]
    total = {k: float(sum(w[k] for w in ws)) for k in ("bytes", "flops")}
    if case["call"] == "request":
        total["bytes"] += case["nx"] * case["ny"] * case["nz"] * 4 * 8.0     # the maps, read and laid out
    return total


# --------------------------------------------------------------------------- 64-bit values

def _diff(f, axis, plus):
    """4th-order staggered difference with zero extension: plus, the value at i + 1/2."""
    dim = 2 - axis
    lo, hi = (1, 2) if plus else (2, 1)
    pad = [0, 0] * axis + [lo, hi]
    g = F.pad(f, pad)
    n = f.shape[dim]
    t = [g.narrow(dim, q, n) for q in range(4)]
    return (9.0 / 8.0 * (t[2] - t[1]) - 1.0 / 24.0 * (t[3] - t[0])) * (1.0 / DX)


def _up(f, *axes):
    """f at the upper neighbour along the axes, the last cell replicated."""
    for a in axes:
        dim = 2 - a
        f = torch.cat([f.narrow(dim, 1, f.shape[dim] - 1), f.narrow(dim, f.shape[dim] - 1, 1)], dim)
    return f


def _layer(case, pr, n, axis, half, cmax):
    """C-PML coefficients a, b along an axis, broadcastable."""
    P, dt = case["npml"], pr["dt"]
    d0 = -3.0 * cmax * math.log(1e-3) / (2.0 * P * DX)
    x = np.arange(n) + 0.5 * half
    xi = np.clip(np.maximum(P - x, x - (n - 1 - P)) / P, 0.0, 1.0)
    d, beta = d0 * xi ** 2, math.pi * 1500.0 / (8.0 * DX) * (1.0 - xi)
    b = np.exp(-(d + beta) * dt)
    with np.errstate(invalid="ignore"):
        a = np.where(xi > 0, d / np.where(d + beta > 0, d + beta, 1.0) * (b - 1.0), 0.0)
    shape = [1, 1, 1]
    shape[2 - axis] = n
    return tuple(torch.from_numpy(v).cuda().reshape(shape) for v in (a, b))


def _forward64(case, pr, p0):
    """Traces of the scheme in 64 bits; differentiable in p0."""
    lam, mu, rho, alpha = (pr[k].double() for k in ("lam", "mu", "rho", "alpha"))
    dt, n = pr["dt"], [lam.shape[2], lam.shape[1], lam.shape[0]]
    cmax = float(torch.sqrt(((lam + 2.0 * mu) / rho).max()))
    decay, push = [], []
    for c in range(3):
        decay.append(1.0 - dt * 0.5 * (alpha + _up(alpha, c)))
        push.append(dt / (0.5 * (rho + _up(rho, c))))
    edge = {}
    for a, b in ((1, 2), (0, 2), (0, 1)):
        q = [mu, _up(mu, a), _up(mu, b), _up(mu, a, b)]
        edge[(a, b)] = 4.0 / sum(1.0 / v for v in q)
    sheared = bool((mu > 0).any())
    pml = None
    if case["npml"] > 0:
        pml = [[_layer(case, pr, n[a], a, half, cmax) for half in (0, 1)] for a in range(3)]
    relax = []
    if case["relax"]:
        ar = pr["alpha_r"].double()
        for c in range(3):
            beta = 0.5 * (ar + _up(ar, c))
            relax.append([(w * beta, math.exp(-om * dt)) for om, w in MECHANISMS])
    # receivers: trilinear weights of the eight corners
    x = pr["rec"] / DX
    base = np.minimum(np.floor(x).astype(np.int64), np.array(n) - 2)
    f = x - base
    idx, wts = [], []
    for q in range(8):
        o = np.array([q & 1, q >> 1 & 1, q >> 2 & 1])
        cell = base + o
        idx.append(cell[:, 0] + n[0] * (cell[:, 1] + n[1] * cell[:, 2]))
        wts.append(np.prod(np.where(o, f, 1.0 - f), axis=1))
    idx, wts = torch.from_numpy(np.stack(idx)).cuda(), torch.from_numpy(np.stack(wts)).cuda()

    key = lambda c, a: (min(c, a), max(c, a))
    s = {(c, c): p0 * (-1.0 / 3.0) for c in range(3)}
    zero = torch.zeros_like(lam)
    for e in edge:
        s[e] = zero
    u = [zero, zero, zero]
    phi, psi = {}, {}
    zeta = [[zero] * len(MECHANISMS) for _ in range(3)]
    used = [(c, a) for c in range(3) for a in range(3) if sheared or c == a]
    rows = []
    for m in range(case["nsteps"]):
        if m > 0:
            acc = [zero, zero, zero]
            for c, a in used:
                d = _diff(s[key(c, a)], a, c == a)
                if pml:
                    ca, cb = pml[a][1 if c == a else 0]
                    phi[c, a] = ca * d + (cb * phi[c, a] if (c, a) in phi else 0.0)
                    d = d + phi[c, a]
                acc[c] = acc[c] + d
            for c in range(3):
                u[c] = decay[c] * u[c] + push[c] * acc[c]
                if relax:
                    num, den = u[c], 1.0
                    for l, (bl, cl) in enumerate(relax[c]):
                        num, den = num + dt * bl * zeta[c][l], den + dt * bl
                    u[c] = num * (1.0 / den)
                    for l, (bl, cl) in enumerate(relax[c]):
                        zeta[c][l] = cl * zeta[c][l] + (1.0 - cl) * u[c]
            e = {}
            for c, a in used:
                d = _diff(u[c], a, c != a)
                if pml:
                    ca, cb = pml[a][1 if c != a else 0]
                    psi[c, a] = ca * d + (cb * psi[c, a] if (c, a) in psi else 0.0)
                    d = d + psi[c, a]
                e[c, a] = d
            tr = dt * (lam * (e[0, 0] + e[1, 1] + e[2, 2]))
            for c in range(3):
                s[c, c] = s[c, c] + tr + ((2.0 * dt) * mu * e[c, c] if sheared else 0.0)
            if sheared:
                for (a, b), m_ab in edge.items():
                    s[a, b] = s[a, b] + (dt * m_ab) * (e[a, b] + e[b, a])
        total = (s[0, 0] + s[1, 1] + s[2, 2]).reshape(-1)
        rows.append(-(total[idx] * wts).sum(0))
    return torch.stack(rows)


def _seconds(case, shape, transpose):
    """Rough time of the 64-bit values on the GPU."""
    cells = shape[0] * shape[1] * shape[2]
    per = max(cells * 1.3e-9, 2.0e-3) * (0.5 if case["medium"] == "tissue" else 1.0)
    return case["nsteps"] * per * (4.0 if transpose else 1.0)


def _traces64(case, pr):
    with torch.no_grad():
        return _forward64(case, pr, pr["p0"].double())


def _image64(case, pr, y):
    p0 = torch.zeros_like(pr["p0"], dtype=torch.float64).requires_grad_(True)
    return torch.autograd.grad(_forward64(case, pr, p0), p0, y)[0]


def exact(case, seed):
    call, room = case["call"], 12.0
    if call == "response":
        h, y = _taps(case, seed), _traces(case, seed)
        out = [torch.zeros_like(y), torch.zeros_like(y)]
        for k, w in enumerate(h[:case["nsteps"]]):
            rest = case["nsteps"] - k
            out[0][k:] += float(w) * y[:rest]
            out[1][:rest] += float(w) * y[k:]
        return out
    shapes = _served_shapes(case) if call == "served" else [(case["nz"], case["ny"], case["nx"])]
    wanted = {"forward": [0], "adjoint": [1], "served": [0, 1, 0, 1]}.get(call, [0, 1])
    if call == "gradient":
        if _seconds(case, shapes[0], True) > room:
            return None
        pr = _problem(case, seed)
        r = _traces64(case, pr) - pr["y"]
        return [0.5 * torch.sum(r * r), _image64(case, pr, r)]
    out, prs = [], {}
    for q, op in enumerate(wanted):
        k = q if call == "served" else 0
        cost = _seconds(case, shapes[k], op == 1)
        if cost > room:
            out.append(None)
            continue
        room -= cost
        if k not in prs:
            prs[k] = _problem(case, seed + 1000 * k, shapes[k])
        out.append(_image64(case, prs[k], prs[k]["y"]) if op else _traces64(case, prs[k]))
    return out if any(v is not None for v in out) else None
