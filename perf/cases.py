"""Performance cases of the thin-film library: the work its users have it do.

Every case goes through the package's public entry points (`Sim`, `TFLBMRun`)
on one GPU.  `listed()` names the fixed cases, `draw()` gives others of the
same ranges; `prepare()` makes what a user's program holds before the call,
`run()` is one pass, `exact()` the same outputs from plain torch in FP64.

A case is a dict of plain values:
  kind     "run":     init, `steps` time steps, read h and u
           "track":   init, then `samples` times `steps` time steps and the height
           "monitor": init, then `samples` times `steps` time steps, the mass and
                      the term-balance norms; at the end read h and u
           "grad":    one differentiable run (`steps` steps, checkpoint interval
                      `K`) and the backward pass of a misfit to a target height
  film     the initial film and its parameters: "dewet" (flat thin film on a
           patterned substrate), "drop" (spherical cap on a precursor film),
           "hang" (hanging film, no wetting term)
  nx, ny, prec, tau; g, ax (gravity, body acceleration along x); theta (a
  contact-angle field rather than a uniform angle); gamma (a surface tension
  field); radius, angle0, hstar, delta ("drop" only: the initial cap).
"""
import math

import torch

from paper_1810_07642_amd import Sim, TFLBMRun

F64 = torch.float64
GAMMA = 0.01
LARGEST = 4096 * 4096 * 120   # site-steps of the largest forward case
LARGEST_GRAD = 2048 * 2048 * 32

_DEFAULTS = dict(kind="run", film="dewet", nx=512, ny=512, prec="fp32", tau=1.0, g=0.0, ax=0.0, theta=True,
                 gamma=False, radius=20.0, angle0=math.pi / 6, hstar=0.5, delta=4.0, steps=100, samples=1, K=64)


def _case(**kw):
    return {**_DEFAULTS, **kw}


def listed():
    return [
        # the smallest lattice in use: a sessile drop relaxing on its precursor film
        _case(name="relax_64_fp64", film="drop", nx=64, ny=64, prec="fp64", radius=20.0, angle0=math.pi / 4,
              hstar=0.05, delta=1.0, steps=1000),
        # one iteration of the contact-angle design loop at the size of its twin
        # experiment: every step's capture kept
        _case(name="grad_128_fp32_keep", kind="grad", nx=128, ny=128, prec="fp32", steps=300, K=0),
        # spreading drop at another viscosity than tau = 1, sampled in time
        _case(name="spread_512_fp64_tau09", kind="track", film="drop", nx=512, ny=512, prec="fp64", tau=0.9,
              radius=100.0, hstar=0.5, delta=4.0, steps=40, samples=6),
        # hanging film (Rayleigh-Taylor), gravity in the equilibrium, no contact-angle field
        _case(name="hang_512_fp32", film="hang", nx=512, ny=512, prec="fp32", g=-1.0e-4, theta=False, steps=500),
        # a drop sliding down an incline
        _case(name="slide_1024x512_fp32", film="drop", nx=1024, ny=512, prec="fp32", ax=1.0e-5, radius=40.0,
              hstar=0.5, delta=1.0, steps=400),
        # an odd-sized lattice with a surface tension field and another viscosity
        _case(name="gamma_901x641_fp32_tau12", nx=901, ny=641, prec="fp32", tau=1.2, g=1.0e-3, gamma=True, steps=150),
        # an odd-sized FP64 run watched by its mass and term balance
        _case(name="monitor_1003x750_fp64", kind="monitor", nx=1003, ny=750, prec="fp64", steps=20, samples=4),
        # inverse design at its full lattice: checkpoints and recompute
        _case(name="grad_512_fp32_ckpt", kind="grad", nx=512, ny=512, prec="fp32", steps=256, K=64),
        # the reverse pass on a lattice that fills the GPU
        _case(name="grad_2048_fp32_ckpt", kind="grad", nx=2048, ny=2048, prec="fp32", steps=32, K=16),
        # patterned dewetting in the half-precision storage form
        _case(name="dewet_2048_fp16s", nx=2048, ny=2048, prec="fp16s", steps=100),
        # patterned dewetting, the headline lattice, in FP64 and FP32
        _case(name="dewet_4096_fp64", nx=4096, ny=4096, prec="fp64", steps=60),
        _case(name="dewet_4096_fp32", nx=4096, ny=4096, prec="fp32", steps=120),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run", "run", "run", "track", "monitor", "grad"])
    c = _case(kind=kind, prec=rng.choice(["fp64", "fp32", "fp32", "fp16s"]), film=rng.choice(["dewet", "drop", "hang"]),
              tau=rng.choice([1.0, 1.0, 1.0, 0.8, 0.9, 1.2]), ax=rng.choice([0.0, 1.0e-5]), theta=rng.random() < 0.7)
    if kind == "grad":
        c["prec"] = rng.choice(["fp64", "fp32"])
        c["film"] = "dewet"
        c["theta"] = True
    top = 2048 if kind == "grad" else 4096
    c["nx"], c["ny"] = _size(rng, 64, top), _size(rng, 64, top)
    if rng.random() < 0.3:  # a multiple of 64, as most users pick them
        c["nx"], c["ny"] = (max(64, v // 64 * 64) for v in (c["nx"], c["ny"]))
    if c["film"] == "hang":
        c["g"], c["theta"] = -1.0e-4, False
    elif rng.random() < 0.3:
        c["g"] = 1.0e-3
    if c["film"] == "drop":
        c["radius"] = min(100.0, rng.uniform(0.2, 0.3) * min(c["nx"], c["ny"]))
        c["delta"] = rng.choice([1.0, 4.0])
    c["gamma"] = kind != "grad" and rng.random() < 0.2
    sites = c["nx"] * c["ny"]
    cap = (LARGEST_GRAD if kind == "grad" else LARGEST // 2) / sites
    if kind in ("track", "monitor"):
        c["samples"] = rng.randint(2, 6)
        cap /= c["samples"]
    # a launch-bound lattice costs its steps, a large one its site-steps
    c["steps"] = max(1, min(int(cap), _size(rng, 1, 60 if kind in ("track", "monitor") else 600)))
    if kind == "grad":
        c["steps"] = min(c["steps"], 256)
        c["K"] = rng.choice([0, 16, 64])
    return c


# ---- inputs --------------------------------------------------------------------
def _film(c, seed, dev):
    """(parameters, h0, theta field or None, gamma field or None) on `dev`."""
    nx, ny = c["nx"], c["ny"]
    gen = torch.Generator(device=dev).manual_seed(int(seed))

    def noise():
        return torch.rand((ny, nx), generator=gen, dtype=F64, device=dev) * 2.0 - 1.0

    p = dict(tau=c["tau"], gamma=GAMMA, g=c["g"], n=9, m=3, ax=c["ax"])
    x = torch.arange(nx, dtype=F64, device=dev).view(1, -1)
    y = torch.arange(ny, dtype=F64, device=dev).view(-1, 1)
    if c["film"] == "dewet":
        p.update(hstar=0.09, delta=1.0)
        h0, href, angle = 0.1 + 1.0e-4 * noise(), 0.1, math.pi / 6
    elif c["film"] == "hang":
        p.update(hstar=0.05, delta=0.5)
        h0, href, angle = 1.0 + 1.0e-3 * noise(), 1.0, 0.0
    else:
        p.update(hstar=c["hstar"], delta=c["delta"])
        # a cap at a seeded place, within 5 % of the radius asked for
        r = c["radius"] * (1.0 + 0.05 * (2.0 * torch.rand((), generator=gen, dtype=F64, device=dev) - 1.0))
        at = torch.rand((2,), generator=gen, dtype=F64, device=dev)
        big = r / math.sin(c["angle0"])
        dx = torch.remainder(x - at[0] * nx + nx / 2, nx) - nx / 2
        dy = torch.remainder(y - at[1] * ny + ny / 2, ny) - ny / 2
        cap = torch.sqrt((big * big - dx * dx - dy * dy).clamp(min=0.0)) - big * math.cos(c["angle0"])
        h0, href, angle = cap.clamp(min=c["hstar"]), c["hstar"], math.pi / 9
    p["theta0"] = angle
    p["href"] = href if c["prec"] != "fp64" else 0.0
    theta = gam = None
    if c["theta"]:
        if c["film"] == "dewet" and c["kind"] != "grad":
            # stripes of period 256 (a quarter of a small lattice) between pi/9 and pi/4, smooth edges
            period = 256 if nx >= 512 else max(16, nx // 4)
            s = 0.5 * (1.0 + torch.tanh(8.0 * torch.sin(2.0 * math.pi * x / period)))
            theta = (math.pi / 9 + (math.pi / 4 - math.pi / 9) * s).expand(ny, nx).contiguous()
        else:
            theta = angle + 0.05 * noise() if c["film"] == "dewet" else torch.full((ny, nx), angle, dtype=F64, device=dev)
    if c["gamma"]:
        gam = GAMMA * (1.0 + 0.2 * torch.sin(2.0 * math.pi * x / nx) * torch.cos(2.0 * math.pi * y / ny)
                       + 0.05 * noise())
    return p, h0, theta, gam


def _target(c, seed, dev):
    """A smooth target height for the design loop's misfit."""
    gen = torch.Generator(device=dev).manual_seed(int(seed) + 7919)
    a = 2.0 * math.pi * torch.rand((4,), generator=gen, dtype=F64, device=dev)
    x = 2.0 * math.pi * torch.arange(c["nx"], dtype=F64, device=dev).view(1, -1) / c["nx"]
    y = 2.0 * math.pi * torch.arange(c["ny"], dtype=F64, device=dev).view(-1, 1) / c["ny"]
    return 0.1 + 0.005 * (torch.sin(3 * x + a[0]) * torch.cos(2 * y + a[1]) + torch.cos(x + a[2]) * torch.sin(4 * y + a[3]))


def prepare(case, seed):
    c, dev = case, torch.device("cuda", torch.cuda.current_device())
    p, h0, theta, gam = _film(c, seed, dev)
    s = {"case": c, "p": p, "h0": h0, "theta": theta, "gamma": gam}
    if c["kind"] == "grad":
        s["h0"] = h0.requires_grad_(True)
        s["theta"] = theta.requires_grad_(True)
        s["target"] = _target(c, seed, dev)
    else:
        s["sim"] = Sim(c["nx"], c["ny"], c["prec"], device=dev, gamma_field=gam is not None, **p)
    return s


def run(state):
    c = state["case"]
    if c["kind"] == "grad":
        h0, theta = state["h0"], state["theta"]
        h = TFLBMRun.apply(h0, theta, state["p"], c["steps"], c["K"], c["prec"])
        loss = 0.5 * ((h - state["target"]) ** 2).sum()
        return (h,) + torch.autograd.grad(loss, (h0, theta))
    sim = state["sim"].init(state["h0"], state["theta"], state["gamma"])
    if c["kind"] == "run":
        return sim.step(c["steps"]).read()
    if c["kind"] == "track":
        return [sim.step(c["steps"]).height() for _ in range(c["samples"])]
    watched = []
    for _ in range(c["samples"]):
        sim.step(c["steps"])
        watched += [sim.mass()] + list(sim.term_norms().values())
    return watched, sim.read()


def work(case):
    """Inputs read once and outputs written once (FP64 arrays); about 200
    floating-point operations per site of a step, 450 of a reverse step."""
    c = case
    sites, steps = c["nx"] * c["ny"], c["steps"] * c["samples"]
    ins = 8 * (1 + bool(c["theta"]) + bool(c["gamma"]) + (c["kind"] == "grad"))
    outs = {"run": 24, "track": 8 * c["samples"], "monitor": 24, "grad": 24}[c["kind"]]
    return {"bytes": sites * (ins + outs), "flops": sites * steps * (650 if c["kind"] == "grad" else 200)}


# ---- the same in plain torch, FP64 ---------------------------------------------
_C = [(0, 0), (1, 0), (1, 1), (0, 1), (-1, 1), (-1, 0), (-1, -1), (0, -1), (1, -1)]


def _at(a, c):
    """b(x) = a(x + c), periodic."""
    return torch.roll(a, (-c[1], -c[0]), (-2, -1)) if c != (0, 0) else a


def _gradient(a):
    gx = gy = 0.0
    for l, (cx, cy) in enumerate(_C[1:], 1):
        b = _at(a, (cx, cy)) * (1.0 / 3.0 if l % 2 else 1.0 / 12.0)
        gx, gy = gx + cx * b, gy + cy * b
    return gx, gy


def _laplacian(a):
    s = -20.0 * a
    for l, c in enumerate(_C[1:], 1):
        s = s + (4.0 if l % 2 else 1.0) * _at(a, c)
    return s / 6.0


def _moments(f):
    h = sum(f[1:], f[0])
    return h, f[1] + f[2] - f[4] - f[5] - f[6] + f[8], f[2] + f[3] + f[4] - f[6] - f[7] - f[8]


def _pressure(h, kap, gam, p):
    r = p["hstar"] / h
    return -gam * (_laplacian(h) + kap * (r ** p["n"] - r ** p["m"]))


def _friction(h, p):
    nu = (p["tau"] - 0.5) / 3.0
    return nu * 6.0 * h / (2.0 * h * h + 6.0 * p["delta"] * h + 3.0 * p["delta"] ** 2)


def _equilibrium(h, ux, uy, g):
    usq, out = ux * ux + uy * uy, []
    for l, (cx, cy) in enumerate(_C):
        cu = cx * ux + cy * uy
        if l == 0:
            out.append(h - 5.0 * g * h * h / 6.0 - 2.0 * h * usq / 3.0)
        elif l % 2:
            out.append(g * h * h / 6.0 + h * (cu / 3.0 + cu * cu / 2.0 - usq / 6.0))
        else:
            out.append(g * h * h / 24.0 + h * (cu / 12.0 + cu * cu / 8.0 - usq / 24.0))
    return out


def _step(p, kap, gam, *f):
    h, jx, jy = _moments(f)
    ux, uy = jx / h, jy / h
    gx, gy = _gradient(_pressure(h, kap, gam, p))
    fric = _friction(h, p)
    fx, fy = h * (p["ax"] - gx) - fric * ux, -h * gy - fric * uy
    out = []
    for l, ((cx, cy), fe) in enumerate(zip(_C, _equilibrium(h, ux, uy, p["g"]))):
        w3 = 0.0 if l == 0 else (1.0 / 3.0 if l % 2 else 1.0 / 12.0)
        post = f[l] + (fe - f[l]) / p["tau"] + w3 * (cx * fx + cy * fy)
        out.append(_at(post, (-cx, -cy)))
    return tuple(out)


def _norms(p, f, kap, gam):
    h, jx, jy = _moments(f)
    ux, uy, nu = jx / h, jy / h, (p["tau"] - 0.5) / 3.0
    gx, gy = _gradient(_pressure(h, kap, gam, p))
    fric = _friction(h, p)
    dx, dy = _gradient(_gradient(jx)[0] + _gradient(jy)[1])
    terms = [-h * gx, -fric * ux, nu * _laplacian(jx) + 2 * nu * dx, _gradient(jx * ux)[0] + _gradient(jy * ux)[1],
             -h * gy, -fric * uy, nu * _laplacian(jy) + 2 * nu * dy, _gradient(jx * uy)[0] + _gradient(jy * uy)[1]]
    return [float(t.square().mean().sqrt()) for t in terms]


def exact(case, seed):
    c, dev = case, torch.device("cuda", torch.cuda.current_device())
    p, h0, theta, gam = _film(c, seed, dev)
    kc = (p["n"] - 1) * (p["m"] - 1) / ((p["n"] - p["m"]) * p["hstar"])
    grad = c["kind"] == "grad"
    if grad:
        h0, theta = h0.requires_grad_(True), theta.requires_grad_(True)
    kap = (1.0 - math.cos(p["theta0"])) * kc if theta is None else (1.0 - torch.cos(theta)) * kc
    g = p["gamma"] if gam is None else gam
    z = torch.zeros_like(h0)
    f = tuple(_equilibrium(h0, z, z, p["g"]))
    if grad:
        from torch.utils.checkpoint import checkpoint
        for _ in range(c["steps"]):
            f = checkpoint(_step, p, kap, g, *f, use_reentrant=False)
        h = _moments(f)[0]
        loss = 0.5 * ((h - _target(c, seed, dev)) ** 2).sum()
        gh, gt = torch.autograd.grad(loss, (h0, theta))
        return h.detach(), gh, gt
    heights, watched = [], []
    for _ in range(c["samples"]):
        for _ in range(c["steps"]):
            f = _step(p, kap, g, *f)
        if c["kind"] == "track":
            heights.append(_moments(f)[0])
        elif c["kind"] == "monitor":
            watched += [float(_moments(f)[0].sum())] + _norms(p, f, kap, g)
    if c["kind"] == "track":
        return heights
    h, jx, jy = _moments(f)
    end = (h, jx / h, jy / h)
    return end if c["kind"] == "run" else (watched, end)
