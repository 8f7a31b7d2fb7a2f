"""The work whose speed is followed: calls of the public entry points over the
sizes, models, opening angles and options that the workloads, the tests and the
benchmark of this repository use.

A case is a dict of plain values; its "kind" says which entry points one pass
calls:

  static   tree_force_static: build + force without a context (n <= 65536)
  force    Tree.build + Tree.force on new positions
  step     leapfrog steps, then the state is read out
  vjp      Tree.build + Tree.force + the force's adjoint
  grad     a differentiated run: leapfrog steps, surface density, squared
           error, and its gradient in the initial state and the masses
  direct   FP64 direct sum at some of the particles
  density  surface density and its adjoint on new positions
  domains  local essential trees and forces of several domains

The particles are drawn on the GPU: a Plummer sphere, or an exponential disk
(a fifth of the particles) in a Hernquist halo, the two models of the
workloads.
"""
import math

import torch
import torch.utils.checkpoint

import paper_1412_0659_amd as bh
from paper_1412_0659_amd import binding
from paper_1412_0659_amd.autograd import leapfrog, surface_density

DEV = "cuda"
GRID = (0.2, 4.0, 16, 32)      # surface density: r_min, r_max, n_r, n_phi
SMALL_GRID = (0.2, 4.0, 8, 8)  # the same for a few thousand particles


def listed():
    return [
        # a serving loop or harness around a small cluster: launches and latency count
        dict(name="static_plummer_1000", kind="static", model="plummer", n=1000, theta=0.5, eps=0.01),
        # the 16k Plummer workload: forces on new positions
        dict(name="force_plummer_16k", kind="force", model="plummer", n=16384, theta=0.5, eps=0.01,
             fp16=False, curve="morton", pairs=0),
        # a ragged count, the paper's curve, paired target sets
        dict(name="force_ph_pairs_100003", kind="force", model="disk", n=100003, theta=0.6,
             eps=0.005, fp16=False, curve="ph", pairs=48),
        # the FP16 far field
        dict(name="force_fp16_1m", kind="force", model="disk", n=1000000, theta=0.4, eps=0.005,
             fp16=True, curve="morton", pairs=0),
        # a small run that is advanced step by step, FP64 position master
        dict(name="step_plummer_4099", kind="step", model="plummer", n=4099, theta=0.5, eps=0.01,
             steps=8, fp64=True),
        # the 1M disk + halo workload
        dict(name="step_disk_1m", kind="step", model="disk", n=1000000, theta=0.4, eps=0.005,
             steps=4, fp64=False),
        # the benchmark's 13M workload
        dict(name="step_disk_13m", kind="step", model="disk", n=13000000, theta=0.4, eps=0.002,
             steps=1, fp64=False),
        # force and its adjoint at the differentiation workload's size
        dict(name="vjp_disk_1m", kind="vjp", model="disk", n=1000000, theta=0.4, eps=0.005,
             pairs=0),
        # the 4096-particle differentiation workload, a quarter of its steps
        dict(name="grad_disk_4096", kind="grad", model="disk", n=4096, theta=0.4, eps=0.005,
             steps=16, every=8),
        # error of a tree force against the direct sum at a sample of targets
        dict(name="direct_8192_of_1m", kind="direct", model="disk", n=1000000, targets=8192,
             eps=0.005),
        # the observable of the differentiation workload and its adjoint
        dict(name="density_1m", kind="density", model="disk", n=1000000),
        # four domains on one device: trees exchanged, then forces
        dict(name="domains4_262144", kind="domains", model="disk", n=262144, theta=0.4, eps=0.005,
             domains=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["static", "force", "force", "step", "vjp", "grad", "direct", "density",
                       "domains"])
    model = rng.choice(["plummer", "disk"])
    theta = round(rng.uniform(0.3, 0.8), 3)
    eps = rng.choice([0.002, 0.005, 0.01])
    if kind == "static":
        return dict(kind=kind, model=model, n=_log(rng, 64, 65536), theta=theta, eps=eps)
    if kind == "force":
        return dict(kind=kind, model=model, n=_log(rng, 300, 4000000), theta=theta, eps=eps,
                    fp16=rng.random() < 0.3, curve=rng.choice(["morton", "ph"]),
                    pairs=rng.choice([0, 0, 32, 48, 64]))
    if kind == "step":
        n = _log(rng, 500, 6000000)
        return dict(kind=kind, model=model, n=n, theta=theta, eps=eps,
                    steps=1 if n > 1000000 else rng.randint(1, 8), fp64=rng.random() < 0.5)
    if kind == "vjp":
        return dict(kind=kind, model=model, n=_log(rng, 500, 1000000), theta=theta, eps=eps,
                    pairs=rng.choice([0, 0, 48]))
    if kind == "grad":
        return dict(kind=kind, model="disk", n=_log(rng, 1000, 16384), theta=theta, eps=0.005,
                    steps=rng.randint(4, 16), every=rng.choice([4, 8]))
    if kind == "direct":
        n = _log(rng, 2000, 2000000)
        return dict(kind=kind, model=model, n=n, targets=min(n, _log(rng, 64, 8192)), eps=eps)
    if kind == "density":
        return dict(kind=kind, model="disk", n=_log(rng, 2000, 4000000))
    return dict(kind=kind, model=model, n=_log(rng, 20000, 1000000), theta=theta, eps=eps,
                domains=rng.randint(2, 8))


# ---- particles ---------------------------------------------------------------


def _unit(n, g):
    z = 2.0 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64) - 1.0
    ph = 2.0 * math.pi * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    s = torch.sqrt(torch.clamp(1.0 - z * z, min=0.0))
    return torch.stack([s * torch.cos(ph), s * torch.sin(ph), z], 1)


def _plummer(n, g):
    u = 1.0 - torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    r = 1.0 / torch.sqrt(torch.clamp(u ** (-2.0 / 3.0) - 1.0, min=1e-12))
    pos = r[:, None] * _unit(n, g)
    sig = torch.sqrt(1.0 / (6.0 * torch.sqrt(1.0 + r * r)))
    vel = sig[:, None] * torch.randn(n, 3, generator=g, device=DEV, dtype=torch.float64)
    return pos, vel, torch.full((n,), 1.0 / n, device=DEV, dtype=torch.float64)


def _disk_halo(n, g):
    nd = max(1, n // 5)
    nh = n - nd
    # disk: surface density exp(-R) to R = 10, sech^2(z / 0.1) to |z| = 1, mass 0.1
    R = -torch.log(torch.rand(2, nd, generator=g, device=DEV, dtype=torch.float64) + 1e-300).sum(0)
    R = torch.where(R < 10.0, R, torch.remainder(R, 10.0))
    ph = 2.0 * math.pi * torch.rand(nd, generator=g, device=DEV, dtype=torch.float64)
    w = 2.0 * torch.rand(nd, generator=g, device=DEV, dtype=torch.float64) - 1.0
    z = torch.clamp(0.1 * torch.atanh(torch.clamp(w, -1.0 + 1e-8, 1.0 - 1e-8)), -1.0, 1.0)
    c, s = torch.cos(ph), torch.sin(ph)
    dpos = torch.stack([R * c, R * s, z], 1)
    # halo: Hernquist, mass 1, scale 5, to 20 scale radii
    q = torch.sqrt(torch.rand(nh, generator=g, device=DEV, dtype=torch.float64)) * (20.0 / 21.0)
    r = 5.0 * q / (1.0 - q)
    hpos = r[:, None] * _unit(nh, g)

    def enclosed(x):
        return x * x / (x + 5.0) ** 2 + 0.1 * (1.0 - (1.0 + x) * torch.exp(-x))

    vc = torch.sqrt(enclosed(R) / torch.clamp(R, min=1e-9))
    k = 0.1 * vc[:, None] * torch.randn(nd, 3, generator=g, device=DEV, dtype=torch.float64)
    dvel = torch.stack([k[:, 0] - vc * s, k[:, 1] + vc * c, k[:, 2]], 1)
    sig = torch.sqrt(enclosed(r) / torch.clamp(3.0 * r, min=1e-9))
    hvel = sig[:, None] * torch.randn(nh, 3, generator=g, device=DEV, dtype=torch.float64)
    mass = torch.cat([torch.full((nd,), 0.1 / nd, device=DEV, dtype=torch.float64),
                      torch.full((nh,), 1.0 / max(nh, 1), device=DEV, dtype=torch.float64)])
    return torch.cat([dpos, hpos]), torch.cat([dvel, hvel]), mass


def _particles(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    n = case["n"]
    pos, vel, mass = (_plummer if case["model"] == "plummer" else _disk_halo)(n, g)
    f = torch.float32
    return pos.to(f).contiguous(), vel.to(f).contiguous(), mass.to(f).contiguous(), g


def _disk_mask(n):
    sel = torch.zeros(n, dtype=torch.uint8, device=DEV)
    sel[:max(1, n // 5)] = 1
    return sel


# ---- one pass ----------------------------------------------------------------


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    pos, vel, mass, g = _particles(case, seed)
    s = dict(case=case, pos=pos, mass=mass)
    if kind == "static":
        s["acc"] = torch.empty((n, 3), dtype=torch.float32, device=DEV)
        s["pot"] = torch.empty((n,), dtype=torch.float32, device=DEV)
    elif kind == "force":
        s["tree"] = bh.Tree(n, far_fp16=case["fp16"], curve=case["curve"],
                            pair_groups=case["pairs"])
    elif kind == "step":
        s["tree"] = bh.Tree(n, pos_fp64=case["fp64"])
        s["tree"].set_state(pos, vel, mass)
    elif kind == "vjp":
        s["tree"] = bh.Tree(n, adjoint=True, pair_groups=case["pairs"])
        s["u"] = torch.randn(n, 3, generator=g, device=DEV)
    elif kind == "grad":
        s["tree"] = bh.Tree(n, adjoint=True, pos_fp64=True)
        s["vel"] = vel
        s["sel"] = _disk_mask(n)
        # the density to fit: another realisation of the model
        other, _, om, _ = _particles(case, seed + 1000003)
        s["target"] = surface_density(other, om, s["sel"], s["tree"], SMALL_GRID)
    elif kind == "direct":
        s["tree"] = bh.Tree(n)
        s["tree"].build(pos, mass)
        s["targets"] = torch.randperm(n, generator=g, device=DEV)[:case["targets"]].contiguous()
    elif kind == "density":
        s["tree"] = bh.Tree(n)
        s["sel"] = _disk_mask(n)
        s["target"] = torch.rand(GRID[2], GRID[3], generator=g, device=DEV) * 0.01
    elif kind == "domains":
        s["dom"] = bh.Domains(pos, mass, case["domains"], case["theta"], case["eps"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "static":
        binding.tree_force_static(s["pos"], s["mass"], case["theta"], case["eps"], s["acc"],
                                  s["pot"])
        return s["acc"], s["pot"]
    if kind == "force":
        s["tree"].build(s["pos"], s["mass"])
        return s["tree"].force(case["theta"], case["eps"])
    if kind == "step":
        for _ in range(case["steps"]):
            s["tree"].step(1e-3, case["theta"], case["eps"])
        return s["tree"].state()
    if kind == "vjp":
        t = s["tree"]
        t.build(s["pos"], s["mass"])
        acc, pot = t.force(case["theta"], case["eps"])
        gp, gm = torch.zeros_like(s["pos"]), torch.zeros_like(s["mass"])
        t.force_vjp(case["theta"], case["eps"], s["u"], 1.0, gp, gm)
        return acc, pot, gp, gm
    if kind == "grad":
        x0, v0, m = (s[k].detach().requires_grad_(True) for k in ("pos", "vel", "mass"))
        xk, vk = leapfrog(x0, v0, m, s["tree"], 1e-3, case["steps"], case["theta"], case["eps"],
                          case["every"])
        den = surface_density(xk, m, s["sel"], s["tree"], SMALL_GRID)
        loss = ((den - s["target"]) ** 2).sum()
        return (xk.detach(), vk.detach(), den.detach()) + torch.autograd.grad(loss, (x0, v0, m))
    if kind == "direct":
        return s["tree"].direct(s["targets"], case["eps"])
    if kind == "density":
        p, m = (s[k].detach().requires_grad_(True) for k in ("pos", "mass"))
        den = surface_density(p, m, s["sel"], s["tree"], GRID)
        loss = ((den - s["target"]) ** 2).sum()
        return (den.detach(),) + torch.autograd.grad(loss, (p, m))
    s["dom"].build_lets()
    return s["dom"].forces()


# ---- what a pass cannot do without ---------------------------------------------


def _terms(n, theta):
    """Particle-particle and particle-cell terms per particle: the counts of the
    4M disk + halo set, (0.4 / theta)^2 and a logarithm in n away from it."""
    f = (0.4 / theta) ** 2.1 * math.log(max(n, 2)) / math.log(4e6)
    pp, pc = min(1413.0 * f, n), 4302.0 * f
    return pp, min(pc, max(n - pp, 0.0))


def _force_flops(n, theta):
    pp, pc = _terms(n, theta)
    return n * (23.0 * pp + 65.0 * pc)


def work(case):
    kind, n = case["kind"], case["n"]
    if kind in ("static", "force"):
        return dict(bytes=32.0 * n, flops=_force_flops(n, case["theta"]))
    if kind == "step":
        return dict(bytes=case["steps"] * 56.0 * n, flops=case["steps"] * _force_flops(n, case["theta"]))
    if kind == "vjp":  # the adjoint of a term costs about 2.8 times the term
        return dict(bytes=60.0 * n, flops=3.8 * _force_flops(n, case["theta"]))
    if kind == "grad":
        return dict(bytes=case["steps"] * 100.0 * n,
                    flops=4.8 * case["steps"] * _force_flops(n, case["theta"]))
    if kind == "direct":
        return dict(bytes=16.0 * n + 40.0 * case["targets"], flops=20.0 * n * case["targets"])
    if kind == "density":
        return dict(bytes=17.0 * n + 33.0 * n, flops=60.0 * n)
    return dict(bytes=32.0 * n, flops=_force_flops(n, case["theta"]))


# ---- the same in 64 bits ---------------------------------------------------------


def _direct(x, m, eps, targets=None):
    """Acceleration and potential of the FP64 direct sum, self pair excluded."""
    n = x.shape[0]
    idx = torch.arange(n, device=x.device) if targets is None else targets
    acc = torch.empty(idx.shape[0], 3, device=x.device, dtype=torch.float64)
    pot = torch.empty(idx.shape[0], device=x.device, dtype=torch.float64)
    step = max(1, int(2.5e8) // n)
    xs = [x[:, k].contiguous() for k in range(3)]
    for a in range(0, idx.shape[0], step):
        i = idx[a:a + step]
        d = [xs[k][None, :] - xs[k][i][:, None] for k in range(3)]
        r2 = d[0] * d[0]
        r2.addcmul_(d[1], d[1]).addcmul_(d[2], d[2]).add_(eps * eps)
        w = r2.rsqrt_()
        w[torch.arange(i.shape[0], device=x.device), i] = 0.0
        mw = w * m[None, :]
        pot[a:a + step] = -mw.sum(1)
        mw.mul_(w).mul_(w)
        for k in range(3):
            acc[a:a + step, k] = (mw * d[k]).sum(1)
    return acc, pot


def _acc64(x, m, eps):
    """Differentiable FP64 direct-sum acceleration (a few thousand particles)."""
    d = x[None, :, :] - x[:, None, :]
    r2 = (d * d).sum(2) + eps * eps
    return ((m[None, :] * r2 ** -1.5)[:, :, None] * d).sum(1)


def _density64(x, m, sel, grid):
    r0, r1, nr, nphi = grid
    dr, dphi = (r1 - r0) / nr, 2.0 * math.pi / nphi
    R = torch.sqrt(x[:, 0] ** 2 + x[:, 1] ** 2)
    ph = torch.atan2(x[:, 1], x[:, 0])
    ph = torch.where(ph < 0, ph + 2.0 * math.pi, ph)
    u, v = (R - r0) / dr - 0.5, ph / dphi - 0.5
    i0, j0 = torch.floor(u.detach()), torch.floor(v.detach())
    fu, fv = u - i0, v - j0
    inside = (sel > 0) & (R >= r0) & (R < r1)
    out = torch.zeros(nr * nphi, device=x.device, dtype=torch.float64)
    for a in (0, 1):
        i = i0.long() + a
        wu = fu if a else 1.0 - fu
        for b in (0, 1):
            j = torch.remainder(j0.long() + b, nphi)
            wv = fv if b else 1.0 - fv
            ok = inside & (i >= 0) & (i < nr)
            out = out.index_add(0, (i * nphi + j)[ok], (m * wu * wv)[ok])
    edge = r0 + dr * torch.arange(nr + 1, device=x.device, dtype=torch.float64)
    area = 0.5 * dphi * (edge[1:] ** 2 - edge[:-1] ** 2)
    return out.reshape(nr, nphi) / area[:, None]


def _leapfrog64(x, v, m, dt, steps, eps, force):
    a = force(x, m, eps)
    for _ in range(steps):
        v = v + 0.5 * dt * a
        x = x + dt * v
        a = force(x, m, eps)
        v = v + 0.5 * dt * a
    return x, v


def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    eps, dt = _f32(case.get("eps", 0.0)), _f32(1e-3)
    if kind in ("static", "force", "domains") and n > 300000:
        return None
    if kind == "step" and (case["steps"] + 1) * float(n) ** 2 > 5e10:
        return None
    if kind == "vjp" and n > 20000 or kind == "grad" and n > 4096:
        return None
    pos, vel, mass, g = _particles(case, seed)
    x, v, m = pos.double(), vel.double(), mass.double()
    if kind in ("static", "force", "domains"):
        return _direct(x, m, eps)
    if kind == "step":
        return _leapfrog64(x, v, m, dt, case["steps"], eps, lambda a, b, e: _direct(a, b, e)[0])
    if kind == "vjp":
        u = torch.randn(n, 3, generator=g, device=DEV).double()
        acc, pot = _direct(x, m, eps)
        gp, gm = torch.zeros_like(x), torch.zeros_like(m)
        step = max(1, int(1e8) // n)
        for a in range(0, n, step):
            d = x[None, :, :] - x[a:a + step, None, :]
            ri = torch.rsqrt((d * d).sum(2) + eps * eps)
            ud = (u[a:a + step, None, :] * d).sum(2)
            ri3 = ri ** 3
            gm += (ud * ri3).sum(0)
            w = m[None, :, None] * (u[a:a + step, None, :] * ri3[:, :, None]
                                    - 3.0 * (ud * ri3 * ri * ri)[:, :, None] * d)
            gp += w.sum(0)
            gp[a:a + step] -= w.sum(1)
        return acc, pot, gp, gm
    if kind == "grad":
        sel = _disk_mask(n)
        other, _, om, _ = _particles(case, seed + 1000003)
        target = _density64(other.double(), om.double(), sel, SMALL_GRID)
        x, v, m = (t.requires_grad_(True) for t in (x, v, m))
        ck = torch.utils.checkpoint.checkpoint
        xk, vk = _leapfrog64(x, v, m, dt, case["steps"], eps,
                             lambda a, b, e: ck(_acc64, a, b, e, use_reentrant=False))
        den = _density64(xk, m, sel, SMALL_GRID)
        gr = torch.autograd.grad(((den - target) ** 2).sum(), (x, v, m))
        return (xk.detach(), vk.detach(), den.detach()) + gr
    if kind == "direct":
        t = torch.randperm(n, generator=g, device=DEV)[:case["targets"]].contiguous()
        return _direct(x, m, eps, t)
    sel = _disk_mask(n)
    target = (torch.rand(GRID[2], GRID[3], generator=g, device=DEV) * 0.01).double()
    x, m = x.requires_grad_(True), m.requires_grad_(True)
    den = _density64(x, m, sel, GRID)
    return (den.detach(),) + torch.autograd.grad(((den - target) ** 2).sum(), (x, m))
