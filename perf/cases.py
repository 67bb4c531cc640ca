"""The work a user of this package has it do, as cases that can be timed.

A case is a dict of plain values.  `path` says which public entry points it
goes through:

  run     Context.run on one problem, then its results (packets, or the
          spectrum of the escaped ones, and the peel-off cubes)
  batch   batch_run over many uneven problems in one launch
  adjoint the differentiable peel-off image: forward and gradients of a step
  replay  raycast_image and raycast_image_backward (no crossing list kept)
  tau     Context.tau: optical depths of rays to the domain border

`model` names the set-up, all of them this package's own configurations
(slab, sphere, dusty sphere on the adaptive mesh, outflowing shell, Fe II
wind, H + D sphere, thick sphere with core-skipping, galaxy-like mesh) at
optical depths and packet counts where one complete pass takes at most a
second or so.  `max_events` > 0 stops every packet at that interaction, as the
package's own timings do: at full optical depth it gives the bulk of a run
without its last, longest walks; the cases without it run every walk to its
end.
"""
import functools
import math

import numpy as np
import torch

from paper_2001_11252_amd import rmc
from paper_2001_11252_amd import workloads as W

DEV = "cuda:0"
STATS = ("emitted", "escaped", "absorbed", "stuck", "scatterings", "dust_scatterings", "crossings", "peel_rays",
         "peel_crossings", "peel_dropped")


# ------------------------------------------------------------------- cases
def _run(model, precision, tau0, packets, **kw):
    c = dict(path="run", model=model, precision=precision, tau0=float(tau0), packets=int(packets), level=3, observers=0,
             pixels=0, bins=0, v_kms=0.0, max_events=0, skip=False, voigt=False, result="packets")
    c.update(kw)
    return c


def _rays(path, mesh, precision, rays, **kw):
    c = dict(path=path, mesh=mesh, precision=precision, rays=int(rays), per_source=100, pixels=512, spread=20.0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a hundred packets through a thin slab, where
        # launches, copies and the latency of one walk are everything
        dict(_run("slab", "fp64", 100.0, 100), name="slab64_small"),
        # the plain slab test (1000 packets) to the end in double: one lane
        # after another walks its packet, the longest walk sets the time
        dict(_run("slab", "fp64", 1000.0, 1000), name="slab64"),
        # the headline: the dusty sphere at full depth on the adaptive mesh
        # with its observer's cube, the bulk of a float run
        dict(_run("dusty", "fp32", 1e6, 500_000, observers=1, pixels=128, bins=100, max_events=4000), name="dusty32_bulk"),
        # the same in double
        dict(_run("dusty", "fp64", 1e6, 150_000, observers=1, pixels=128, bins=100, max_events=2000), name="dusty64_bulk"),
        # a complete float run of the dusty sphere, long walks included
        dict(_run("dusty", "fp32", 5e3, 200_000, observers=1, pixels=128, bins=100), name="dusty32"),
        # the outflowing shell with its three observers (three peel-off rays
        # an event), complete, an odd packet count
        dict(_run("shell", "fp32", 1e5, 100_003, observers=3, pixels=96, bins=100, v_kms=200.0), name="shell32"),
        # the Fe II wind: continuum packets with few scatterings, two lines
        # with fluorescence; the user wants the emergent spectrum
        dict(_run("wind", "fp32", 0.0, 2_000_000, level=6, result="spectrum"), name="wind32"),
        # H + D: two lines in one medium, an observer, complete
        dict(_run("deuterium", "fp32", 1.2e3, 150_001, observers=1, pixels=128, bins=100), name="deuterium32"),
        # a survey: many uneven small problems in one launch
        dict(path="batch", precision="fp32", problems=24, packets=0.05, max_level=5, log_tau_max=3.7, name="batch32"),
        # a step of a fit: image and gradients with respect to the gas of a
        # galaxy-like adaptive mesh, float fields
        dict(_rays("adjoint", "galaxy", "fp32", 4_000_000), name="adjoint32"),
        # the same without crossing lists, in double, odd sizes
        dict(_rays("replay", "galaxy", "fp64", 300_007, per_source=37, pixels=201), name="replay64"),
        # column densities: optical depths of host-side rays
        dict(_rays("tau", "dusty", "fp64", 20_001, per_source=1, pixels=0), name="tau64"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """One more case: any path and model above, sizes log-uniform over the
    listed range, either precision."""
    kind = rng.choice(["slab", "sphere", "dusty", "bulk", "shell", "wind", "deuterium", "thick", "batch", "adjoint",
                       "replay", "tau"])
    prec = rng.choice(["fp32", "fp64"])
    if kind in ("slab", "sphere"):
        exact_h = prec == "fp64" and rng.random() < 0.3
        return _run(kind, prec, _log(rng, 30, 1000), _log(rng, 64, 20_000), level=rng.choice([0, 2, 3, 4, 5]),
                    observers=rng.choice([0, 0, 1]) if kind == "sphere" else 0, pixels=rng.randint(16, 64),
                    bins=rng.randint(20, 100), voigt=exact_h)
    if kind == "dusty":
        return _run(kind, prec, _log(rng, 300, 3000), _log(rng, 1000, 200_000), observers=rng.choice([0, 1, 2]),
                    pixels=rng.randint(16, 128), bins=rng.randint(20, 100))
    if kind == "bulk":
        return _run("dusty", prec, _log(rng, 1e5, 1e6), _log(rng, 20_000, 300_000 if prec == "fp32" else 100_000),
                    observers=1, pixels=rng.randint(32, 128), bins=rng.randint(20, 100),
                    max_events=rng.randint(200, 3000 if prec == "fp32" else 1500))
    if kind == "shell":
        return _run(kind, prec, _log(rng, 1e4, 1e5), _log(rng, 1000, 100_000), observers=rng.choice([1, 2, 3]),
                    pixels=rng.randint(16, 96), bins=rng.randint(20, 100), v_kms=200.0)
    if kind == "wind":
        return _run(kind, prec, 0.0, _log(rng, 10_000, 2_000_000), level=rng.choice([4, 5, 6]), result="spectrum")
    if kind == "deuterium":
        return _run(kind, prec, _log(rng, 100, 800), _log(rng, 1000, 100_000), observers=rng.choice([0, 1]),
                    pixels=rng.randint(16, 128), bins=rng.randint(20, 100))
    if kind == "thick":
        return _run(kind, prec, _log(rng, 1e4, 1e7), _log(rng, 1000, 100_000), skip=True, observers=1,
                    pixels=rng.randint(16, 128), bins=rng.randint(20, 100), max_events=rng.randint(300, 3000))
    if kind == "batch":
        return dict(path="batch", precision=prec, problems=rng.randint(3, 24), packets=_log(rng, 0.005, 0.05),
                    max_level=rng.choice([3, 4, 5]), log_tau_max=rng.uniform(2.5, 3.5))
    mesh = rng.choice(["galaxy", "dusty"])
    if kind == "tau":
        return _rays("tau", mesh, prec, _log(rng, 100, 200_000), per_source=1, pixels=0)
    return _rays(kind, mesh, prec, _log(rng, 2000, 4_000_000 if prec == "fp32" else 1_000_000),
                 per_source=rng.choice([1, 10, 37, 100]), pixels=rng.randint(20, 512), spread=rng.uniform(5.0, 20.0))


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=None)
def _mesh(name):
    if name == "dusty":
        return W.c2_mesh()
    if name == "shell":
        return W.c3_mesh(max_level=8)
    # galaxy: leaves refined on the gas mass of a k^-3 lognormal field
    dens = np.exp(2.0 * W.gaussian_field(64, -3.0, 0x5EED0005) - 2.0)
    rule = lambda lev, lo, hi: W._trilinear_periodic(dens, 0.5 * (lo + hi)) * 8.0 ** -lev > 6e-6  # noqa: E731
    return W.refined_mesh(5, 8, rule)


@functools.lru_cache(maxsize=None)
def _density(name):
    """Mean density field (mean about 1) of a mesh's leaves."""
    m = _mesh(name)
    if name != "galaxy":
        return np.ones(m.n)
    dens = np.exp(2.0 * W.gaussian_field(64, -3.0, 0x5EED0005) - 2.0)
    return W._trilinear_periodic(dens, m.centres()[0]).astype(np.float64)


def _problem(c, seed):
    n, tau0 = c["packets"], c["tau0"]
    if c["model"] == "slab":
        pb = W.static_slab(rmc.sigma0, tau0, 1e4, n, level=c["level"])
    elif c["model"] == "sphere":
        pb = W.static_sphere(rmc.sigma0, tau0, 1e4, n, level=c["level"], tau_dust=0.5)
    elif c["model"] == "dusty":
        pb = W.c2_dusty_sphere(rmc.sigma0, n, tau0, mesh=_mesh("dusty"))
    elif c["model"] == "shell":
        pb = W.c3_shell(rmc.sigma0, c["v_kms"], n, tau0, mesh=_mesh("shell"))
    elif c["model"] == "wind":
        pb = W.feii_wind(rmc.sigma0, n, level=c["level"])
    elif c["model"] == "deuterium":
        pb = W.deuterium_sphere(rmc.sigma0, n, N_HI=tau0 / rmc.sigma0(W.LYA, 1e4))
    else:
        pb = W.thick_sphere(rmc.sigma0, n, tau0)
    s3 = 1.0 / math.sqrt(3.0)
    half = 0.25 if c["model"] == "shell" else 0.5
    pb.observers = [W.Observer(k, c["pixels"], c["pixels"], c["bins"], (-half, half, -half, half), -60.0, 60.0)
                    for k in ((0.0, 0.0, 1.0), (1.0, 0.0, 0.0), (s3, s3, s3))[:c["observers"]]]
    pb.seed = seed
    return pb


def _context(c, pb):
    ctx = rmc.Context.from_problem(pb, c["precision"])
    ctx.set_stream(torch.cuda.current_stream())
    if c["max_events"]:
        ctx.set_option(rmc.OPT_MAX_EVENTS, c["max_events"])
    if c["skip"]:
        ctx.set_core_skip(1.0, 0.2)
    if c["voigt"]:
        ctx.set_option(rmc.OPT_VOIGT, 1)
    return ctx


def _ray_inputs(c, seed):
    """Gas fields and rays (on the GPU) of a ray case, from the seed."""
    m = _mesh(c["mesh"])
    g = torch.Generator(device=DEV).manual_seed(seed)
    rnd = lambda *s: torch.rand(*s, generator=g, device=DEV, dtype=torch.float64)  # noqa: E731
    nrm = lambda *s: torch.randn(*s, generator=g, device=DEV, dtype=torch.float64)  # noqa: E731
    T = 1e4
    rho = torch.as_tensor(_density(c["mesh"]), device=DEV) * torch.exp(0.3 * nrm(m.n))
    tau_mean = 1e4 if c["mesh"] == "galaxy" else 1e6
    n_hi = rho * (tau_mean / (rmc.sigma0(W.LYA, T) * m.box_cm))
    kd = rho / m.box_cm
    v = nrm(m.n, 3) * 3.0e6
    h = torch.as_tensor(np.ldexp(1.0, -m.level.astype(np.int64)), device=DEV)
    ijk = torch.as_tensor(m.ijk.astype(np.float64), device=DEV)
    n = c["rays"]
    ns = -(-n // c["per_source"])
    wts = rho * h ** 3
    cen = (ijk + 0.5) * h[:, None]
    wts = torch.where(((cen - 0.5) ** 2).sum(1) < 0.2, wts, torch.zeros_like(wts))   # well inside either domain
    leaf = torch.searchsorted(torch.cumsum(wts, 0) / wts.sum(), rnd(ns)).clamp_(max=m.n - 1)
    src = (ijk[leaf] + rnd(ns, 3)) * h[leaf][:, None]
    o = src.repeat_interleave(c["per_source"], 0)[:n].contiguous()
    x = (2.0 * rnd(n) - 1.0) * c["spread"]
    r = dict(mesh=m, T=T, n_hi=n_hi, kd=kd, v=v, o=o, x=x, w=torch.full((n,), 1.0 / (4.0 * math.pi), device=DEV,
                                                                       dtype=torch.float64))
    if c["path"] == "tau":
        d = nrm(n, 3)
        r["k"] = d / d.norm(dim=1, keepdim=True)
    else:
        r["G"] = nrm(c["pixels"], c["pixels"])
        r["k"] = torch.tensor([0.0, 0.0, 1.0], device=DEV, dtype=torch.float64).expand(n, 3)
    if c["precision"] == "fp32" and c["path"] == "adjoint":
        for f in ("n_hi", "kd", "v"):
            r[f] = r[f].float()
    return r


def _domain(c):
    return (W.DOM_BOX, (0.0, 0.0, 0.0, 0.0)) if c["mesh"] == "galaxy" else (W.DOM_SPHERE, (0.5, 0.5, 0.5, 0.5))


def prepare(case, seed):
    c = case
    s = dict(case=c, seed=seed)
    if c["path"] == "run":
        pb = _problem(c, seed)
        s["ctx"] = _context(c, pb)
    elif c["path"] == "batch":
        pbs = W.c4_batch(rmc.sigma0, n_problems=c["problems"], packet_scale=c["packets"], max_level=c["max_level"],
                         log_tau_range=(2.0, c["log_tau_max"]))
        rng = np.random.default_rng(seed)
        for i, p in enumerate(pbs):          # the survey's problems, each with a gas of its own
            p.gas.n_hi *= np.exp(0.3 * rng.standard_normal(p.mesh.n))
            p.seed = seed * 64 + i
        s["ctxs"] = [rmc.Context.from_problem(p, c["precision"]) for p in pbs]
        for x in s["ctxs"]:
            x.set_stream(torch.cuda.current_stream())
        s["seeds"] = [p.seed for p in pbs]
        s["packets"] = [len(p.sources.x) for p in pbs]
    else:
        r = _ray_inputs(c, seed)
        ctx = rmc.Context(c["precision"])
        ctx.set_stream(torch.cuda.current_stream())
        ctx.set_mesh(r["mesh"].level, r["mesh"].ijk, r["mesh"].box_cm)
        ctx.set_lines([W.LYA], r["T"])
        ctx.set_domain(*_domain(c))
        T = torch.full_like(r["n_hi"], r["T"])
        ctx.set_gas(r["n_hi"], T, r["v"].contiguous(), r["kd"])
        if c["pixels"]:
            ctx.add_observer((0.0, 0.0, 1.0), c["pixels"], c["pixels"], 1, (-0.5, 0.5, -0.5, 0.5), -1e30, 1e30)
        if c["path"] == "tau":
            s["rays"] = [t.cpu().numpy() for t in (r["o"], r["k"], r["x"])]
        else:
            s["r"], s["T"] = r, T
            if c["path"] == "adjoint":
                s["fn"] = rmc.raycast_image_fn()
                s["gas"] = [r[f].detach().requires_grad_() for f in ("n_hi", "kd", "v")]
        s["ctx"] = ctx
    return s


# -------------------------------------------------------------------- pass
def _stats(d):
    return np.array([d[k] for k in STATS], dtype=np.int64)


def run(state):
    c, ctx = state["case"], state.get("ctx")
    if c["path"] == "run":
        if c["observers"]:
            ctx.reset_cubes()
        out = dict(stats=_stats(ctx.run(state["seed"], 0, c["packets"])))
        if c["result"] == "packets":
            out["packets"] = ctx.get_packets()
        else:
            out["spectrum"] = ctx.get_spectrum(700, -400.0, 400.0)
        dt = np.float32 if c["precision"] == "fp32" else np.float64
        out["cubes"] = [ctx.get_cube(o, dt) for o in range(c["observers"])]
        return out
    if c["path"] == "batch":
        per, tot = rmc.batch_run(state["ctxs"], state["seeds"], state["packets"])
        pk = [x.get_packets() for x in state["ctxs"]]
        return dict(per=np.stack([_stats(p) for p in per]), total=_stats(tot),
                    packets={k: np.concatenate([p[k] for p in pk]) for k in pk[0]})
    if c["path"] == "tau":
        return ctx.tau(*state["rays"])
    r = state["r"]
    if c["path"] == "adjoint":
        n_hi, kd, v = state["gas"]
        img = state["fn"].apply(n_hi, kd, v, ctx, state["T"], 0, r["o"], r["x"], r["w"])
        return [img.detach()] + list(torch.autograd.grad(img, (n_hi, kd, v), r["G"]))
    img = ctx.raycast_image(0, r["o"], r["x"], r["w"])
    return [img] + list(ctx.raycast_image_backward(0, r["o"], r["x"], r["w"], r["G"]))


# -------------------------------------------------------------------- work
def work(case):
    """Bytes in and out and the arithmetic of the physics: 480 operations a
    scattering and 110 a cell crossing (the package's own counts)."""
    c = case
    if c["path"] == "run":
        n = c["packets"]
        if c["model"] == "wind":
            scat, cross = 0.25, 2.0 ** c["level"] * 0.5
        else:
            walk = 3.0 if c["model"] == "shell" else (1.6 if c["model"] == "slab" else 0.9) * c["tau0"]
            if c["skip"]:
                walk *= 0.5
            scat = min(walk, c["max_events"] or walk)
            cross = 20.0 + (0.0 if c["max_events"] else 0.02 * scat)
        flops = n * (480.0 * scat + 110.0 * (cross + c["observers"] * scat))
        out = 72.0 * n if c["result"] == "packets" else 700 * 8.0
        esz = 4 if c["precision"] == "fp32" else 8
        leaves = 8 ** c["level"] if c["model"] not in ("dusty", "shell") else 300_000
        return dict(bytes=32.0 * n + out + 8.0 * esz * leaves + c["observers"] * c["pixels"] ** 2 * c["bins"] * esz,
                    flops=flops)
    if c["path"] == "batch":
        n = c["problems"] * 1.4e5 * c["packets"]      # mean of 10^U(3,6) packets
        return dict(bytes=104.0 * n, flops=n * 480.0 * 10.0 ** (0.5 * (2.0 + c["log_tau_max"])))
    leaves = 500_000
    esz = 4.0 if c["precision"] == "fp32" else 8.0
    cross = c["rays"] * (60.0 if c["mesh"] == "galaxy" else 30.0)
    if c["path"] == "tau":
        return dict(bytes=64.0 * c["rays"] + 8.0 * esz * leaves, flops=110.0 * cross)
    return dict(bytes=2 * 40.0 * c["rays"] + 16.0 * esz * leaves + 40.0 * leaves + 16.0 * c["pixels"] ** 2,
                flops=2 * 110.0 * cross)


# ------------------------------------------------------- 64-bit values
C_CMS, KB, E_CGS, ME, AMU = 2.99792458e10, 1.380649e-16, 4.80320471e-10, 9.1093837015e-28, 1.66053906660e-24
LAM, A_UL, F_LU, MASS = 1215.67e-8, 6.265e8, 0.416, 1.00794   # Lya


def _voigt(a, x):
    """H(a, x) by the form of Tasitsiomi (2006) and its derivative."""
    x2 = x * x
    z = (x2 - 0.855) / (x2 + 3.42)
    p = ((5.674 * z - 9.207) * z + 4.421) * z + 0.1117
    dp = (17.022 * z - 18.414) * z + 4.421
    big = z > 0
    sx = torch.where(big, x, torch.ones_like(x))
    s2 = sx * sx
    dz = 2.0 * sx * 4.275 / (s2 + 3.42) ** 2
    f = (1.0 + 21.0 / s2) * a / (math.pi * (s2 + 1.0))
    df = (-42.0 / (s2 * sx)) * a / (math.pi * (s2 + 1.0)) - f * 2.0 * sx / (s2 + 1.0)
    e = torch.exp(-x2)
    rp = math.sqrt(math.pi)
    h = e + torch.where(big, rp * z * f * p, torch.zeros_like(x))
    dh = -2.0 * x * e + torch.where(big, rp * (dz * f * p + z * df * p + z * f * dp * dz), torch.zeros_like(x))
    return h, dh


def _leaf_grid(m):
    """Leaf of every cell of the deepest level, [z][y][x]."""
    L = int(m.level.max())
    grid = None
    for lev in range(L + 1):
        s = 1 << lev
        if grid is not None:
            grid = grid.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)
        else:
            grid = torch.full((s, s, s), -1, dtype=torch.int32, device=DEV)
        idx = np.nonzero(m.level == lev)[0]
        if len(idx):
            q = torch.as_tensor(m.ijk[idx].astype(np.int64), device=DEV)
            grid[q[:, 2], q[:, 1], q[:, 0]] = torch.as_tensor(idx.astype(np.int32), device=DEV)
    return grid.reshape(-1), L


def _walk(c, r, visit):
    """All rays cell by cell to the domain border: visit(rays, leaf, segment)
    for each step."""
    grid, L = _leaf_grid(r["mesh"])
    side = 1 << L
    h = torch.as_tensor(np.ldexp(1.0, -r["mesh"].level.astype(np.int64)), device=DEV)
    org = torch.as_tensor(r["mesh"].ijk.astype(np.float64), device=DEV) * h[:, None]
    p, k = r["o"].clone(), r["k"].contiguous()
    ray = torch.arange(len(p), device=DEV)
    ball = c["mesh"] != "galaxy"
    for _ in range(100_000):
        s = p * side
        q = torch.where(k >= 0, torch.floor(s), torch.ceil(s) - 1.0)
        ok = ((q >= 0) & (q < side)).all(1)
        p, k, ray, q = p[ok], k[ok], ray[ok], q[ok].long()
        if not len(ray):
            return
        leaf = grid[(q[:, 2] * side + q[:, 1]) * side + q[:, 0]].long()
        lo = org[leaf]
        hi = lo + h[leaf][:, None]
        t = torch.where(k != 0, (torch.where(k > 0, hi, lo) - p) / k, torch.full_like(p, math.inf))
        te, ax = t.min(1)
        te = te.clamp(min=0.0)
        seg, last = te, torch.zeros_like(te, dtype=torch.bool)
        if ball:
            d = p - 0.5
            b = (d * k).sum(1)
            disc = b * b - ((d * d).sum(1) - 0.25)
            td = torch.where(disc > 0, -b + torch.sqrt(disc.clamp(min=0.0)), torch.zeros_like(b)).clamp(min=0.0)
            last = td <= te
            seg = torch.minimum(te, td)
        visit(ray, leaf, seg)
        pn = torch.minimum(torch.maximum(p + te[:, None] * k, lo), hi)
        face = torch.where(k > 0, hi, lo)
        pn = torch.where(t <= te[:, None], face, pn)
        go = ~last
        p, k, ray = pn[go], k[go], ray[go]


def exact(case, seed):
    """Optical depths, images and gradients in 64 bits; a random walk has no
    such value."""
    c = case
    if c["path"] in ("run", "batch"):
        return None
    r = _ray_inputs(c, seed)
    n_hi, kd, v = (r[f].double() for f in ("n_hi", "kd", "v"))
    box = r["mesh"].box_cm
    vth = math.sqrt(2.0 * KB * r["T"] / (MASS * AMU))
    b = vth / C_CMS
    dnu = vth / LAM
    a = A_UL / (4.0 * math.pi * dnu)
    s0 = math.sqrt(math.pi) * E_CGS ** 2 * F_LU / (ME * C_CMS * dnu)
    tau = torch.zeros(len(r["o"]), dtype=torch.float64, device=DEV)

    def x_of(ray, leaf):
        w = (r["k"][ray] * v[leaf]).sum(1) / vth
        return (r["x"][ray] - w) / (1.0 + b * w), w

    def add(ray, leaf, seg):
        h, _ = _voigt(a, x_of(ray, leaf)[0])
        tau[ray] += (n_hi[leaf] * s0 * h + kd[leaf]) * seg * box

    _walk(c, r, add)
    if c["path"] == "tau":
        return tau.cpu().numpy()
    px = c["pixels"]
    # the image's axes for +z: x and y, from -1/2 to 1/2
    i = torch.floor(r["o"][:, 0] * px).long().clamp(0, px - 1)
    j = torch.floor(r["o"][:, 1] * px).long().clamp(0, px - 1)
    dep = r["w"] * torch.exp(-tau)
    img = torch.zeros(px * px, dtype=torch.float64, device=DEV).index_add_(0, j * px + i, dep)
    g = -r["G"].reshape(-1)[j * px + i] * dep
    gn, gk, gv = (torch.zeros_like(n_hi) for _ in range(3))

    def grad(ray, leaf, seg):
        x, w = x_of(ray, leaf)
        h, dh = _voigt(a, x)
        q = g[ray] * seg * box
        gn.index_add_(0, leaf, q * s0 * h)
        gk.index_add_(0, leaf, q)
        gv.index_add_(0, leaf, -q * n_hi[leaf] * s0 * dh * (1.0 + b * r["x"][ray]) / (1.0 + b * w) ** 2 / vth)

    _walk(c, r, grad)
    img = img.reshape(px, px)
    if c["path"] == "adjoint":
        return [img, gn, gk, torch.stack([torch.zeros_like(gv), torch.zeros_like(gv), gv], 1)]
    return [img, gn, gk, gv]
