"""The calls that stand for this library's use, for timing and for comparing two versions of it.

Every case goes through the Python entry points of paper_1902_03252_amd on inputs resident in GPU memory:
the image-plane chi^2 of one lens model (mixed and FP64), of a batch of proposals and of a Metropolis step, the
deflection field (FP64, FP32, the mixed-precision SIE gradient, NFW halos), its vector-Jacobian product and a
Hamiltonian step on the source-plane chi^2.  Sizes follow the package's own workloads (a 128^2 single lens, the
1024^2 / 50-potential cluster, the 4096^2 / 200-potential cluster, the 6730^2 image with 702 halos, the 512^2
differentiation grid, batches of 10 to 200 potentials on 256^2 to 2048^2 grids) and ragged ones between them.

A chi^2 case returns the chi^2, the per-system chi^2, the predicted-image counts, the sorted hits with their
positions and the pairing.  The `stats` array is left out: its counters say how the work was divided (how many
tests FP32 could not decide, how many tiles were culled), not what the lens model predicts.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

import paper_1902_03252_amd as lens

DEV = "cuda"
F64 = torch.float64
C_KMS = 299792.458
ARCSEC = 206264.80624709636
OBS_SIGMA = 0.1  # arcsec, positional error of an observed image


# ---------------------------------------------------------------- cases

def listed():
    return [
        # the smallest call: a single cored lens on a coarse grid, where launches and latency count
        dict(name="chi2_small", kind="chi2", prec="mixed", nx=128, ny=128, half=40.0, p=1, s=2, lens="single"),
        # a cluster model as a sampler evaluates it, mixed precision
        dict(name="chi2_cluster", kind="chi2", prec="mixed", nx=1024, ny=1024, half=80.0, p=50, s=20, lens="cluster"),
        # the largest chi^2: 200 potentials, a 4096^2 grid, 100 multiple-image systems
        dict(name="chi2_large", kind="chi2", prec="mixed", nx=4096, ny=4096, half=100.0, p=200, s=100, lens="cluster"),
        # the FP64 path on a ragged grid
        dict(name="chi2_fp64_ragged", kind="chi2", prec="fp64", nx=1000, ny=777, half=80.0, p=75, s=20, lens="cluster"),
        # a sampler's proposals: uneven potential counts and grid sides in one call
        dict(name="batch", kind="batch", prec="mixed", n=96, p_min=10, p_max=200, side_min=256, side_max=2048, s=20),
        # one Metropolis step of many chains on the differentiation grid
        dict(name="metropolis", kind="mh", prec="mixed", chains=256, nx=512, ny=512, half=80.0, p=50, s=20),
        # one Hamiltonian step (10 leapfrogs) on the source-plane chi^2: small kernels in a chain
        dict(name="hmc", kind="hmc", p=50, s=20, leapfrog=10),
        # a FP64 deflection map for plotting or for a pixelised source reconstruction
        dict(name="deflect_fp64", kind="deflect", prec="fp64", nx=2047, ny=1531, half=80.0, p=120, lens="cluster"),
        # a small FP32 deflection map, the ordinary interactive call
        dict(name="deflect_fp32", kind="deflect", prec="fp32", nx=411, ny=300, half=60.0, p=50, lens="cluster"),
        # the paper's own benchmark: mixed-precision SIE gradient of an HST image
        dict(name="sie_mixed", kind="sie_mixed", nx=6730, ny=6730, p=702),
        # the NFW cluster of the precision study
        dict(name="nfw_fp32", kind="nfw", prec="fp32", nx=4096, ny=4096, p=702),
        # forward and backward of the differentiable deflection field
        dict(name="vjp_fp64", kind="vjp", prec="fp64", nx=512, ny=512, half=80.0, p=50, lens="cluster"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes over their logarithms, odd ones among them."""
    kind = rng.choice(["chi2", "chi2", "batch", "mh", "hmc", "deflect", "deflect", "sie_mixed", "nfw", "vjp"])
    nx = _log(rng, 100, 4096)
    ny = max(64, min(4096, int(nx * rng.uniform(0.6, 1.5))))
    p = _log(rng, 1, 250)
    prec = rng.choice(["mixed", "fp64"])
    half = rng.choice([40.0, 60.0, 80.0, 100.0])
    if kind == "chi2":
        # FP64 costs about three times as much per node and potential
        while nx * ny * p > (3e9 if prec == "mixed" else 1e9):
            nx, ny = nx // 2 + 1, ny // 2 + 1
        return dict(kind=kind, prec=prec, nx=nx, ny=ny, half=half, p=p, s=_log(rng, 2, 100),
                    lens="single" if p == 1 else "cluster")
    if kind == "batch":
        return dict(kind=kind, prec=prec, n=_log(rng, 2, 96 if prec == "mixed" else 32), p_min=5,
                    p_max=rng.randint(20, 200), side_min=rng.randint(100, 256), side_max=rng.choice([500, 1024, 2048]),
                    s=_log(rng, 4, 40))
    if kind == "mh":
        return dict(kind=kind, prec="mixed", chains=_log(rng, 4, 256), nx=rng.randint(100, 512), ny=rng.randint(100, 512),
                    half=80.0, p=rng.randint(5, 60), s=_log(rng, 4, 20))
    if kind == "hmc":
        return dict(kind=kind, p=_log(rng, 2, 250), s=_log(rng, 2, 100), leapfrog=rng.randint(3, 20))
    if kind == "deflect":
        prec = rng.choice(["fp32", "fp64"])
        while nx * ny * p > (3e9 if prec == "fp32" else 1e9):
            nx, ny = nx // 2 + 1, ny // 2 + 1
        return dict(kind=kind, prec=prec, nx=nx, ny=ny, half=half, p=p, lens=rng.choice(["cluster", "sie"]))
    if kind == "sie_mixed":
        return dict(kind=kind, nx=nx, ny=ny, p=_log(rng, 3, 702))
    if kind == "nfw":
        prec = rng.choice(["fp32", "fp64"])
        p = _log(rng, 3, 702)
        while nx * ny * p > (1e10 if prec == "fp32" else 2e9):
            nx, ny = nx // 2 + 1, ny // 2 + 1
        return dict(kind=kind, prec=prec, nx=nx, ny=ny, p=p)
    nx, ny = _log(rng, 64, 1024), _log(rng, 64, 1024)
    return dict(kind="vjp", prec=rng.choice(["fp64", "mixed"]), nx=nx, ny=ny, half=80.0, p=_log(rng, 2, 100), lens="cluster")


# ---------------------------------------------------------------- inputs

def _t(a, dtype=F64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device=DEV)


def _grid(nx, ny, half):
    """nx x ny nodes centred on the origin, the longer side spanning [-half, half]."""
    h = 2.0 * half / (max(nx, ny) - 1)
    return types.SimpleNamespace(x0=-0.5 * (nx - 1) * h, y0=-0.5 * (ny - 1) * h, h=h, nx=nx, ny=ny)


def _image(nx, ny):
    """An image of 0.03 arcsec pixels centred on the origin."""
    h = 0.03
    return types.SimpleNamespace(x0=-0.5 * (nx - 1) * h, y0=-0.5 * (ny - 1) * h, h=h, nx=nx, ny=ny)


def _potentials(g, p, kind, half):
    """[7, p] table (x, y, eps, phi, r_core, r_cut, sigma_v): one lens at the centre; a cluster halo and galaxies
    over three quarters of the field; or singular uncut isothermal halos."""
    t = np.zeros((7, p))
    if kind == "sie":
        t[0], t[1] = g.uniform(-half, half, p), g.uniform(-half, half, p)
        t[2], t[3] = g.uniform(0.0, 0.3, p), g.uniform(0.0, math.pi, p)
        t[5], t[6] = np.inf, g.uniform(50.0, 400.0, p)
        return t
    if p > 1:
        n = p - 1
        t[0, 1:], t[1, 1:] = g.uniform(-0.75 * half, 0.75 * half, n), g.uniform(-0.75 * half, 0.75 * half, n)
        t[2, 1:], t[3, 1:] = g.uniform(0.0, 0.5, n), g.uniform(0.0, math.pi, n)
        t[4, 1:], t[5, 1:] = g.uniform(0.05, 0.3, n), g.uniform(20.0, 80.0, n)
        t[6, 1:] = np.exp(g.uniform(math.log(100.0), math.log(300.0), n))
    t[:, 0] = (0.0, 0.0, 0.05, 0.0, 5.0, 1000.0, 1000.0) if kind == "cluster" else (0.0, 0.0, 0.2, 0.52, 0.5, 300.0, 800.0)
    t[0, 0], t[1, 0] = g.normal(0.0, 0.3, 2)
    return t


def _halos(g, grid, p):
    """x, y, eps, phi of two cluster-scale halos and p - 2 galaxy-scale ones over the image."""
    lx, ly = 0.5 * (grid.nx - 1) * grid.h, 0.5 * (grid.ny - 1) * grid.h
    t = np.zeros((4, p))
    t[0], t[1] = g.uniform(-lx, lx, p), g.uniform(-ly, ly, p)
    t[2], t[3] = g.uniform(0.0, 0.15, p), g.uniform(0.0, math.pi, p)
    t[:, 0], t[:, 1] = (-0.2 * lx, -0.1 * ly, 0.05, 0.5), (0.25 * lx, 0.15 * ly, 0.04, 2.0)
    return t


def _dls(z_lens, z):
    """D_LS / D_OS in a flat universe with Omega_m = 0.3 (Simpson's rule)."""
    def comoving(x):
        u = np.linspace(0.0, 1.0, 4097)[None] * np.asarray(x, dtype=float)[:, None]
        f = 1.0 / np.sqrt(0.3 * (1 + u) ** 3 + 0.7)
        w = np.ones(4097)
        w[1:-1:2], w[2:-1:2] = 4.0, 2.0
        return (f * w).sum(1) * np.asarray(x) / 4096 / 3.0
    return 1.0 - comoving([z_lens])[0] / comoving(z)


def _systems(g, truth, s, half):
    """Multiple-image systems of the lens `truth` ([7, P] table), three observed images each: sources in the inner
    field whose images a 512^2 grid finds (three to five, as far as 4 s draws give them; an image is observed twice
    where there are fewer), positions with 0.1 arcsec noise."""
    n = max(4 * s, 16)
    radius = 2.0 if truth.shape[1] == 1 else 15.0
    rad, ang = radius * np.sqrt(g.uniform(0.0, 1.0, n)), g.uniform(0.0, 2.0 * math.pi, n)
    src = np.stack([rad * np.cos(ang), rad * np.sin(ang)], 1)
    dls = _dls(0.3, g.uniform(1.0, 6.0, n))
    noise = g.normal(0.0, OBS_SIGMA, (n, 3, 2))
    grid = _grid(512, 512, half)
    ax, ay = _alpha(_t(truth), grid)
    found = _hits(ax, ay, grid, _t(src[:, 0]), _t(src[:, 1]), _t(dls))
    images = [[] for _ in range(n)]
    for sys, x, y in zip(found[0].tolist(), found[2].tolist(), found[3].tolist()):
        images[int(sys)].append((x, y))
    order = sorted(range(n), key=lambda k: (not 3 <= len(images[k]) <= 5, not images[k], k))[:s]
    xy, off = [], [0]
    for k in order:
        here = images[k] or [tuple(src[k])]
        xy.append(np.array([here[m % len(here)] for m in range(3)]) + noise[k])
        off.append(off[-1] + 3)
    xy = np.concatenate(xy)
    return dict(sys_off=np.array(off, dtype=np.int32), x=xy[:, 0].copy(), y=xy[:, 1].copy(),
                sigma=np.full(len(xy), OBS_SIGMA), dls=dls[order])


def _proposal(g, truth, scale=0.002):
    """A sampler's proposal near the truth: every parameter times 1 + scale N(0, 1)."""
    t = truth * (1.0 + scale * g.normal(0.0, 1.0, truth.shape))
    t[2] = np.clip(t[2], 0.0, 0.5)
    return t


def _steps(p):
    """Metropolis / leapfrog step sizes: the halo's centre, shape, core and dispersion, the galaxies' dispersions."""
    st = np.zeros((7, p))
    st[0, 0] = st[1, 0] = 1e-3
    st[2, 0], st[3, 0], st[4, 0], st[6, 0] = 1e-4, 1e-3, 1e-3, 0.25
    st[6, 1:] = 0.1
    return st


def _inputs(case, seed):
    """Host inputs of a case, from the seed alone."""
    g, kind = np.random.Generator(np.random.PCG64(seed)), case["kind"]
    d = types.SimpleNamespace()
    if kind in ("chi2", "deflect", "vjp"):
        d.grid = _grid(case["nx"], case["ny"], case["half"])
        truth = _potentials(g, case["p"], case["lens"], case["half"])
        d.params = truth
        if kind == "chi2":
            d.obs = _systems(g, truth, case["s"], case["half"])
            d.params = _proposal(g, truth)
    elif kind == "batch":
        n = case["n"]
        truth = _potentials(g, 50, "cluster", 80.0)
        d.obs = _systems(g, truth, case["s"], 80.0)
        counts = g.integers(case["p_min"], case["p_max"] + 1, n)
        sides = np.exp(g.uniform(math.log(case["side_min"]), math.log(case["side_max"]), n))
        power = 2 ** np.clip(np.rint(np.log2(sides)), math.ceil(math.log2(case["side_min"])), math.floor(math.log2(case["side_max"])))
        sides = np.where(g.uniform(size=n) < 0.75, power, np.rint(sides)).astype(int)
        sides[0] = case["side_max"]
        d.grids = [_grid(int(v), int(v), 80.0) for v in sides]
        blocks = []
        for k in range(n):
            extra = _potentials(g, int(counts[k]) + 1, "cluster", 80.0)[:, 1:]
            keep = min(int(counts[k]), 50)
            extra[:, :keep] = truth[:, :keep]
            blocks.append(_proposal(g, extra, 0.02))
        d.params = np.concatenate(blocks, 1)
        d.pot_off = np.concatenate([[0], np.cumsum(counts)])
    elif kind in ("mh", "hmc"):
        half = case.get("half", 80.0)
        truth = _potentials(g, case["p"], "cluster", half)
        d.obs = _systems(g, truth, case["s"], half)
        d.step = _steps(case["p"])
        if kind == "mh":
            d.grid = _grid(case["nx"], case["ny"], half)
            d.params = np.tile(_proposal(g, truth, 5e-4), (1, case["chains"]))
            d.noise = g.normal(0.0, 1.0, d.params.shape)
            d.u = g.uniform(0.0, 1.0, case["chains"])
        else:
            d.params = _proposal(g, truth, 5e-4)
            d.noise = g.normal(0.0, 1.0, d.params.shape)
            d.u = g.uniform(0.0, 1.0, 1)
            d.step *= 0.1
    elif kind == "sie_mixed":
        d.grid = _image(case["nx"], case["ny"])
        t = np.zeros((7, case["p"]))
        t[:4] = _halos(g, d.grid, case["p"])
        t[5], t[6] = np.inf, g.uniform(10.0, 15.0, case["p"])
        t[6, 0], t[6, 1] = 1000.0, 700.0
        d.params = t
    else:
        d.grid = _image(case["nx"], case["ny"])
        t = np.zeros((6, case["p"]))
        t[:4] = _halos(g, d.grid, case["p"])
        t[4], t[5] = g.uniform(1.0, 4.0, case["p"]), g.uniform(0.01, 0.05, case["p"])
        t[4:, 0], t[4:, 1] = (40.0, 0.25), (30.0, 0.2)
        d.params = t
    return d


def prepare(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    s = types.SimpleNamespace(case=case, params=_t(d.params), grid=getattr(d, "grid", None))
    if kind in ("chi2", "batch", "mh", "hmc"):
        s.obs = lens.Obs.from_numpy(d.obs)
    if kind == "chi2":
        s.out = lens.chi2_buffers(s.obs, 4096, DEV)
    elif kind == "batch":
        s.layout = lens.BatchLayout(d.pot_off, d.grids)
        s.out = lens.batch_buffers(s.layout.n, s.obs, DEV, hits=True)
    elif kind in ("mh", "hmc"):
        s.step, s.noise, s.u = _t(d.step), _t(d.noise), _t(d.u)
        if kind == "mh":
            layout = lens.BatchLayout([k * case["p"] for k in range(case["chains"] + 1)], [s.grid] * case["chains"])
            s.chi2 = lens.lens_image_chi2_batched(s.params, layout, s.obs, prec=case["prec"]).chi2.clone()
    elif kind == "sie_mixed":
        s.out = lens.mixed_buffers(s.grid, DEV)
    elif kind == "vjp":
        g = torch.Generator(device=DEV).manual_seed(int(seed) + 17)
        s.params.requires_grad_(True)
        dt = F64 if case["prec"] == "fp64" else torch.float32
        s.cot = [torch.randn((s.grid.ny, s.grid.nx), generator=g, device=DEV, dtype=F64).to(dt) for _ in range(2)]
    return s


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "chi2":
        r = lens.lens_image_chi2(s.params, s.grid, s.obs, prec=case["prec"], out=s.out)
        return {k: getattr(r, k) for k in ("chi2", "chi2_sys", "n_pred", "hits", "img_xy", "match")}
    if kind == "batch":
        r = lens.lens_image_chi2_batched(s.params, s.layout, s.obs, prec=case["prec"], out=s.out)
        return {k: getattr(r, k) for k in ("chi2", "chi2_sys", "n_pred", "status", "n_hits", "hits", "img_xy")}
    if kind == "mh":
        acc = lens.mh_step_batched(s.params, case["chains"], s.grid, s.obs, s.step, s.noise, s.u, s.chi2, prec=case["prec"])
        return {"states": s.params, "chi2": s.chi2, "accepted": acc}
    if kind == "hmc":
        chi2, acc = lens.hmc_step(s.params, s.obs, s.step, case["leapfrog"], s.noise, s.u)
        return {"state": s.params, "chi2": chi2, "accepted": acc}
    if kind == "deflect":
        return lens.lens_deflect(s.params, s.grid, case["prec"])
    if kind == "nfw":
        return lens.lens_deflect_nfw(s.params, s.grid, case["prec"])
    if kind == "sie_mixed":
        r = lens.lens_deflect_mixed(s.params, s.grid, 2, out=s.out)
        return {"ax": r.ax, "ay": r.ay, "mask": r.mask, "stats": r.stats}
    ax, ay = lens.DeflectFn.apply(s.params, s.grid, case["prec"])
    (grad,) = torch.autograd.grad((ax, ay), s.params, s.cot)
    return {"ax": ax, "ay": ay, "grad": grad}


# ---------------------------------------------------------------- work

def work(case):
    """Bytes: the inputs once and the outputs once (a chi^2 has no field among its outputs).  Flops: at least one
    profile evaluation (34 flops; 26 for the SIE, about 60 for the NFW) per node and per (image, potential)."""
    kind = case["kind"]
    if kind == "hmc":
        n = case["p"] * case["s"] * 3.0 * (case["leapfrog"] + 1)
        return {"bytes": 8.0 * 7 * case["p"] * 4 + 32.0 * case["s"] * 3, "flops": (34.0 + 78.0) * n}
    if kind == "batch":
        mean_side2 = (case["side_max"] ** 2 - case["side_min"] ** 2) / (2 * math.log(case["side_max"] / case["side_min"]))
        nodes, pots = case["n"] * mean_side2, case["n"] * 0.5 * (case["p_min"] + case["p_max"])
        return {"bytes": 56.0 * pots + 20.0 * case["n"] * case["s"], "flops": 34.0 * (nodes + 3 * case["s"] * pots)}
    nodes = float(case["nx"]) * case["ny"]
    if kind == "chi2":
        return {"bytes": 56.0 * case["p"] + 150.0 * case["s"], "flops": 34.0 * (nodes + 3.0 * case["s"] * case["p"])}
    if kind == "mh":
        return {"bytes": 200.0 * case["p"] * case["chains"],
                "flops": 34.0 * case["chains"] * (nodes + 3.0 * case["s"] * case["p"])}
    if kind == "deflect":
        return {"bytes": nodes * (16 if case["prec"] == "fp64" else 8) + 56.0 * case["p"], "flops": 34.0 * nodes}
    if kind == "sie_mixed":
        return {"bytes": 17.0 * nodes + 56.0 * case["p"], "flops": 26.0 * nodes}
    if kind == "nfw":
        return {"bytes": nodes * (16 if case["prec"] == "fp64" else 8) + 48.0 * case["p"], "flops": 60.0 * nodes}
    per = 16 if case["prec"] == "fp64" else 8  # the field written, the cotangent read
    return {"bytes": 2.0 * nodes * per + 112.0 * case["p"], "flops": (34.0 + 78.0) * nodes}


# ---------------------------------------------------------------- plain torch in 64 bits

def _alpha_one(q, X, Y):
    """Deflection of one potential (7 scalars or 0-d tensors) at X, Y."""
    x, y, eps, phi, a, s, sig = q
    cut = math.isfinite(float(s))
    b0 = 4.0 * math.pi * (sig / C_KMS) ** 2 * ARCSEC
    c, n = torch.cos(torch.as_tensor(phi, dtype=F64)), torch.sin(torch.as_tensor(phi, dtype=F64))
    dx, dy = X - x, Y - y
    u, v = c * dx + n * dy, c * dy - n * dx
    mu, mv = (1.0 - eps) * u, (1.0 + eps) * v
    r2 = mu * u + mv * v
    qa = torch.sqrt(a * a + r2)
    if cut:
        qs = torch.sqrt(s * s + r2)
        f = b0 * s / (s - a) * (((s * s - a * a) / (qs + qa)) + (s - a)) / ((qa + a) * (qs + s))
    else:
        f = b0 / torch.where(qa + a > 0, qa + a, torch.full_like(qa, math.inf))
    mu, mv = f * mu, f * mv
    return c * mu - n * mv, n * mu + c * mv


def _alpha(params, grid):
    """(ax, ay) [ny, nx] of a [7, P] table."""
    X = (grid.x0 + torch.arange(grid.nx, dtype=F64, device=DEV) * grid.h)[None, :]
    Y = (grid.y0 + torch.arange(grid.ny, dtype=F64, device=DEV) * grid.h)[:, None]
    ax = torch.zeros((grid.ny, grid.nx), dtype=F64, device=DEV)
    ay = torch.zeros_like(ax)
    for q in params.detach().cpu().numpy().T:
        tx, ty = _alpha_one([float(v) for v in q], X, Y)
        ax += tx
        ay += ty
    return ax, ay


def _nfw(params, grid):
    X = (grid.x0 + torch.arange(grid.nx, dtype=F64, device=DEV) * grid.h)[None, :]
    Y = (grid.y0 + torch.arange(grid.ny, dtype=F64, device=DEV) * grid.h)[:, None]
    ax = torch.zeros((grid.ny, grid.nx), dtype=F64, device=DEV)
    ay = torch.zeros_like(ax)
    for x, y, eps, phi, rs, ks in params.detach().cpu().numpy().T:
        c, n = math.cos(phi), math.sin(phi)
        dx, dy = X - x, Y - y
        u, v = c * dx + n * dy, c * dy - n * dx
        mu, mv = (1.0 - eps) * u, (1.0 + eps) * v
        r2 = mu * u + mv * v
        x2 = (r2 / (rs * rs)).clamp(min=1e-200)
        t = torch.sqrt(x2)
        d = torch.sqrt((1.0 - x2).abs()).clamp(min=1e-150)
        small = x2 < 0.25
        outer = (torch.log(0.5 * t) + torch.where(x2 < 1.0, torch.atanh(torch.where(x2 < 1.0, d, 0.0)), torch.atan(d)) / d) / x2
        si = torch.sqrt((1.0 - x2).clamp(min=0.25))
        inner = (torch.log(2.0 / t) / (1.0 + si) + torch.log1p((-x2 / (2.0 * (1.0 + si))).clamp(min=-0.5)) / x2) / si
        f = 4.0 * ks * torch.where(small, inner, outer)
        f = torch.where(r2 > 0, f, 0.0)
        mu, mv = f * mu, f * mv
        ax += c * mu - n * mv
        ay += n * mu + c * mv
    return ax, ay


def _hits(ax, ay, grid, bx, by, dls):
    """Triangles of the grid that contain the sources (bx, by): (system, triangle id, x, y), sorted."""
    nx, ny, h = grid.nx, grid.ny, grid.h
    X = (grid.x0 + torch.arange(nx, dtype=F64, device=DEV) * h)[None, :]
    Y = (grid.y0 + torch.arange(ny, dtype=F64, device=DEV) * h)[:, None]
    got = []
    for s in range(len(bx)):
        px, py = X - dls[s] * ax - bx[s], Y - dls[s] * ay - by[s]
        v = {(0, 0): (px[:-1, :-1], py[:-1, :-1]), (1, 0): (px[:-1, 1:], py[:-1, 1:]),
             (0, 1): (px[1:, :-1], py[1:, :-1]), (1, 1): (px[1:, 1:], py[1:, 1:])}
        for k, t in enumerate((((0, 0), (1, 0), (0, 1)), ((1, 1), (0, 1), (1, 0)))):
            c = [v[t[i]][0] * v[t[(i + 1) % 3]][1] - v[t[i]][1] * v[t[(i + 1) % 3]][0] for i in range(3)]
            inside = ((c[0] > 0) & (c[1] > 0) & (c[2] > 0)) | ((c[0] < 0) & (c[1] < 0) & (c[2] < 0))
            j, i = torch.nonzero(inside, as_tuple=True)
            if not len(i):
                continue
            c = [q[inside] for q in c]
            lam = [c[(m + 1) % 3] / (c[0] + c[1] + c[2]) for m in range(3)]
            x = sum(lam[m] * (grid.x0 + (i + t[m][0]).to(F64) * h) for m in range(3))
            y = sum(lam[m] * (grid.y0 + (j + t[m][1]).to(F64) * h) for m in range(3))
            got.append(torch.stack([torch.full_like(x, s), (2 * (j * (nx - 1) + i) + k).to(F64), x, y]))
    if not got:
        return np.zeros((4, 0))
    got = torch.cat(got, 1).cpu().numpy()
    return got[:, np.lexsort((got[1], got[0]))]


def _exact_chi2(params, grid, obs):
    """chi^2, per-system chi^2 and image positions of one model ([7, P] tensor) and the observed systems."""
    off, s = obs["sys_off"], len(obs["dls"])
    of = np.repeat(np.arange(s), np.diff(off))
    X, Y = _t(obs["x"]), _t(obs["y"])
    axo, ayo = torch.zeros_like(X), torch.zeros_like(Y)
    for q in params.detach().cpu().numpy().T:
        tx, ty = _alpha_one([float(v) for v in q], X, Y)
        axo, ayo = axo + tx, ayo + ty
    sx = obs["x"] - obs["dls"][of] * axo.cpu().numpy()
    sy = obs["y"] - obs["dls"][of] * ayo.cpu().numpy()
    bx = np.array([sx[off[k]:off[k + 1]].mean() for k in range(s)])
    by = np.array([sy[off[k]:off[k + 1]].mean() for k in range(s)])
    ax, ay = _alpha(params, grid)
    found = _hits(ax, ay, grid, bx.tolist(), by.tolist(), obs["dls"].tolist())
    per = np.zeros(s)
    for k in range(s):
        m = found[0] == k
        if not m.any():
            per[k] = np.inf
            continue
        for j in range(off[k], off[k + 1]):
            per[k] += np.min((obs["x"][j] - found[2, m]) ** 2 + (obs["y"][j] - found[3, m]) ** 2) / obs["sigma"][j] ** 2
    return per.sum(), per, found[2:].T


def _src_chi2(q, obs):
    off, s = obs["sys_off"], len(obs["dls"])
    of = torch.as_tensor(np.repeat(np.arange(s), np.diff(off)), device=DEV)
    X, Y, r = _t(obs["x"]), _t(obs["y"]), _t(obs["dls"])[of]
    sx, sy = X, Y
    for k in range(q.shape[1]):
        tx, ty = _alpha_one([q[m, k] for m in range(7)], X, Y)
        sx, sy = sx - r * tx, sy - r * ty
    n = torch.bincount(of, minlength=s).to(F64)
    mx = torch.zeros(s, dtype=F64, device=DEV).index_add(0, of, sx) / n
    my = torch.zeros(s, dtype=F64, device=DEV).index_add(0, of, sy) / n
    return (((sx - mx[of]) ** 2 + (sy - my[of]) ** 2) / _t(obs["sigma"]) ** 2).sum()


def _padded(rows, cap):
    out = np.zeros((cap, 2))
    out[:len(rows)] = rows
    return out


def exact(case, seed):
    d, kind = _inputs(case, seed), case["kind"]
    if kind == "chi2":
        total, per, xy = _exact_chi2(_t(d.params), d.grid, d.obs)
        return {"chi2": np.array([total]), "chi2_sys": per, "n_pred": None, "hits": None, "img_xy": _padded(xy, 4096),
                "match": None}
    if kind == "batch":
        got = [_exact_chi2(_t(d.params[:, d.pot_off[k]:d.pot_off[k + 1]]), d.grids[k], d.obs) for k in range(case["n"])]
        return {"chi2": np.array([g[0] for g in got]), "chi2_sys": np.stack([g[1] for g in got]), "n_pred": None,
                "status": None, "n_hits": None, "hits": None, "img_xy": np.stack([_padded(g[2], 1024) for g in got])}
    if kind == "mh":
        p = case["p"]
        old = _exact_chi2(_t(d.params[:, :p]), d.grid, d.obs)[0]
        states, chi2 = d.params.copy(), np.full(case["chains"], old)
        for b in range(case["chains"]):
            cols = slice(b * p, (b + 1) * p)
            prop = d.params[:, cols] + d.step * d.noise[:, cols]
            if (prop[2] < 0).any() or (prop[2] >= 1).any() or (prop[4] < 0).any():
                continue
            new = _exact_chi2(_t(prop), d.grid, d.obs)[0]
            if math.isfinite(new) and (not math.isfinite(old) or math.log(d.u[b]) < -0.5 * (new - old)):
                states[:, cols], chi2[b] = prop, new
        return {"states": states, "chi2": chi2, "accepted": None}
    if kind == "hmc":
        def grad(q):
            q = q.clone().requires_grad_(True)
            c = _src_chi2(q, d.obs)
            return float(c), torch.autograd.grad(c, q)[0]
        step, q, m = _t(d.step), _t(d.params), _t(d.noise)
        m = torch.where(step != 0, m, 0.0)
        h0 = m.square().sum()
        c0, g = grad(q)
        m = m - 0.5 * step * 0.5 * g
        for k in range(case["leapfrog"]):
            q = q + step * m
            c1, g = grad(q)
            m = m - (1.0 if k + 1 < case["leapfrog"] else 0.5) * step * 0.5 * g
        take = d.u[0] < math.exp(min(0.0, 0.5 * float(c0 - c1 + h0 - m.square().sum())))
        return {"state": q if take else d.params, "chi2": np.array([c1 if take else c0]), "accepted": None}
    if kind == "deflect":
        return _alpha(_t(d.params), d.grid)
    if kind == "nfw":
        return _nfw(_t(d.params), d.grid)
    if kind == "sie_mixed":
        ax, ay = _alpha(_t(d.params), d.grid)
        return {"ax": ax, "ay": ay, "mask": None, "stats": None}
    cot = [c.to(F64) for c in prepare(case, seed).cot] if case["prec"] == "fp64" else None
    if cot is None:
        return None
    X = (d.grid.x0 + torch.arange(d.grid.nx, dtype=F64, device=DEV) * d.grid.h)[None, :]
    Y = (d.grid.y0 + torch.arange(d.grid.ny, dtype=F64, device=DEV) * d.grid.h)[:, None]
    ax, ay = _alpha(_t(d.params), d.grid)
    grads = []
    for q in d.params.T:
        q = _t(q).requires_grad_(True)
        tx, ty = _alpha_one(list(q.unbind()), X, Y)
        grads.append(torch.autograd.grad((cot[0] * tx + cot[1] * ty).sum(), q)[0])
    return {"ax": ax, "ay": ay, "grad": torch.stack(grads, 1)}
