"""The work that this package is used for, as cases that can be timed.

Every case goes through the public entry points of `paper_1204_6367_amd.api`
as a simulation program calls them.  Sizes are those of the package's own
workloads (64^3 sphere, 128x128x96 adjoint phantom, 256x256x160 pelvis,
512x512x256 pelvis; 64x48, 256x192 and 512x384 detectors; 60/120/360 angles)
and odd ones between them.  Inputs are made on the GPU from the seed: ellipsoid
phantoms over air with 5 % density texture per voxel, the 120 kVp spectrum
behind a bowtie or a 60 keV line, Poisson scatter images.

Kinds of case:
  majorant   Woodcock majorant of one volume
  project    one Monte Carlo projection of one volume
  batch      several phantoms and angles in one persistent launch
  adjoint    differentiable projection: forward and d(loss)/d(density)
  primary    ray-traced primary of one or many angles (Eq. 1)
  denoise    Poisson denoising of a stack of scatter images (Eq. 5)
  noise      noise assembly of a stack of images (Sec. 2.6)
  scan       a whole simulated scan: MC batch, primary, denoising, noise
"""
import functools
import math

import numpy as np
import torch

from paper_1204_6367_amd import api
from paper_1204_6367_amd import workloads as W

MATERIALS = W.ELLIPSOID_MATERIALS
EXTENT_MM = (500.0, 500.0, 400.0)          # a pelvis-sized field of view
BODY_MM = (0.42, 0.30, 0.45)               # body semi-axes over the extents
MARGIN = 2.0 ** -20
ADJ_MARGIN, ADJ_RHO_MIN = 0.1, 0.05        # the bounds of a differentiable run
CUBE_MM = 40.0                             # edge of the local majorants' cubes
TUNED = dict(block=1024, defer=8, coll_defer=12, chunk=512)   # the shape the package's autotuner ships for its batch


def listed():
    return [
        # a majorant table on its own, for a small phantom: the smallest call, launches and latency
        dict(name="majorant_64", kind="majorant", nx=64, ny=64, nz=64, interp=True),
        # a quick look at one small projection: 60 keV line, 64x48 pixels, interactive use and tests
        dict(name="project_small", kind="project", nx=64, ny=64, nz=64, nu=64, nv=48, photons=100_000, poly=False,
             joint=False, local=False, sumsq=True, interp=True),
        # one projection as `project` gives it by default (single majorant, variance planes)
        dict(name="project_pelvis", kind="project", nx=256, ny=256, nz=160, nu=256, nv=192, photons=10_000_000,
             poly=True, joint=False, local=False, sumsq=True, interp=True),
        # the paper's projection: 1e8 photons, here with local majorants
        dict(name="project_pelvis_local", kind="project", nx=256, ny=256, nz=160, nu=256, nv=192,
             photons=100_000_000, poly=True, joint=False, local=True, sumsq=False, interp=True),
        # three phantoms at many angles in one launch, tuned launch shape: production of projection sets
        dict(name="batch_three", kind="batch", volumes=3, angles=24, photons=10_000_000, tuned=True, joint=False,
             local=True, sumsq=False),
        # one iteration of a density fit: forward tallies, loss, gradient (128x128x96)
        dict(name="adjoint_fit", kind="adjoint", nx=128, ny=128, nz=96, nu=256, nv=192, angles=4, photons=1_000_000,
             local=True),
        # the ray-traced primary of a single view of a mid-sized phantom
        dict(name="primary_one", kind="primary", nx=256, ny=256, nz=160, nu=256, nv=192, angles=1, interp=True),
        # the primaries of a 60-view scan of the largest phantom
        dict(name="primary_scan", kind="primary", nx=512, ny=512, nz=256, nu=256, nv=192, angles=60, interp=True),
        # one full-resolution scatter image (512x384), as after a single projection
        dict(name="denoise_one", kind="denoise", images=1, nu=512, nv=384, iters=256),
        # the scatter images of a 360-view scan
        dict(name="denoise_scan", kind="denoise", images=360, nu=256, nv=192, iters=256),
        # noise of a 360-view scan at a given mAs: one streaming pass
        dict(name="noise_scan", kind="noise", images=360, nu=256, nv=192),
        # a whole short scan, all four steps, with odd sizes
        dict(name="scan_short", kind="scan", nx=150, ny=130, nz=75, nu=200, nv=150, angles=40, photons=250_000,
             local=True, iters=100),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["majorant", "project", "project", "batch", "adjoint", "primary", "primary", "denoise",
                       "denoise", "noise", "scan"])
    nx = _log_int(rng, 32, 512)
    ny = max(24, min(512, int(nx * rng.uniform(0.7, 1.2))))
    nz = max(16, min(256, int(nx * rng.uniform(0.4, 0.8))))
    nu = _log_int(rng, 48, 512)
    nv = max(32, int(nu * rng.uniform(0.5, 1.0)))
    vol = dict(nx=nx, ny=ny, nz=nz)
    det = dict(nu=nu, nv=nv)
    if kind == "majorant":
        return dict(kind=kind, **vol, interp=rng.random() < 0.8)
    if kind == "project":
        local = rng.random() < 0.5
        joint = rng.random() < 0.2
        return dict(kind=kind, **vol, **det, photons=_log_int(rng, 30_000, 100_000_000 if local else 30_000_000),
                    poly=joint or rng.random() < 0.8, joint=joint, local=local, sumsq=rng.random() < 0.5,
                    interp=rng.random() < 0.9)
    if kind == "batch":
        angles = _log_int(rng, 3, 60)
        return dict(kind=kind, volumes=rng.choice([1, 2, 3]), angles=angles,
                    photons=_log_int(rng, 50_000, max(100_000, 200_000_000 // angles)), tuned=rng.random() < 0.5,
                    joint=rng.random() < 0.2, local=rng.random() < 0.8, sumsq=rng.random() < 0.3)
    if kind == "adjoint":
        vol = {k: min(v, 256) for k, v in vol.items()}
        return dict(kind=kind, **vol, **det, angles=rng.choice([1, 2, 4, 8]),
                    photons=_log_int(rng, 100_000, 5_000_000), local=rng.random() < 0.7)
    if kind == "primary":
        pixels = 60 * 256 * 192
        return dict(kind=kind, **vol, **det, angles=_log_int(rng, 1, max(2, min(360, pixels // (nu * nv)))),
                    interp=rng.random() < 0.8)
    if kind == "denoise":
        return dict(kind=kind, images=_log_int(rng, 1, max(2, min(360, 360 * 256 * 192 // (nu * nv)))), **det,
                    iters=_log_int(rng, 16, 256))
    if kind == "noise":
        return dict(kind=kind, images=_log_int(rng, 1, max(2, min(720, 720 * 256 * 192 // (nu * nv)))), **det)
    return dict(kind=kind, **{k: min(v, 256) for k, v in vol.items()}, **det, angles=_log_int(rng, 4, 60),
                photons=_log_int(rng, 20_000, 1_000_000), local=rng.random() < 0.8, iters=_log_int(rng, 50, 200))


# --- inputs -------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _mu_table():
    return W.cross_section_table(MATERIALS)


@functools.lru_cache(maxsize=32)
def _source_arrays(nu, nv, du, dv, poly, joint):
    geom = W.Geometry(nu=nu, nv=nv, du_mm=du, dv_mm=dv)
    if not poly:
        e, p = W.mono_spectrum(60.0)
        return W.Source(e, p, W.fluence_map(geom))
    return W.pelvis_source(geom, joint=joint)


def _generator(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _phantom(nx, ny, nz, seed, salt=0, extent=EXTENT_MM):
    """Density and material [nz][ny][nx] on the GPU: a soft-tissue body ellipsoid
    with eleven bone, lung and soft-tissue ellipsoids, +-5 % density per voxel."""
    rng = np.random.Generator(np.random.PCG64([int(seed), salt]))
    sp = np.array([extent[0] / nx, extent[1] / ny, extent[2] / nz])
    ax = [torch.as_tensor((np.arange(n) + 0.5 - n / 2.0) * d, dtype=torch.float32, device="cuda")
          for n, d in zip((nx, ny, nz), sp)]
    z, y, x = ax[2][:, None, None], ax[1][None, :, None], ax[0][None, None, :]
    body = np.array(BODY_MM) * np.array(extent)
    scale = min(extent) / 400.0
    mat = torch.zeros((nz, ny, nx), dtype=torch.uint8, device="cuda")
    ells = [(np.zeros(3), body, np.eye(3), 1)]
    for _ in range(11):
        p = rng.uniform(-1.0, 1.0, 3)
        p /= max(1.0, np.linalg.norm(p))
        q, r = np.linalg.qr(rng.standard_normal((3, 3)))
        ells.append((0.7 * body * p, rng.uniform(10.0, 60.0, 3) * scale, q * np.sign(np.diag(r))[None, :],
                     int(rng.choice([2, 3, 1], p=[0.45, 0.20, 0.35]))))
    for c, axes, rot, m in ells:
        d2 = 0.0
        for k in range(3):
            v = [float(rot[i, k] / axes[k]) for i in range(3)]
            d2 = d2 + ((x - float(c[0])) * v[0] + (y - float(c[1])) * v[1] + (z - float(c[2])) * v[2]) ** 2
        mat[d2 <= 1.0] = m
    rho = torch.tensor([W.MATERIALS[n].density for n in MATERIALS], dtype=torch.float32, device="cuda")
    tex = torch.rand(mat.shape, generator=_generator(seed, 17 + salt), device="cuda")
    return rho[mat.long()] * (0.95 + 0.1 * tex), mat, tuple(float(s) for s in sp)


def _volume(nx, ny, nz, seed, salt=0, local=False, adjoint=False):
    dens, mat, sp = _phantom(nx, ny, nz, seed, salt)
    v = api.DeviceVolume(dens, mat, sp)
    if local:
        v.local_majorants(max(1, int(round(CUBE_MM / min(sp)))), ADJ_MARGIN if adjoint else MARGIN,
                          ADJ_RHO_MIN if adjoint else 0.0)
    return v


def _physics():
    g = W.EnergyGrid()
    return api.DevicePhysics(_mu_table(), g.e0_kev, g.de_kev)


def _detector(nu, nv):
    """Pixel pitch that covers the 397 x 298 mm panel of the 256x192 detector."""
    return 256 * 1.552 / nu, 192 * 1.552 / nv


def _geom(nu, nv, phi=0.0):
    du, dv = _detector(nu, nv)
    return W.Geometry(nu=nu, nv=nv, du_mm=du, dv_mm=dv, phi_rad=phi)


def _source(nu, nv, poly=True, joint=False):
    du, dv = _detector(nu, nv)
    s = _source_arrays(nu, nv, du, dv, poly, joint)
    return api.DeviceSource(s.spec_e, s.spec_p, s.fluence)


def _angle(seed, k, n):
    return 2.0 * math.pi * (k + (int(seed) % 97) / 97.0) / n


def _scatter_images(images, nv, nu, seed):
    """Poisson counts over a smooth scatter field, as an MC tally leaves them."""
    g = _generator(seed, 5)
    v = torch.linspace(-1.0, 1.0, nv, device="cuda", dtype=torch.float32)[None, :, None]
    u = torch.linspace(-1.0, 1.0, nu, device="cuda", dtype=torch.float32)[None, None, :]
    c = 0.6 * torch.rand((images, 1, 1), generator=g, device="cuda") - 0.3
    lam = 60.0 * torch.exp(-((u - c) ** 2) - 0.7 * v ** 2) + 20.0
    return torch.poisson(lam, generator=g).to(torch.float64)


def prepare(case, seed):
    c, kind = dict(case), case["kind"]
    s = dict(case=c, seed=int(seed))
    if kind == "majorant":
        s.update(vol=_volume(c["nx"], c["ny"], c["nz"], seed), phys=_physics())
    elif kind == "project":
        s.update(vol=_volume(c["nx"], c["ny"], c["nz"], seed, local=c["local"]), phys=_physics(),
                 src=_source(c["nu"], c["nv"], c["poly"], c["joint"]), geom=_geom(c["nu"], c["nv"], _angle(seed, 0, 1)))
    elif kind == "batch":
        shapes = [(512, 512, 256), (256, 256, 160), (128, 128, 64)][-c["volumes"]:]
        vols = [_volume(*sh, seed, salt=k, local=c["local"]) for k, sh in enumerate(shapes)]
        jobs, weights = [], [1.0, 0.3, 0.1][-c["volumes"]:]
        per = [max(1, round(c["angles"] * w)) for w in [1 / 6, 1 / 3, 1 / 2][-c["volumes"]:]]
        for k, n in enumerate(per):
            for a in range(n):
                jobs.append(api.JobSpec(_geom(256, 192, _angle(seed, a, n)),
                                        max(1000, int(c["photons"] * weights[k] / weights[0])), len(jobs), volume=k))
        batch = api.Batch(vols, _physics(), [_source(256, 192, True, c["joint"])], jobs)
        s.update(batch=batch, out=torch.zeros(batch.tally_elems, dtype=torch.float64, device="cuda"),
                 tune=TUNED if c["tuned"] else None)
    elif kind == "adjoint":
        vol = _volume(c["nx"], c["ny"], c["nz"], seed, local=c["local"], adjoint=True)
        n = c["angles"]
        jobs = [api.JobSpec(_geom(c["nu"], c["nv"], _angle(seed, a, n)), c["photons"], a) for a in range(n)]
        batch = api.Batch([vol], _physics(), [_source(c["nu"], c["nv"])], jobs)
        tex = torch.rand(vol.shape, generator=_generator(seed, 29), device="cuda")
        target = vol.density * (0.95 + 0.1 * tex)
        with torch.no_grad():
            goal = api.GdrrProject.apply(target, batch, int(seed) + 1, True, ADJ_MARGIN)[:, 1].clone()
        s.update(batch=batch, density=vol.density.clone(), goal=goal)
    elif kind == "primary":
        vol = _volume(c["nx"], c["ny"], c["nz"], seed)
        n = c["angles"]
        jobs = [api.JobSpec(_geom(c["nu"], c["nv"], _angle(seed, a, n)), 0, a) for a in range(n)]
        s.update(batch=api.Batch([vol], _physics(), [_source(c["nu"], c["nv"])], jobs),
                 out=torch.zeros(n * c["nu"] * c["nv"], dtype=torch.float64, device="cuda"))
    elif kind == "denoise":
        s.update(shat=_scatter_images(c["images"], c["nv"], c["nu"], seed))
    elif kind == "noise":
        n, nv, nu = c["images"], c["nv"], c["nu"]
        g = _generator(seed, 7)
        s.update(tally=torch.rand((n, 4, nv, nu), generator=g, device="cuda", dtype=torch.float64),
                 p=torch.rand((n, nv, nu), generator=g, device="cuda", dtype=torch.float64),
                 sc=torch.rand((n, nv, nu), generator=g, device="cuda", dtype=torch.float64),
                 alpha=api.noise_scale(5.0e8, 5.2913e9, 0.4 + 0.01 * (int(seed) % 50)))
    elif kind == "scan":
        vol = _volume(c["nx"], c["ny"], c["nz"], seed, local=c["local"])
        n = c["angles"]
        jobs = [api.JobSpec(_geom(c["nu"], c["nv"], _angle(seed, a, n)), c["photons"], a) for a in range(n)]
        batch = api.Batch([vol], _physics(), [_source(c["nu"], c["nv"])], jobs)
        s.update(batch=batch, tallies=torch.zeros(batch.tally_elems, dtype=torch.float64, device="cuda"),
                 prim=torch.zeros(n * c["nu"] * c["nv"], dtype=torch.float64, device="cuda"),
                 alpha=api.noise_scale(c["photons"], 5.2913e9, 0.4))
    return s


def run(s):
    c, kind, seed = s["case"], s["case"]["kind"], s["seed"]
    if kind == "majorant":
        return api.majorant(s["vol"], s["phys"], interp=c["interp"])
    if kind == "project":
        return api.project(s["vol"], s["phys"], s["src"], s["geom"], c["photons"], seed=seed, interp=c["interp"],
                           sumsq=c["sumsq"])
    if kind == "batch":
        return s["batch"].project(seed=seed, sumsq=c["sumsq"], tune=s["tune"], out=s["out"])
    if kind == "adjoint":
        x = s["density"].detach().requires_grad_(True)
        ps = api.GdrrProject.apply(x, s["batch"], seed, True, ADJ_MARGIN)
        loss = 0.5 * ((ps[:, 1] - s["goal"]) ** 2).sum() * (c["nu"] * c["nv"]) ** 2
        (grad,) = torch.autograd.grad(loss, x)
        return {"tallies": ps.detach(), "grad": grad}
    if kind == "primary":
        s["batch"].primary(interp=c["interp"], out=s["out"])
        return s["out"].view(c["angles"], c["nv"], c["nu"])
    if kind == "denoise":
        return api.denoise(s["shat"], beta=0.05, iters=c["iters"], s_floor=1e-3)
    if kind == "noise":
        noise, image = api.noise(s["tally"][:, 0], s["p"], s["tally"][:, 2], s["sc"], s["alpha"])
        return {"noise": noise, "image": image}
    n, nv, nu = c["angles"], c["nv"], c["nu"]
    t = s["batch"].project(seed=seed, sumsq=False, out=s["tallies"]).view(n, 4, nv, nu)
    s["batch"].primary(out=s["prim"])
    prim = s["prim"].view(n, nv, nu)
    mean = 2.0 / (nu * nv)                       # keV of scatter per pixel and source photon, about
    smooth = api.denoise(t[:, 2], beta=4.0 / mean, iters=c["iters"], s_floor=1e-3 * mean)
    noise, image = api.noise(t[:, 0], prim, t[:, 2], smooth, s["alpha"])
    return {"tallies": t, "primary": prim, "scatter": smooth, "noise": noise, "image": image}


# --- what a pass cannot do without ---------------------------------------------
# Operations of one photon history (int and float32 alike): two source blocks and
# the source sample, six Philox blocks of flight pairs, about seven free flights,
# 2.5 collisions with three sampler tries.
OPS_HISTORY = 1200.0


def _image_bytes(c):
    return 8.0 * c["nu"] * c["nv"]


def work(case):
    c, kind = case, case["kind"]
    if kind == "batch":
        sh = [(512, 512, 256), (256, 256, 160), (128, 128, 64)][-c["volumes"]:]
        w = [1.0, 0.3, 0.1][-c["volumes"]:]
        per = [max(1, round(c["angles"] * x)) for x in [1 / 6, 1 / 3, 1 / 2][-c["volumes"]:]]
        hist = sum(n * c["photons"] * x / w[0] for n, x in zip(per, w))
        return dict(bytes=5.0 * sum(a * b * d for a, b, d in sh) + sum(per) * (4.0 if c["sumsq"] else 2.0) * 8 * 256 * 192,
                    flops=OPS_HISTORY * hist)
    if kind in ("denoise", "noise"):
        px = float(c["images"] * c["nu"] * c["nv"])
        if kind == "noise":
            return dict(bytes=48.0 * px, flops=7.0 * px)
        return dict(bytes=16.0 * px, flops=13.0 * c["iters"] * px)
    voxels = float(c["nx"]) * c["ny"] * c["nz"]
    if kind == "majorant":
        return dict(bytes=5.0 * voxels + 4 * 298, flops=(26.0 if c["interp"] else 1.0) * voxels)
    if kind == "project":
        return dict(bytes=5.0 * voxels + (4.0 if c["sumsq"] else 2.0) * _image_bytes(c),
                    flops=OPS_HISTORY * c["photons"])
    if kind == "adjoint":
        return dict(bytes=17.0 * voxels + 4.0 * _image_bytes(c) * c["angles"],
                    flops=3.0 * OPS_HISTORY * c["photons"] * c["angles"])
    rays = float(c["angles"]) * c["nu"] * c["nv"]
    steps = 300.0 / (0.5 * min(EXTENT_MM[0] / c["nx"], EXTENT_MM[1] / c["ny"], EXTENT_MM[2] / c["nz"]))
    march = rays * (steps * 46.0 + 119 * 10.0)
    if kind == "primary":
        return dict(bytes=5.0 * voxels + 8.0 * rays, flops=march)
    return dict(bytes=5.0 * voxels + 32.0 * rays, flops=march + rays * (13.0 * c["iters"] + 7.0) +
                OPS_HISTORY * c["photons"] * c["angles"])


# --- values in 64 bits -----------------------------------------------------------
def _f32(x):
    return float(np.float32(x))


def _exact_majorant(s):
    c, vol = s["case"], s["vol"]
    rho = vol.density.double()
    if c["interp"]:
        rho = torch.nn.functional.max_pool3d(rho[None, None], 3, stride=1, padding=1)[0, 0]
    mu = s["phys"].mu.double().sum(-1)                         # [n_mat][n_e]
    hi = torch.maximum(mu[:, :-1], mu[:, 1:])
    best = torch.zeros_like(hi[0])
    for m in range(mu.shape[0]):
        sel = vol.material == m
        if bool(sel.any()):
            best = torch.maximum(best, rho[sel].max() * hi[m])
    return best * (1.0 + MARGIN)


def _exact_primary(batch, interp):
    """Eq. 1 marched in 64 bits, all the rays of the jobs side by side."""
    vol, phys, src = batch.vols[0], batch.phys, batch.srcs[0]
    dev = vol.density.device
    nz, ny, nx = vol.shape
    d = [_f32(v) for v in vol.spacing_mm]
    n = (nx, ny, nz)
    dl = 0.5 * min(d)
    flat_r, flat_m = vol.density.reshape(-1), vol.material.reshape(-1)
    starts, dirs = [], []
    for j in batch.jobs:
        g = j.geom
        phi, th = _f32(g.phi_rad), _f32(g.theta_rad)
        q = phi + th
        S = (-_f32(g.sad_mm) * math.cos(phi), -_f32(g.sad_mm) * math.sin(phi), 0.0)
        u = (torch.arange(g.nu, device=dev, dtype=torch.float64) + 0.5 - 0.5 * g.nu) * _f32(g.du_mm)
        v = (torch.arange(g.nv, device=dev, dtype=torch.float64) + 0.5 - 0.5 * g.nv) * _f32(g.dv_mm)
        aid = _f32(g.aid_mm)
        x = (aid * math.cos(q) - math.sin(q) * u - S[0])[None, :].expand(g.nv, g.nu)
        y = (aid * math.sin(q) + math.cos(q) * u - S[1])[None, :].expand(g.nv, g.nu)
        dirs.append(torch.stack([x, y, v[:, None].expand(g.nv, g.nu)]).reshape(3, -1))
        starts.append(torch.tensor(S, device=dev, dtype=torch.float64)[:, None].expand(3, g.nu * g.nv))
    D, S = torch.cat(dirs, 1), torch.cat(starts, 1)
    length = D.square().sum(0).sqrt()
    D = D / length
    t0, t1 = torch.zeros_like(length), length.clone()
    for a in range(3):
        h = 0.5 * n[a] * d[a]
        ta, tb = (-h - S[a]) / D[a], (h - S[a]) / D[a]
        inside = (S[a].abs() <= h) if a == 2 else torch.zeros_like(length, dtype=torch.bool)
        flat = D[a] == 0
        t0 = torch.maximum(t0, torch.where(flat, torch.where(inside, t0, t1 + 1), torch.minimum(ta, tb)))
        t1 = torch.minimum(t1, torch.where(flat, t1, torch.maximum(ta, tb)))
    hit = t0 < t1
    n_mat = phys.mu.shape[0]
    L = torch.zeros((n_mat, D.shape[1]), dtype=torch.float64, device=dev)
    if bool(hit.any()):
        for j in range(int(t0[hit].min() / dl), int(t1[hit].max() / dl) + 1):
            a = torch.clamp(t0, min=j * dl)
            e = torch.clamp(t1, max=(j + 1) * dl)
            h = torch.where(hit, (e - a).clamp(min=0.0), 0.0)
            t = 0.5 * (a + e)
            lo, fr = [], []
            for k in range(3):
                gk = (S[k] + t * D[k]) / d[k] + 0.5 * n[k] - 0.5
                fl = torch.floor(gk)
                lo.append(fl.clamp(-1, n[k] - 1).long())
                fr.append((gk - fl).clamp(0.0, 1.0))
            if not interp:
                vx = [torch.clamp(lo[k] + (fr[k] >= 0.5).long(), 0, n[k] - 1) for k in range(3)]
                at = (vx[2] * ny + vx[1]) * nx + vx[0]
                L.scatter_add_(0, flat_m[at].long()[None], (h * flat_r[at])[None])
                continue
            for corner in range(8):
                w, at = h, 0
                for k in (2, 1, 0):
                    up = (corner >> k) & 1
                    w = w * (fr[k] if up else 1.0 - fr[k])
                    at = at * n[k] + torch.clamp(lo[k] + up, 0, n[k] - 1)
                L.scatter_add_(0, flat_m[at].long()[None], (w * flat_r[at])[None])
    e0, de = _f32(phys.e0), _f32(phys.de)
    mu = phys.mu.double().sum(-1)
    E, w = src.spec_e.double(), src.spec_p.double()
    if w.dim() == 2:
        return None
    gE = (E - e0) / de
    jE = torch.floor(gE).long().clamp(0, mu.shape[1] - 2)
    tab = mu[:, jE] + (gE - jE) * (mu[:, jE + 1] - mu[:, jE])       # [n_mat][n_spec]
    out = torch.zeros_like(length)
    for k in range(E.shape[0]):
        out += w[k] / w.sum() * E[k] * torch.exp(-0.1 * (tab[:, k, None] * L).sum(0))
    flu = src.fluence.double()
    nv, nu = flu.shape
    return out.view(-1, nv, nu) * (flu / flu.sum())


def _exact_denoise(shat, beta, iters, s_floor, omega=0.8):
    s = shat.clamp(min=s_floor)
    for _ in range(iters):
        up = torch.cat([s[:, :1], s[:, :-1]], 1)
        dn = torch.cat([s[:, 1:], s[:, -1:]], 1)
        lf = torch.cat([s[:, :, :1], s[:, :, :-1]], 2)
        rt = torch.cat([s[:, :, 1:], s[:, :, -1:]], 2)
        data = torch.where(shat == 0.0, torch.ones_like(s), 1.0 - shat / s)
        s = ((1.0 - omega) * s + 0.25 * omega * (up + dn + lf + rt - data / beta)).clamp(min=s_floor)
    return s


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("project", "batch"):
        return None                              # a Monte Carlo estimate: no value of its own
    s = prepare(case, seed)
    if kind == "majorant":
        return _exact_majorant(s)
    if kind == "primary":
        return _exact_primary(s["batch"], c["interp"])
    if kind == "denoise":
        return _exact_denoise(s["shat"], 0.05, c["iters"], _f32(1e-3))
    if kind == "noise":
        t = s["tally"]
        noise = s["alpha"] * ((t[:, 0] - s["p"]) + (t[:, 2] - s["sc"]))
        return {"noise": noise, "image": s["p"] + s["sc"] + noise}
    if kind == "scan":
        return {"tallies": None, "primary": _exact_primary(s["batch"], True), "scatter": None, "noise": None,
                "image": None}
    return None
