"""Performance cases of the reconstruction library, through its public Python
entry points: single projections, gradients and objectives, iterations of a
running reconstruction, and whole calls, in 2D and fully 3D.

A case names a kind of call and its sizes; prepare() makes the buffers and
handles that a program holds before the call, run() makes one pass, and
exact() gives the same outputs in FP64 with plain torch (an independent
Siddon walk: every cut of a ray is evaluated at the middle of its pieces).

The data are simulated from random ellipses (ellipsoids): analytic line
integrals scaled to a count level, a uniform background, Poisson noise.  The
image is the phantom with voxel noise over a low floor, as an iterate in the
middle of a reconstruction looks.  Steps of an iteration are of a size at which
the method contracts (a late position k, or a small lambda0), so that the
outputs do not amplify the rounding of single sums.
"""
import math
import random

import torch

import paper_2111_07886_amd as pet

DEV = "cuda"
FOV_MM = 300.0
DET_RADIUS_MM = 576 * 4.0 / (2 * math.pi)      # 576 detectors of 4 mm
SUBRAYS, PSF_MM, MU_WATER = 32, 6.59, 0.0096   # the paper's full 2D model


def _case(name, kind, nx, ny=None, nz=1, angles=60, radial=None, rd=0, subsets=4, **more):
    ny = nx if ny is None else ny
    radial = 2 * math.ceil(max(nx, ny) / math.sqrt(2)) + 3 if radial is None else radial
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, angles=angles, radial=radial, rd=rd, subsets=subsets, **more)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a whole forward projection of the smallest image: launch and latency
        _case("forward2d_64", "forward", 64, angles=60, radial=95, subset=0),
        # one subset's back-projection of a ragged image (a program's own loop)
        _case("back2d_177x161", "back", 177, 161, angles=203, radial=255, subsets=9, subset=3),
        # one iteration of a running 2D reconstruction: 24 subiterations
        _case("iterate2d_256", "iterate", 256, angles=288, radial=367, subsets=24, mode="P2", k0=40),
        # the same with the paper's full system model (sub-rays, PSF, attenuation)
        _case("iterate2d_full_256", "iterate", 256, angles=288, radial=367, subsets=24, mode="P2", k0=40, full=True),
        # OSEM initialisation of a larger 2D image, one iteration
        _case("osem2d_320", "iterate", 320, angles=360, radial=457, subsets=16, mode="OSEM", k0=0),
        # uneven 2D requests reconstructed together in one call
        _case("batch2d_24", "batch", 320, angles=360, subsets=32, count=24, mix=14, iters=2),
        # a subset's forward projection, fully 3D
        _case("forward3d_128x32", "forward", 128, nz=32, angles=180, radial=185, rd=7, subsets=20, subset=4),
        # a subset's back-projection, ragged 3D
        _case("back3d_127x125x29", "back", 127, 125, nz=29, angles=175, radial=181, rd=9, subsets=18, subset=2),
        # the subset gradient (gradient-consistency study, a program's own optimiser)
        _case("gradient3d_200x64", "gradient", 200, nz=64, angles=224, radial=281, rd=15, subsets=28, subset=5),
        # the objective over every ray
        _case("objective3d_200x64", "objective", 200, nz=64, angles=224, radial=281, rd=15, subsets=28),
        # a whole short reconstruction call with its own scratch and data check
        _case("reconstruct3d_128x32", "reconstruct", 128, nz=32, angles=180, radial=185, rd=7, subsets=20,
              mode="P2", iters=2),
        # one iteration of a running fully 3D reconstruction: 28 subiterations
        _case("iterate3d_200x64", "iterate", 200, nz=64, angles=224, radial=281, rd=15, subsets=28, mode="P2", k0=20),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["forward", "back", "gradient", "objective", "iterate", "iterate", "reconstruct", "batch"])
    if kind == "batch":
        return _case(None, "batch", 320, angles=360, subsets=32, count=rng.randint(2, 24), mix=rng.randint(0, 10 ** 6),
                     iters=rng.randint(1, 2))
    if rng.random() < 0.5:
        nx = log_int(48, 320)
        ny = nx if rng.random() < 0.5 else max(32, nx - rng.randint(1, 24))
        angles, subsets = rng.randint(60, 360), rng.randint(4, 32)
        c = dict(nx=nx, ny=ny, angles=angles, subsets=subsets)
    else:
        nx = log_int(40, 176)
        ny = nx if rng.random() < 0.5 else max(32, nx - rng.randint(1, 16))
        nz = log_int(8, 64)
        angles, subsets = rng.randint(60, 200), rng.randint(8, 28)
        c = dict(nx=nx, ny=ny, nz=nz, angles=angles, subsets=subsets, rd=rng.randint(1, min(15, nz - 1)))
    c["radial"] = 2 * math.ceil(max(c["nx"], c["ny"]) / math.sqrt(2)) + rng.randint(2, 5)
    if kind in ("forward", "back", "gradient"):
        c["subset"] = 0 if rng.random() < 0.25 else rng.randint(1, subsets)
    if kind == "iterate":
        c["mode"] = rng.choice(["P2", "P2", "P1", "BSREM", "OSEM"])
        c["k0"] = 0 if c["mode"] == "OSEM" else rng.randint(20, 60)
        if "nz" not in c and rng.random() < 0.25:
            c["full"] = True
    if kind == "reconstruct":
        c["mode"] = rng.choice(["P2", "M2", "BSREM"])
        c["iters"] = rng.randint(1, 2)
    return _case(None, kind, **c)


# ------------------------------------------------------------------ inputs

def _desc(c):
    v = FOV_MM / max(c["nx"], c["ny"])
    d3 = c["nz"] > 1
    d = dict(dim=3 if d3 else 2, nx=c["nx"], ny=c["ny"], nz=c["nz"], vx=v, vy=v, vz=3.0 if d3 else 1.0,
             n_angles=c["angles"], n_radial=c["radial"], ds=v, n_rings=c["nz"], max_ring_diff=c["rd"],
             ring_pitch=3.0 if d3 else 1.0, det_radius=DET_RADIUS_MM, n_subsets=c["subsets"])
    if c.get("full"):
        d.update(n_subrays=SUBRAYS, psf_fwhm=PSF_MM)
    return d


def _requests(c):
    """The single-request cases of a batch: uneven sizes from its mix number."""
    rng = random.Random(c["mix"])
    out = []
    for _ in range(c["count"]):
        n = rng.choice(range(64, c["nx"] + 1, 16))
        M = rng.randint(4, c["subsets"])
        Na = max(2 * M, rng.randint(60, c["angles"]) // M * M)
        out.append(_case(None, "reconstruct", n, angles=Na, subsets=M, mode="P2", iters=c["iters"]))
    return out


def _angles(c):
    th = [a * math.pi / c["angles"] for a in range(c["angles"])]
    cs = [math.cos(t) for t in th]
    sn = [math.sin(t) for t in th]
    cs[0], sn[0] = 1.0, 0.0
    if c["angles"] % 2 == 0:
        cs[c["angles"] // 2], sn[c["angles"] // 2] = 0.0, 1.0
    return cs, sn


def _planes(c):
    """(first ring, ring difference) of every plane, in span-1 order."""
    out = []
    for d in [0] + [s * k for k in range(1, c["rd"] + 1) for s in (1, -1)]:
        out += [(r1, d) for r1 in range(max(0, -d), min(c["nz"], c["nz"] - d))]
    return out


def _ellipsoids(c, seed):
    rng = random.Random(seed)
    R, hz = 0.5 * FOV_MM * min(c["nx"], c["ny"]) / max(c["nx"], c["ny"]), 1.5 * c["nz"]
    out = [(0.0, 0.0, 0.0, 0.8 * R, 0.62 * R, 0.9 * hz, rng.uniform(0.0, math.pi), 1.0)]
    for _ in range(6):
        rad, ang = 0.45 * R * math.sqrt(rng.random()), rng.uniform(0, 2 * math.pi)
        out.append((rad * math.cos(ang), rad * math.sin(ang), rng.uniform(-0.5, 0.5) * hz, rng.uniform(0.06, 0.3) * R,
                    rng.uniform(0.06, 0.3) * R, rng.uniform(0.2, 0.5) * hz, rng.uniform(0.0, math.pi),
                    rng.uniform(0.5, 4.0)))
    return out


def _sinogram(c, ells):
    """Line integrals [plane][angle][bin] of the ellipsoids (2D: ellipses), FP32."""
    v = FOV_MM / max(c["nx"], c["ny"])
    cs, sn = (torch.tensor(x, dtype=torch.float32, device=DEV)[:, None] for x in _angles(c))
    sb = (torch.arange(c["radial"], device=DEV, dtype=torch.float32) - 0.5 * (c["radial"] - 1))[None, :] * v
    d3 = c["nz"] > 1
    if d3:
        h = torch.sqrt(DET_RADIUS_MM ** 2 - sb ** 2)[None]
        pl = torch.tensor(_planes(c), dtype=torch.float32, device=DEV)
        z1 = (pl[:, 0] - 0.5 * (c["nz"] - 1))[:, None, None] * 3.0
        mz = (pl[:, 1] * 3.0)[:, None, None] / (2 * h)
        zc = z1 + mz * h
        mz, zc = mz.expand(-1, c["angles"], -1), zc.expand(-1, c["angles"], -1)
    out = torch.zeros((len(_planes(c)) if d3 else 1, c["angles"], c["radial"]), dtype=torch.float32, device=DEV)
    for x0, y0, z0, A, B, C, phi, val in ells:
        cp, sp = math.cos(phi), math.sin(phi)
        ex = (sb * cs - x0) * cp + (sb * sn - y0) * sp
        ey = -(sb * cs - x0) * sp + (sb * sn - y0) * cp
        qx, qy = -sn * cp + cs * sp, sn * sp + cs * cp
        a = ((qx / A) ** 2 + (qy / B) ** 2).expand_as(ex)
        b = ex * qx / A ** 2 + ey * qy / B ** 2
        cc = (ex / A) ** 2 + (ey / B) ** 2 - 1.0
        if not d3:
            out[0] += (2 * val / a) * torch.sqrt((b * b - a * cc).clamp_min(0))
            continue
        for p in range(0, out.shape[0], 128):
            m, w = mz[p:p + 128], zc[p:p + 128] - z0
            aa = a + (m / C) ** 2
            bb = b + w * m / C ** 2
            q = bb * bb - aa * (cc + (w / C) ** 2)
            out[p:p + 128] += (2 * val / aa) * torch.sqrt(q.clamp_min(0) * (1 + m * m))
    return out


def _inputs(c, seed):
    """Image f, counts y, background r (and attenuation) of a single request."""
    ells = _ellipsoids(c, seed)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    d = _desc(c)
    x = (torch.arange(c["nx"], device=DEV) - 0.5 * (c["nx"] - 1)) * d["vx"]
    y = (torch.arange(c["ny"], device=DEV) - 0.5 * (c["ny"] - 1))[:, None] * d["vy"]
    z = (torch.arange(c["nz"], device=DEV) - 0.5 * (c["nz"] - 1))[:, None, None] * d["vz"]
    img = torch.zeros((c["nz"], c["ny"], c["nx"]), dtype=torch.float32, device=DEV)
    for x0, y0, z0, A, B, C, phi, val in ells:
        cp, sp = math.cos(phi), math.sin(phi)
        q = (((x - x0) * cp + (y - y0) * sp) / A) ** 2 + (((y - y0) * cp - (x - x0) * sp) / B) ** 2
        img += val * ((q + ((z - z0) / C) ** 2 if c["nz"] > 1 else q[None]) <= 1.0)
    sino = _sinogram(c, ells)
    att = None
    if c.get("full"):
        att = torch.exp(-MU_WATER * _sinogram(c, ells[:1]))
        sino = sino * att
    # counts per bin as in the workloads of the benchmark: 5e6 over 105,696
    # bins in 2D, 4.6 in 3D (5e8 over 109 million)
    scale = (47.0 if c["nz"] == 1 else 4.6) / 100.0
    img = img * scale
    f = (img * (1.0 + 0.1 * torch.randn(img.shape, generator=gen, device=DEV)) + 0.03 * scale).clamp_min(0.01 * scale)
    r = 0.2 * scale * 100.0 * (1.0 + 0.2 * torch.rand(sino.shape, generator=gen, device=DEV))
    yc = torch.poisson(sino * scale + r, generator=gen)
    return f.reshape(_img_shape(c)).contiguous(), yc, r, att


def _img_shape(c):
    return (c["nz"], c["ny"], c["nx"]) if c["nz"] > 1 else (c["ny"], c["nx"])


def _params(c):
    mode = c.get("mode", "P2")
    if mode == "OSEM":
        return pet.osem_params()
    U = 1e3 * 8.0
    p = dict(mode=mode, gamma_R=2.0, eps=1e-12, t_clip=1e-4, U=U, beta=0.1, J1=10 ** 6, objective_every=1)
    if c["nz"] > 1:
        p.update(lambda0=1.6, a=0.25, rho=2.2, delta1=0.1, delta2=1.6, nu1=0.6, nu2=1.25, J0=0)
    else:
        p.update(lambda0=1.0, a=0.45, rho=4.0, delta1=3.0, delta2=3.0, nu1=0.8, nu2=1.8, J0=3)
    if c["kind"] == "reconstruct":
        p["lambda0"] = 0.1
    return p


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    if case["kind"] == "batch":
        reqs = _requests(case)
        s = dict(kind="batch", geoms=[], params=[], f0=[], f=[], y=[], r=[], iters=[q["iters"] for q in reqs])
        for k, q in enumerate(reqs):
            f, y, r, _ = _inputs(q, seed * 1000 + k)
            s["geoms"].append(pet.Geometry(_desc(q)))
            s["params"].append(_params(q))
            s["f0"].append(f)
            s["f"].append(torch.empty_like(f))
            s["y"].append(y)
            s["r"].append(r)
        return s
    f, y, r, att = _inputs(case, seed)
    geom = pet.Geometry(_desc(case), att=None if att is None else att.cpu().numpy())
    s = dict(case, geom=geom, params=_params(case), f0=f)
    if case["kind"] == "forward":
        s["out"] = torch.zeros(geom.sino_shape, dtype=torch.float32, device=DEV)
        return s
    if case["kind"] == "back":
        s["w"] = (1.0 - y / (y.mean() + r)).contiguous()
        s["out"] = torch.empty_like(f)
        return s
    s.update(y=y, r=r, f=torch.empty_like(f))
    if case["kind"] == "iterate":
        s["state"] = pet.State(geom, s["params"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "forward":
        return s["geom"].forward(s["f0"], subset=s["subset"], out=s["out"])
    if kind == "back":
        return s["geom"].back(s["w"], subset=s["subset"], out=s["out"])
    if kind == "gradient":
        return s["geom"].subset_gradient(s["params"], s["f0"], s["y"], s["r"], s["subset"], out=s["f"])
    if kind == "objective":
        return s["geom"].objective(s["params"], s["f0"], s["y"], s["r"])
    if kind == "iterate":
        # one more iteration from the iterate in hand (put back for each pass)
        s["f"].copy_(s["f0"])
        s["state"].seek(s["k0"], 1)
        s["state"].run(s["f"], s["y"], s["r"], 1)
        return s["f"]
    if kind == "reconstruct":
        s["f"].copy_(s["f0"])
        pet.reconstruct(s["geom"], s["params"], s["f"], s["y"], s["r"], s["iters"])
        return s["f"]
    for f, f0 in zip(s["f"], s["f0"]):
        f.copy_(f0)
    pet.reconstruct_batch(s["geoms"], s["params"], s["f"], s["y"], s["r"], s["iters"])
    return s["f"]


# ------------------------------------------------------------------ the work

def _nnz(c, angles):
    """Number of nonzero matrix entries of the rays of these angles, from the
    chords of the rays through the image and the crossings per millimetre."""
    v = FOV_MM / max(c["nx"], c["ny"])
    hx, hy = 0.5 * c["nx"] * v, 0.5 * c["ny"] * v
    cs, sn = _angles(c)
    n_rays = sum(c["nz"] - abs(d) for d in range(-c["rd"], c["rd"] + 1)) if c["nz"] > 1 else 1
    climbs = sum((c["nz"] - abs(d)) * abs(d) for d in range(-c["rd"], c["rd"] + 1)) if c["nz"] > 1 else 0
    n = 0.0
    for a in angles:
        ca, sa = abs(cs[a]), abs(sn[a])
        eo, ei = hx * ca + hy * sa, abs(hx * ca - hy * sa)
        lmax = min(2 * hx / sa if sa else math.inf, 2 * hy / ca if ca else math.inf)
        for b in range((c["radial"] + 1) // 2):
            t = (0.5 * (c["radial"] - 1) - b) * v
            mult = 1 if 2 * b == c["radial"] - 1 else 2
            if t >= eo:
                continue
            chord = lmax * min(1.0, (eo - t) / (eo - ei)) if eo > ei else lmax
            n += mult * (n_rays * (chord * (ca + sa) / v) + climbs * chord / (2 * DET_RADIUS_MM))
    return n * (1.7 if c.get("full") else 1.0)   # a strip of sub-rays meets more pixels


def _one(c):
    """(bytes, flops) of a single request's pass."""
    M, q = c["subsets"], c["nx"] * c["ny"] * c["nz"]
    planes = len(_planes(c)) if c["nz"] > 1 else 1
    subset = c.get("subset", 0)
    angles = [a for a in range(c["angles"]) if subset == 0 or a % M == subset - 1]
    nnz, rays = _nnz(c, angles), len(angles) * planes * c["radial"]
    stencil = 280 if c["nz"] > 1 else 90
    kind = c["kind"]
    if kind == "forward" or kind == "back":
        return 4 * q + 4 * rays, 2 * nnz
    if kind == "gradient":
        return 8 * q + 8 * rays, 4 * nnz + 4 * rays + stencil * q
    if kind == "objective":
        return 4 * q + 8 * rays, 2 * nnz + 4 * rays + stencil * q
    it = c.get("iters", 1)
    penalty = 0 if c.get("mode") == "OSEM" else stencil
    # every subiteration reads and writes the image and reads the normaliser,
    # every iteration reads the counts and the background once
    return it * (12 * q * M + 8 * rays), it * (4 * nnz + 4 * rays + (penalty + 14) * q * M)


def work(case):
    parts = [_one(q) for q in _requests(case)] if case["kind"] == "batch" else [_one(case)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ------------------------------------------------------------------ FP64 values

class _Exact:
    """The system model and the method in FP64 (plain torch)."""

    def __init__(self, c, att=None):
        self.c, self.d = c, _desc(c)
        self.cs, self.sn = _angles(c)
        self.v = self.d["vx"]
        self.nx, self.ny, self.nz, self.Nr, self.Na = c["nx"], c["ny"], c["nz"], c["radial"], c["angles"]
        self.base, n = {}, 0
        for i, (r1, dd) in enumerate(_planes(c) if self.nz > 1 else [(0, 0)]):
            self.base.setdefault(dd, i)
            n = i + 1
        self.planes = n
        self.att = None if att is None else att.double()
        self.psf = None
        if c.get("full"):
            sigma = PSF_MM / (2 * math.sqrt(2 * math.log(2)))
            K = math.ceil(3 * sigma / self.v)
            t = torch.arange(-K, K + 1, dtype=torch.float64, device=DEV) * self.v
            w = torch.exp(-t * t / (2 * sigma * sigma))
            self.psf = w / w.sum()

    def angles(self, subset):
        return [a for a in range(self.Na) if subset == 0 or a % self.c["subsets"] == subset - 1]

    def _f64(self, x):
        return torch.as_tensor(x, dtype=torch.float64, device=DEV)

    def transaxial(self, a):
        """Per ray line of angle a (bins, or bins x sub-rays): radial position s,
        minor coordinate at every major boundary, cell cut t, lengths."""
        cs, sn, v = self.cs[a], self.sn[a], self.v
        row = abs(cs) >= abs(sn)
        nmaj, nmin = (self.ny, self.nx) if row else (self.nx, self.ny)
        n_sub = SUBRAYS if self.c.get("full") else 1
        b = torch.arange(self.Nr, dtype=torch.float64, device=DEV)
        s = (b - 0.5 * (self.Nr - 1)) * v
        off = ((torch.arange(n_sub, dtype=torch.float64, device=DEV) + 0.5) / n_sub - 0.5) * v
        s = (s[:, None] + off[None, :]).reshape(-1, 1)
        m = torch.arange(nmaj, dtype=torch.float64, device=DEV)[None, :]
        main, side = (cs, sn) if row else (sn, cs)
        if side == 0.0:
            # in grid units; whole bins exactly, since the bin spacing is the pixel's
            g0 = (2 * b - (self.Nr - 1) + nmin)[:, None] / 2 if n_sub == 1 else (s + 0.5 * nmin * v) / v
            g0 = g0.expand(-1, nmaj)
            return row, s, m, g0, g0, torch.ones_like(g0), v
        Y = (m - 0.5 * nmaj) * v
        g0 = (s - Y * side) / (main * v) + 0.5 * nmin
        Q = -side / main
        g1 = g0 + Q
        t = ((torch.floor(torch.maximum(g0, g1)) - g0) / Q).clamp(0.0, 1.0)
        return row, s, m, g0, g1, t, v / abs(main)

    def pieces(self, a):
        """Of angle a in 2D: (ray, pixel, length) of every piece."""
        row, s, m, g0, g1, t, L = self.transaxial(a)
        nmin = self.nx if row else self.ny
        n_sub = s.shape[0] // self.Nr
        rays, pix, lens = [], [], []
        ray = (torch.arange(s.shape[0], device=DEV) // n_sub)[:, None].expand_as(g0)
        for lo, hi in ((torch.zeros_like(t), t), (t, torch.ones_like(t))):
            cell = torch.floor(g0 + (g1 - g0) * 0.5 * (lo + hi))
            ok = (hi > lo) & (cell >= 0) & (cell < nmin)
            mm = m.expand_as(g0)[ok]
            cell = cell[ok]
            rays.append(ray[ok])
            pix.append((mm * self.nx + cell if row else cell * self.nx + mm).long())
            lens.append(((hi - lo) * L / n_sub)[ok])
        return torch.cat(rays), torch.cat(pix), torch.cat(lens)

    def pieces3(self, a):
        """Of angle a in 3D: per ring difference d (ray, column, slice offset, length)."""
        row, s, m, g0, g1, t, L = self.transaxial(a)
        nmin = self.nx if row else self.ny
        cs, sn = self.cs[a], self.sn[a]
        h = torch.sqrt(DET_RADIUS_MM ** 2 - s * s)
        nmaj = m.shape[1]

        def u(mm):
            Y = (mm - 0.5 * nmaj) * self.v
            return (-(s - Y * sn) / cs * sn + Y * cs) if row else (-Y * sn + (s - Y * cs) / sn * cs)

        tau0 = (u(m) + h) / (2 * h)
        tau1 = (u(m + 1) + h) / (2 * h)
        ray = torch.arange(self.Nr, device=DEV)[:, None].expand_as(g0)
        one, zero = torch.ones_like(t), torch.zeros_like(t)
        for d in range(-self.c["rd"], self.c["rd"] + 1):
            kap = torch.sqrt(1 + (d * 3.0 / (2 * h)) ** 2)
            z0, z1 = 0.5 + d * tau0, 0.5 + d * tau1
            tz = ((torch.floor(torch.maximum(z0, z1)) - z0) / (z1 - z0)).clamp(0.0, 1.0) if d else one
            t1, t2 = torch.minimum(t, tz), torch.maximum(t, tz)
            R, C, O, W = [], [], [], []
            for lo, hi in ((zero, t1), (t1, t2), (t2, one)):
                mid = 0.5 * (lo + hi)
                cell = torch.floor(g0 + (g1 - g0) * mid)
                o = torch.floor(z0 + (z1 - z0) * mid)
                ok = (hi > lo) & (cell >= 0) & (cell < nmin) & (o >= min(0, d)) & (o <= max(0, d))
                mm, cell = m.expand_as(g0)[ok], cell[ok]
                R.append(ray[ok])
                C.append((mm * self.nx + cell if row else cell * self.nx + mm).long())
                O.append(o[ok].long())
                W.append(((hi - lo) * kap * L)[ok])
            yield d, torch.cat(R), torch.cat(C), torch.cat(O), torch.cat(W)

    def blur(self, f):
        if self.psf is None:
            return f
        k = self.psf.numel() // 2
        w = self.psf
        f = torch.nn.functional.conv2d(f[None, None], w[None, None, None, :], padding=(0, k))
        return torch.nn.functional.conv2d(f, w[None, None, :, None], padding=(k, 0))[0, 0]

    def forward(self, f, subset):
        """[plane][angle of the subset][bin]"""
        al = self.angles(subset)
        out = torch.zeros((self.planes, len(al), self.Nr), dtype=torch.float64, device=DEV)
        if self.nz == 1:
            f = self.blur(f).reshape(-1)
            for i, a in enumerate(al):
                ray, pix, ln = self.pieces(a)
                out[0, i].index_add_(0, ray, ln * f[pix])
            return out if self.att is None else out * self.att[:, al]
        fz = f.permute(1, 2, 0).reshape(-1).contiguous()
        for i, a in enumerate(al):
            for d, ray, col, o, ln in self.pieces3(a):
                lo, n = max(0, -d), self.nz - abs(d)
                idx = (col * self.nz + o + lo)[:, None] + torch.arange(n, device=DEV)[None, :]
                q = torch.zeros((self.Nr, n), dtype=torch.float64, device=DEV)
                q.index_add_(0, ray, fz[idx] * ln[:, None])
                out[self.base[d]:self.base[d] + n, i] = q.t()
        return out

    def back(self, w, subset):
        """w: [plane][angle of the subset][bin]"""
        al = self.angles(subset)
        if self.nz == 1:
            if self.att is not None:
                w = w * self.att[:, al]
            out = torch.zeros(self.nx * self.ny, dtype=torch.float64, device=DEV)
            for i, a in enumerate(al):
                ray, pix, ln = self.pieces(a)
                out.index_add_(0, pix, ln * w[0, i][ray])
            return self.blur(out.reshape(self.ny, self.nx))
        out = torch.zeros(self.nx * self.ny * self.nz, dtype=torch.float64, device=DEV)
        for i, a in enumerate(al):
            for d, ray, col, o, ln in self.pieces3(a):
                lo, n = max(0, -d), self.nz - abs(d)
                idx = (col * self.nz + o + lo)[:, None] + torch.arange(n, device=DEV)[None, :]
                wd = w[self.base[d]:self.base[d] + n, i].t().contiguous()
                out.index_add_(0, idx.reshape(-1), (wd[ray] * ln[:, None]).reshape(-1))
        return out.reshape(self.ny, self.nx, self.nz).permute(2, 0, 1).contiguous()

    def ones(self, subset):
        return torch.ones((self.planes, len(self.angles(subset)), self.Nr), dtype=torch.float64, device=DEV)

    def neighbours(self, f):
        """Every in-image neighbour image and its mask, 8 in 2D and 26 in 3D."""
        g = f.reshape(self.nz, self.ny, self.nx)
        zr = (-1, 0, 1) if self.nz > 1 else (0,)
        P = torch.nn.functional.pad(g, (1, 1, 1, 1, 1, 1), value=math.nan)
        for dz in zr:
            for dy in (-1, 0, 1):
                for dx in (-1, 0, 1):
                    if dx or dy or dz:
                        n = P[1 + dz:1 + dz + self.nz, 1 + dy:1 + dy + self.ny, 1 + dx:1 + dx + self.nx]
                        yield torch.nan_to_num(n), ~torch.isnan(n)

    def grad_penalty(self, f, p):
        g = f.reshape(self.nz, self.ny, self.nx)
        acc = torch.zeros_like(g)
        for n, ok in self.neighbours(f):
            d = g - n
            den = g + n + p["gamma_R"] * d.abs() + p["eps"]
            acc += torch.where(ok, d * (p["gamma_R"] * d.abs() + g + 3 * n + 2 * p["eps"]) / den ** 2, torch.zeros_like(g))
        return (2 * acc).reshape(f.shape)

    def penalty(self, f, p):
        g = f.reshape(self.nz, self.ny, self.nx)
        acc = 0.0
        for n, ok in self.neighbours(f):
            d = g - n
            acc += float(torch.where(ok, d * d / (g + n + p["gamma_R"] * d.abs() + p["eps"]), torch.zeros_like(g)).sum())
        return acc

    def mu(self, f):
        g = f.reshape(self.nz, self.ny, self.nx)
        sq = torch.zeros_like(g)
        for ax in range(3):
            if g.shape[ax] > 1:
                sq += torch.gradient(g, dim=ax)[0] ** 2
        return torch.clamp_min(torch.sqrt(sq) / g.mean(), 0.01).reshape(f.shape)

    def gradient(self, f, y, r, subset, p, beta):
        al = self.angles(subset)
        w = 1.0 - y[:, al] / (self.forward(f, subset) + r[:, al])
        return self.back(w, subset) + beta * self.grad_penalty(f, p)

    def iterate(self, f, y, r, p, k0, iters):
        M = self.c["subsets"]
        t, km = 1.0, p["mode"] in ("M2", "P2")
        if p["mode"] != "OSEM":
            s = self.back(self.ones(0), 0)
            pn = torch.where(s > 0, s / M, torch.full_like(s, 1.0 / M))
        for k in range(k0, k0 + iters):
            for i in range(1, M + 1):
                if p["mode"] == "OSEM":
                    al = self.angles(i)
                    si = self.back(self.ones(i), i)
                    b = self.back(y[:, al] / (self.forward(f, i) + r[:, al]), i)
                    f = torch.where(si > 0, f * b / si.clamp_min(1e-300), f)
                    continue
                J = k * M + i
                alpha = 1.0
                if km:
                    alpha = (p["rho"] * (J - 1) + p["delta2"]) / (J - 1 + p["delta1"])
                elif p["mode"] in ("M1", "P1"):
                    tn = 0.5 * (1 + math.sqrt(1 + 4 * t * t))
                    alpha, t = 1 + (t - 1) / tn, tn
                nu = 1.0
                if p["mode"] in ("P1", "P2") and J > p["J0"]:
                    mu = self.mu(f)
                    nu = (mu.mean() / mu).clamp(p["nu1"], p["nu2"])
                G = self.gradient(f, y, r, i, p, p["beta"] / M)
                S = torch.where(f < 0.5 * p["U"], f, p["U"] - f) / pn
                ft = f - p["lambda0"] / (p["a"] * k + 1) * alpha * nu * S * G
                f = torch.where(ft <= 0, torch.full_like(ft, p["t_clip"]),
                                torch.where(ft >= p["U"], torch.full_like(ft, p["U"] - p["t_clip"]), ft))
        return f


def exact(case, seed):
    if case["kind"] == "batch":
        out = []
        for k, q in enumerate(_requests(case)):
            f, y, r, _ = _inputs(q, seed * 1000 + k)
            out.append(_Exact(q).iterate(f.double(), y.double(), r.double(), _params(q), 0, q["iters"]))
        return out
    c = case
    rays = len(_planes(c)) * c["angles"] * c["radial"] if c["nz"] > 1 else 0
    passes = {"iterate": 2, "reconstruct": 2 * c.get("iters", 1)}.get(c["kind"], 1)
    if rays * passes * max(c["nx"], c["ny"]) > 8e9 and c["kind"] in ("iterate", "reconstruct"):
        return None     # tens of seconds
    f, y, r, att = _inputs(c, seed)
    E = _Exact(c, att)
    f, p = f.double(), _params(c)
    if c["kind"] == "forward":
        out = torch.zeros((E.planes, E.Na, E.Nr), dtype=torch.float64, device=DEV)
        out[:, E.angles(c["subset"])] = E.forward(f, c["subset"])
        return out
    if c["kind"] == "back":
        w = (1.0 - y / (y.mean() + r)).double()
        return E.back(w[:, E.angles(c["subset"])].contiguous(), c["subset"])
    y, r = y.double(), r.double()
    if c["kind"] == "gradient":
        M = c["subsets"]
        return E.gradient(f, y, r, c["subset"], p, p["beta"] if c["subset"] == 0 else p["beta"] / M)
    if c["kind"] == "objective":
        total = 0.0
        for i in range(1, c["subsets"] + 1):
            q, al = E.forward(f, i), E.angles(i)
            total += float((q - y[:, al] * torch.log(q + r[:, al])).sum())
        return total + p["beta"] * E.penalty(f, p)
    return E.iterate(f, y, r, p, c.get("k0", 0), c.get("iters", 1))
