"""The work a user has this library do, as cases that can be timed.

One pass is what a model does once per timestep with the library: the forcing
of the step changes w in its lowest levels (surface heating accelerates the
air above the ground), and the provisional velocity is projected in place. The
increment also keeps every pass's divergence, and so its pressure, of the same
size: projecting a projected field again would return round-off for p.

`call` names the entry point: "project" (Plan.project), "stats" (the same with
the per-level mean and max of the outputs), "noalloc" (the workspace in the
library's static array), "batched" (project_batched over an ensemble) and
"var" (Plan.project_var, a density varying in x, y and z). `dtype` is the
plan's: "f64", or "mixed" (FP32 fields, FP64 refinement; "var" keeps FP64
fields and takes the FP32 preconditioner). Plans are made with the library's
defaults, as a program makes them for a grid it has not tuned.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2009_12849_amd as monc

DX = DY = 25.0
# the ensemble's member grids, and members of the other lengths that nested
# or limited-area runs come with
MEMBERS = [(64, 64, 64), (128, 128, 96), (192, 192, 128), (256, 256, 128)]
RAGGED = [(48, 36, 24), (72, 54, 33), (96, 96, 50), (108, 144, 64), (162, 128, 41), (81, 96, 30)]
USUAL = [16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024, 1536, 2048]
LENGTHS = sorted(2 ** a * 3 ** b for a in range(12) for b in range(7) if 16 <= 2 ** a * 3 ** b <= 2048)


def listed():
    def one(name, call, dtype, nx, ny, nz, **kw):
        return dict(name=name, call=call, dtype=dtype, nx=nx, ny=ny, nz=nz, profile="capped", fields="modes", **kw)

    return [
        # a unit-test sized domain: nothing but launches and latency
        one("cube32_f64", "project", "f64", 32, 32, 32),
        # one process's share of a weak-scaling run, inside a program that
        # allocates nothing after start-up
        one("share32_mixed_noalloc", "noalloc", "mixed", 32, 32, 64),
        # an ordinary boundary-layer domain in plain FP64
        one("layer256_f64", "project", "f64", 256, 256, 128),
        # a production step with the diagnostics an I/O server asks for
        one("layer384_mixed_stats", "stats", "mixed", 384, 256, 96),
        # domains sized by the site and not by the FFT: lengths 2^a 3^b
        one("site432_f64", "project", "f64", 432, 288, 75),
        one("site243_mixed", "project", "mixed", 243, 324, 61),
        # a large-eddy run on one GPU
        one("les1024_mixed", "project", "mixed", 1024, 1024, 256),
        # a whole ensemble of uneven members in one call
        dict(name="ensemble48_mixed", call="batched", dtype="mixed", members=48, ragged=False, pick=4000),
        # one GPU's share of a large run: the benchmark's grid, both paths
        dict(name="share2048_mixed", call="project", dtype="mixed", nx=2048, ny=2048, nz=160, profile="stretched",
             fields="spectra"),
        dict(name="share2048_f64", call="project", dtype="f64", nx=2048, ny=2048, nz=160, profile="stretched",
             fields="spectra"),
        # a density that varies along all axes: the Krylov solver with either
        # preconditioner
        one("var256_f64", "var", "f64", 256, 256, 128, amp=0.2),
        one("var288_mixed", "var", "mixed", 288, 216, 48, amp=0.3),
    ]


def _levels(rng):
    return int(round(math.exp(rng.uniform(math.log(8), math.log(256)))))


def draw(rng):
    call = rng.choices(["project", "stats", "noalloc", "batched", "var"], [10, 2, 2, 3, 3])[0]
    dtype = rng.choice(["f64", "mixed"])
    if call == "batched":
        return dict(call=call, dtype=dtype, members=rng.randint(4, 24), ragged=rng.random() < 0.5,
                    pick=rng.randrange(1 << 20))
    top = {"noalloc": 21, "var": 22}.get(call, 26)
    while True:
        points = 2.0 ** rng.uniform(14, top)
        nz = _levels(rng)
        pool = USUAL if rng.random() < 0.5 else LENGTHS
        ny = rng.choice(pool)
        nx = min(pool, key=lambda n: abs(math.log(n * ny * nz / points)))
        if 0.5 < nx * ny * nz / points < 2.0 and max(nx, ny) <= 16 * min(nx, ny):
            break
    case = dict(call=call, dtype=dtype, nx=nx, ny=ny, nz=nz, profile=rng.choice(["capped", "stretched"]),
                fields=rng.choice(["modes", "spectra"]))
    if call == "var":
        case["amp"] = round(rng.uniform(0.1, 0.3), 3)
    return case


# ---------------------------------------------------------------------------
# grids and inputs
# ---------------------------------------------------------------------------
def _rho0(dz, height=8000.0):
    zc = np.cumsum(dz) - 0.5 * dz
    return 1.2 * np.exp(-zc / height)


def _grids(case):
    """[(nx, ny, nz, dz, rho0)] of the case's members."""
    if case["call"] == "batched":
        shapes = RAGGED if case["ragged"] else MEMBERS
        rng = np.random.default_rng(case["pick"])
        out = []
        for s in rng.integers(0, len(shapes), size=case["members"]):
            nx, ny, nz = shapes[s]
            dz = 10.0 * rng.uniform(1.00, 1.02) ** np.arange(nz, dtype=np.float64)
            out.append((nx, ny, nz, dz, _rho0(dz, rng.uniform(6000.0, 10000.0))))
        return out
    nz = case["nz"]
    k = np.arange(nz, dtype=np.float64)
    if case["profile"] == "stretched":
        dz = 5.0 * 20.0 ** (k / max(1, nz - 1))
    else:
        dz = np.minimum(10.0 * 1.015 ** k, 60.0)
    return [(case["nx"], case["ny"], nz, dz, _rho0(dz))]


def _modes(gen, nx, ny, count=8):
    """(ny, nx) sum of low-wavenumber plane waves."""
    x = torch.arange(nx, device="cuda", dtype=torch.float64) / nx
    y = torch.arange(ny, device="cuda", dtype=torch.float64) / ny
    r = torch.rand((count, 2), generator=gen, device="cuda", dtype=torch.float64).cpu()
    mn = torch.randint(-4, 5, (count, 2), generator=gen, device="cuda").cpu()
    out = torch.zeros((ny, nx), device="cuda", dtype=torch.float64)
    for c in range(count):
        m, n = int(mn[c, 0]), int(mn[c, 1])
        if m == 0 and n == 0:
            m = 1
        out += (0.5 + float(r[c, 0])) * torch.cos(
            2 * math.pi * (m * x[None, :] + n * y[:, None] + float(r[c, 1])))
    return out


def _fill(gen, t, std, spectral):
    """Fill t (nz, ny, nx) level block by level block: white noise, or a
    k^-5/3 horizontal spectrum with random phases, of the given deviation."""
    nz, ny, nx = t.shape
    step = max(1, (1 << 26) // (nx * ny))
    if spectral:
        m = torch.arange(nx // 2 + 1, device="cuda", dtype=torch.float64)
        n = torch.fft.fftfreq(ny, 1.0 / ny, device="cuda", dtype=torch.float64)
        kappa = torch.sqrt(n[:, None] ** 2 + m[None, :] ** 2)
        inside = (kappa >= 1.0) & (kappa <= min(nx, ny) / 2.0)
        amp = torch.where(inside, kappa.clamp(min=1.0) ** (-4.0 / 3.0), torch.zeros_like(kappa))
    for k in range(0, nz, step):
        part = t[k:k + step]
        if spectral:
            phase = torch.rand((part.shape[0],) + tuple(amp.shape), generator=gen, device="cuda", dtype=torch.float64)
            f = torch.fft.irfft2(torch.polar(amp.expand_as(phase).contiguous(), 2 * math.pi * phase), s=(ny, nx))
            f *= std / f.std(dim=(1, 2), keepdim=True)
            part.copy_(f)
        else:
            part.copy_(torch.randn(part.shape, generator=gen, device="cuda", dtype=t.dtype) * std)


def _buffers(grids, dtype):
    """One flat zeroed buffer per field for all members, and its views."""
    sizes = [(nx * ny * nz + 63) // 64 * 64 for nx, ny, nz, _, _ in grids]
    flat = torch.zeros(sum(sizes), device="cuda", dtype=dtype)
    views, at = [], 0
    for (nx, ny, nz, _, _), size in zip(grids, sizes):
        views.append(flat[at:at + nx * ny * nz].view(nz, ny, nx))
        at += size
    return flat, views


def _inputs(case, seed):
    """What a pass starts from: the fields of every member, the levels of w
    the step's forcing changes, its increments, and the density field."""
    grids = _grids(case)
    dtype = torch.float32 if case["dtype"] == "mixed" and case["call"] != "var" else torch.float64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    spectral = case.get("fields") == "spectra"
    s = {"grids": grids}
    for name, std in (("u", 2.0), ("v", 2.0), ("w", 0.5)):
        s[name], views = _buffers(grids, dtype)
        s[name + "s"] = views
        for t in views:
            _fill(gen, t, std, spectral)
            if name != "w" and not spectral:
                t += _modes(gen, t.shape[2], t.shape[1]).to(dtype)
    s["slabs"], s["heat"] = [], []
    for t in s["ws"]:
        t[-1] = 0.0
        lowest = t[:max(1, t.shape[0] // 8)]
        heat = torch.empty_like(lowest)
        _fill(gen, heat, 0.25, False)
        s["slabs"].append(lowest)
        s["heat"].append(heat)
    if case["call"] == "var":
        nx, ny, nz, dz, rho0 = grids[0]
        c = torch.from_numpy((np.cumsum(dz) - 0.5 * dz) / dz.sum()).cuda()[:, None, None]
        f1, f2 = (f / f.abs().max() for f in (_modes(gen, nx, ny), _modes(gen, nx, ny)))
        s["rho"] = torch.from_numpy(rho0).cuda()[:, None, None] * (1.0 + case["amp"] * (c * f1 + (1.0 - c) * f2))
        # the plan's reference density: the level means, as a model takes them
        s["grids"] = [(nx, ny, nz, dz, s["rho"].mean(dim=(1, 2)).cpu().numpy())]
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["call"] = case["call"]
    s["plans"] = [monc.Plan(nx, ny, nz, DX, DY, dz, rho0, case["dtype"]) for nx, ny, nz, dz, rho0 in s["grids"]]
    s["p"], s["ps"] = _buffers(s["grids"], s["u"].dtype)
    if case["call"] == "stats":
        s["stats"] = torch.zeros(8 * case["nz"], device="cuda", dtype=torch.float64)
    return s


def run(s):
    out = {"u": s["u"], "v": s["v"], "w": s["w"], "p": s["p"]}
    if s["call"] == "batched":
        torch._foreach_add_(s["slabs"], s["heat"])
        monc.project_batched(s["plans"], s["us"], s["vs"], s["ws"], s["ps"])
        return out
    s["slabs"][0].add_(s["heat"][0])
    plan, fields = s["plans"][0], (s["us"][0], s["vs"][0], s["ws"][0], s["ps"][0])
    if s["call"] == "project":
        plan.project(*fields)
    elif s["call"] == "stats":
        plan.project(*fields, stats=s["stats"])
        out["stats"] = s["stats"]
    elif s["call"] == "noalloc":
        plan.project_noalloc(*fields)
    else:
        # the residual that it stops at is round-off in its own digits: only
        # the iteration count is an output beside the fields
        out["iterations"] = plan.project_var(s["rho"], *fields)[0]
    return out


def work(case):
    """Each input read once, each output written once; the transforms' and
    the column solves' operations of one solve."""
    nbytes = flops = 0.0
    width = 4 if case["dtype"] == "mixed" and case["call"] != "var" else 8
    for nx, ny, nz, _, _ in _grids(case):
        n = float(nx * ny * nz)
        words = 7.0 + (1.0 if case["call"] == "var" else 0.0)   # u, v, w in and out, p out, rho in
        nbytes += n * width * words + nx * ny * max(1, nz // 8) * width
        flops += n * (5.0 * math.log2(max(2, nx * ny)) + 40.0)
    if case["call"] == "stats":
        nbytes += 64.0 * case["nz"]
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# the same results in plain FP64 torch
# ---------------------------------------------------------------------------
def _column(x):
    return torch.as_tensor(x, dtype=torch.float64, device="cuda")[:, None, None]


def _vertical(dz, rho0):
    """Face densities and off-diagonals of the vertical operator."""
    dzc = 0.5 * (dz[:-1] + dz[1:])
    rhow = (dz[1:] * rho0[:-1] + dz[:-1] * rho0[1:]) / (dz[:-1] + dz[1:])
    a, c = np.zeros(len(dz)), np.zeros(len(dz))
    a[1:] = rhow / (dz[1:] * dzc)
    c[:-1] = rhow / (dz[:-1] * dzc)
    return dzc, rhow, a, c


def _solve(b, dz, rho0):
    """Pressure of the separable problem D(G p) = b, gauge sum dz p = 0:
    b is overwritten level by level with what it becomes."""
    nz, ny, nx = b.shape
    _, _, a, c = _vertical(dz, rho0)
    lx = (4.0 / DX ** 2) * np.sin(np.pi * np.arange(nx // 2 + 1) / nx) ** 2
    ly = (4.0 / DY ** 2) * np.sin(np.pi * np.arange(ny) / ny) ** 2
    lam = torch.from_numpy(ly[:, None] + lx[None, :]).cuda()
    spec = [torch.fft.rfft2(b[k]) for k in range(nz)]
    mean = np.array([complex(s[0, 0].item()) for s in spec])
    safe = lam.clone()
    safe[0, 0] = 1.0
    gain = []
    for k in range(nz):  # forward elimination, one level at a time
        den = -(a[k] + c[k]) - rho0[k] * safe
        if k:
            den -= a[k] * gain[-1]
            spec[k] = (spec[k] - a[k] * spec[k - 1]) / den
        else:
            spec[k] = spec[k] / den
        gain.append(c[k] / den)
    for k in range(nz - 1, -1, -1):
        if k < nz - 1:
            spec[k] = spec[k] - gain[k] * spec[k + 1]
        gain[k] = None
    # the mean column: singular, top unknown pinned, then the gauge
    rhs = mean - np.sum(dz * mean) / dz.sum()
    mode = np.zeros(nz, dtype=np.complex128)
    if nz > 1:
        mat = np.diag(-(a + c)) + np.diag(a[1:], -1) + np.diag(c[:-1], 1)
        mode[:-1] = np.linalg.solve(mat[:-1, :-1], rhs[:-1])
    mode -= np.sum(dz * mode) / dz.sum()
    for k in range(nz):
        spec[k][0, 0] = complex(mode[k])
        b[k] = torch.fft.irfft2(spec[k], s=(ny, nx))
        spec[k] = None
    return b


def _correct(u, v, w, p, dz):
    """u - G p, the lid at rest (in place)."""
    dzc = 0.5 * (dz[:-1] + dz[1:])
    u -= (torch.roll(p, -1, 2) - p) / DX
    v -= (torch.roll(p, -1, 1) - p) / DY
    w[:-1] -= (p[1:] - p[:-1]) / _column(dzc)
    w[-1] = 0.0


def _exact_project(u, v, w, dz, rho0):
    _, rhow, _, _ = _vertical(dz, rho0)
    b = (u - torch.roll(u, 1, 2)) / DX
    b += (v - torch.roll(v, 1, 1)) / DY
    b *= _column(rho0)
    flux = _column(rhow) * w[:-1]
    b[:-1] += flux / _column(dz[:-1])
    b[1:] -= flux / _column(dz[1:])
    del flux
    p = _solve(b, dz, rho0)
    _correct(u, v, w, p, dz)
    return p


def _exact_var(u, v, w, rho, dz, rho0):
    """Conjugate gradients to FP64's own limit, the separable solve as the
    preconditioner."""
    rx, ry = 0.5 * (rho + torch.roll(rho, -1, 2)), 0.5 * (rho + torch.roll(rho, -1, 1))
    rz = (_column(dz[1:]) * rho[:-1] + _column(dz[:-1]) * rho[1:]) / _column(dz[:-1] + dz[1:])
    dzc, wt = _column(0.5 * (dz[:-1] + dz[1:])), _column(dz)

    def div(a, b, c):
        fx, fy, fz = rx * a, ry * b, rz * c
        out = (fx - torch.roll(fx, 1, 2)) / DX + (fy - torch.roll(fy, 1, 1)) / DY
        out[:-1] += fz / wt[:-1]
        out[1:] -= fz / wt[1:]
        return out

    def apply(q):
        return div((torch.roll(q, -1, 2) - q) / DX, (torch.roll(q, -1, 1) - q) / DY, (q[1:] - q[:-1]) / dzc)

    def dot(a, b):
        return float((wt * a * b).sum())

    r = div(u, v, w[:-1])
    r -= (wt * r).mean() / wt.mean()
    p = torch.zeros_like(r)
    first, d, rz_old = dot(r, r), None, 0.0
    for _ in range(60):
        if dot(r, r) <= 1e-30 * first:
            break
        z = _solve(r.clone(), dz, rho0)
        rz_new = dot(r, z)
        d = z if d is None else z + (rz_new / rz_old) * d
        q = apply(d)
        alpha = rz_new / dot(d, q)
        p += alpha * d
        r -= alpha * q
        rz_old = rz_new
    p -= (wt * p).mean() / wt.mean()
    _correct(u, v, w, p, dz)
    return p


def exact(case, seed):
    s = _inputs(case, seed)
    for slab, heat in zip(s["slabs"], s["heat"]):
        slab.add_(heat)
    out = {n: s[n].double() for n in ("u", "v", "w")}
    out["p"] = torch.zeros_like(out["u"])
    del s["u"], s["v"], s["w"], s["slabs"], s["heat"]
    stats, at = None, 0
    for i, (nx, ny, nz, dz, rho0) in enumerate(s["grids"]):
        n = nx * ny * nz
        u, v, w, p = (out[name][at:at + n].view(nz, ny, nx) for name in ("u", "v", "w", "p"))
        if case["call"] == "var":
            p.copy_(_exact_var(u, v, w, s["rho"], dz, rho0))
        else:
            p.copy_(_exact_project(u, v, w, dz, rho0))
        if case["call"] == "stats":
            stats = torch.stack([x for f in (u, v, w, p) for x in (f.mean(dim=(1, 2)), f.amax(dim=(1, 2)))])
        at += (n + 63) // 64 * 64
    if stats is not None:
        out["stats"] = stats.reshape(-1)
    if case["call"] == "var":
        out["iterations"] = None
    return out
