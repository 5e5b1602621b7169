"""The work that users of the Gross-Pitaevskii library have it do, as measurable cases.

A case is one call sequence of a user's program on one set of sizes: a stretch of a
simulation with its diagnostics (``evolve``), an ensemble of runs (``ensemble``), a
piece of the imaginary-time preparation (``argle``), a gradient through the split
step (``adjoint``), the analysis of a stored state (``analysis``, ``helicity``) and
the construction of a random-vortex-ring state (``rvr``).  ``listed`` names the
sizes of the repository's own workloads and benchmark, ``draw`` spreads further
ones over the same ranges.  ``exact`` evaluates the same quantities from their
definitions with torch in complex128.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2003_03590_amd as gp

TWO_PI = 2.0 * math.pi
DEV = "cuda"


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest runs: a 32^3 box reported every 20 steps, plan as created
        {"name": "srp32_c128", "kind": "evolve", "nx": 32, "ny": 32, "nz": 32, "prec": "c128", "steps": 20,
         "ic": "srp", "tune": False, "diag": True},
        # an elongated box with three different axes, one of them short, in FP32
        {"name": "box96x48x24_c64", "kind": "evolve", "nx": 96, "ny": 48, "nz": 24, "prec": "c64", "steps": 10,
         "ic": "tangle", "tune": False, "diag": True},
        # the paper's 128^3 quench runs (ten seeds each), plan as created
        {"name": "quench128_c128", "kind": "evolve", "nx": 128, "ny": 128, "nz": 128, "prec": "c128", "steps": 50,
         "ic": "tangle", "tune": False, "diag": True},
        # the benchmark's 256^3 run, autotuned as there: 100 steps between spectra
        {"name": "box256_c128", "kind": "evolve", "nx": 256, "ny": 256, "nz": 256, "prec": "c128", "steps": 100,
         "ic": "tangle", "tune": True, "diag": True},
        {"name": "box256_c64", "kind": "evolve", "nx": 256, "ny": 256, "nz": 256, "prec": "c64", "steps": 100,
         "ic": "tangle", "tune": True, "diag": True},
        # the largest grid, far beyond the caches, steps alone
        {"name": "box1024_c64", "kind": "evolve", "nx": 1024, "ny": 1024, "nz": 1024, "prec": "c64", "steps": 5,
         "ic": "srp", "tune": True, "diag": False},
        # the 48-run ensemble (32 at 64^3, 16 at 96^3), autotuned, 50 steps between reports
        {"name": "ens48_c64", "kind": "ensemble", "runs": "64*32,96*16", "prec": "c64", "steps": 50, "tune": True},
        # imaginary-time preparation at 256^3 with the stopping rule looked at every 10 steps
        {"name": "argle256_c128", "kind": "argle", "n": 256, "steps": 20, "check": 10},
        # the gradient of a spectral energy with respect to the initial phase, checkpoints every 20 steps
        {"name": "adjoint128_c128", "kind": "adjoint", "n": 128, "steps": 40, "ckpt": 20, "smin": 4, "smax": 12},
        # post-processing of a large FP32 state: spectra, structure functions, Mach numbers
        {"name": "analysis512_c64", "kind": "analysis", "n": 512, "prec": "c64"},
        # helicities and their spectra of a vortex tangle
        {"name": "helicity128_c128", "kind": "helicity", "nx": 128, "ny": 128, "nz": 128, "prec": "c128"},
        # the random-vortex-ring state of the 128^3 runs: 200 pairs
        {"name": "rvr128_c128", "kind": "rvr", "n": 128, "pairs": 200, "prec": "c128"},
    ]


LENGTHS = (16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512)


def _near(rng, lo, hi):
    """A length between lo and hi, even over the logarithm."""
    t = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min((v for v in LENGTHS if lo <= v <= hi), key=lambda v: abs(math.log(v / t)))


def _box(rng, lo, hi, most):
    """Three axes about one length; in half of the draws they differ."""
    while True:
        n = _near(rng, lo, hi)
        shape = [n, n, n]
        if rng.random() < 0.5:
            i = LENGTHS.index(n)
            shape = [LENGTHS[max(0, min(len(LENGTHS) - 1, i + rng.randint(-2, 2)))] for _ in range(3)]
        if shape[0] * shape[1] * shape[2] <= most:
            return shape


def draw(rng):
    kind = rng.choice(["evolve"] * 6 + ["ensemble", "argle", "adjoint", "analysis", "helicity", "rvr"])
    prec = rng.choice(["c128", "c64"])
    if kind == "evolve":
        nx, ny, nz = _box(rng, 16, 512, 1 << 27)
        most = 40 if nx * ny * nz <= 1 << 24 else 10
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "prec": prec, "steps": rng.randint(4, most),
                "ic": rng.choice(["srp", "tangle"]), "tune": rng.random() < 0.5, "diag": rng.random() < 0.6}
    if kind == "ensemble":
        sizes = rng.sample([16, 24, 32, 48, 64, 96], rng.randint(1, 3))
        return {"kind": kind, "runs": ",".join(f"{n}*{rng.randint(1, 16)}" for n in sizes), "prec": prec,
                "steps": rng.randint(5, 60), "tune": rng.random() < 0.5}
    if kind == "argle":
        n = _near(rng, 32, 256)
        check = rng.randint(3, 10)
        return {"kind": kind, "n": n, "steps": rng.randint(check, 20), "check": check}
    if kind == "adjoint":
        n = _near(rng, 16, 128)
        ckpt = rng.randint(5, 20)
        return {"kind": kind, "n": n, "steps": rng.randint(ckpt, 40), "ckpt": ckpt, "smin": 2, "smax": n // 8 + 4}
    if kind == "analysis":
        return {"kind": kind, "n": _near(rng, 32, 512), "prec": prec}
    if kind == "helicity":
        nx, ny, nz = _box(rng, 24, 192, 1 << 23)
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "prec": "c128"}
    n = _near(rng, 32, 256)
    return {"kind": kind, "n": n, "pairs": rng.randint(1, 40 if n > 128 else 200), "prec": prec}


# ------------------------------------------------------------------ inputs
def _coef(n):
    """alpha = 6.4/N, beta = N/3.2 (the paper's parameter rule)."""
    return 6.4 / n, n / 3.2


def _dt(n):
    return 1e-3 if n <= 128 else 5e-4 if n <= 512 else 2.5e-4


def _smooth(shape, K, gen):
    """Re sum over |k| <= K of random Gaussian modes, scaled to rms 1 (FP64, [z][y][x])."""
    ks = [torch.arange(-min(K, n // 4), min(K, n // 4) + 1, dtype=torch.float64) for n in shape]
    hat = torch.randn([len(k) for k in ks] + [2], dtype=torch.float64, generator=gen)
    k2 = ks[0][:, None, None] ** 2 + ks[1][None, :, None] ** 2 + ks[2][None, None, :] ** 2
    hat = torch.view_as_complex(hat) * ((k2 > 0) & (k2 <= K * K))
    hat = hat.to(DEV)
    e = [torch.exp(1j * k.to(DEV)[:, None] * (TWO_PI / n) * torch.arange(n, device=DEV, dtype=torch.float64)[None, :])
         for k, n in zip(ks, shape)]
    a = (hat.reshape(-1, hat.shape[2]) @ e[2]).reshape(hat.shape[0], hat.shape[1], shape[2])
    b = torch.stack([e[1].T.contiguous() @ a[i] for i in range(a.shape[0])]).reshape(a.shape[0], -1)
    out = e[0].real.T.contiguous() @ b.real.contiguous()
    out -= e[0].imag.T.contiguous() @ b.imag.contiguous()
    out = out.reshape(shape)
    return out.div_(torch.sqrt(torch.mean(out * out)).clamp_min(1e-30))


def _psi(shape, ic, prec, seed):
    """An initial state: 'srp' a smoothed random phase, 'tangle' a random complex field
    whose zeros are vortex lines with healed cores, 'waves' phase and density waves
    without zeros."""
    gen = torch.Generator().manual_seed(int(seed))
    if ic == "srp":
        psi = torch.polar(torch.ones(shape, dtype=torch.float64, device=DEV), _smooth(shape, 4, gen))
    elif ic == "waves":
        psi = torch.polar(torch.exp(0.15 * _smooth(shape, 4, gen)), _smooth(shape, 4, gen))
    else:
        psi = torch.complex(_smooth(shape, 4, gen), _smooth(shape, 4, gen))
        psi = psi / torch.sqrt(0.05 + psi.real ** 2 + psi.imag ** 2)
    return psi.to(torch.complex64 if prec == "c64" else torch.complex128).contiguous()


def _runs(case):
    out = []
    for part in case["runs"].split(","):
        n, count = (int(v) for v in part.split("*"))
        out += [n] * count
    return out


def _theta(case, seed):
    return _smooth((case["n"],) * 3, 6, torch.Generator().manual_seed(int(seed))).contiguous()


def _argle_inputs(case, seed):
    """A smooth phase field and the Taylor-Green flow moved by a random offset."""
    n = case["n"]
    gen = torch.Generator().manual_seed(int(seed))
    off = torch.rand(3, dtype=torch.float64, generator=gen) * TWO_PI
    x, y, z = [(TWO_PI / n) * torch.arange(n, dtype=torch.float64, device=DEV) + float(o) for o in off]
    x, y, z = x[None, None, :], y[None, :, None], z[:, None, None]
    v = torch.stack([torch.sin(x) * torch.cos(y) * torch.cos(z), -torch.cos(x) * torch.sin(y) * torch.cos(z),
                     torch.zeros((n, n, n), dtype=torch.float64, device=DEV)])
    phi = torch.polar(torch.ones((n, n, n), dtype=torch.float64, device=DEV), 2.0 * _smooth((n, n, n), 3, gen))
    return phi.contiguous(), v.contiguous()


ARGLE_ALPHA, ARGLE_BETA = 0.05, 40.0


def _pairs(case, seed):
    """Ring pairs (R, d, X, Y, Z, permutation) as the library takes them, and the core width."""
    rng = np.random.default_rng(int(seed))
    alpha, beta = _coef(case["n"])
    out = []
    for _ in range(case["pairs"]):
        R = float(rng.uniform(0.3, 1.6))
        X, Y, Z = (float(v) for v in rng.uniform(0.0, TWO_PI, 3))
        out.append((R, 2.0 * R, X, Y, Z, int(rng.integers(0, 6))))
    return out, math.sqrt(alpha / beta)


# ------------------------------------------------------------------ prepare and run
def _plan(shape_xyz, prec, tune=False):
    n = max(shape_xyz)
    alpha, beta = _coef(n)
    plan = gp.Plan(tuple(shape_xyz), alpha, beta, _dt(n), prec)
    if tune:
        plan.autotune(reps=3)
    return plan


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case)
    if kind == "evolve":
        xyz = (case["nx"], case["ny"], case["nz"])
        s["plan"] = _plan(xyz, case["prec"], case["tune"])
        s["psi"] = _psi(xyz[::-1], case["ic"], case["prec"], seed)
        if case["diag"]:
            s["plan"].work()
    elif kind == "ensemble":
        sizes = _runs(case)
        s["plan"] = gp.BatchPlan([dict(n=n, alpha=_coef(n)[0], beta=_coef(n)[1], dt=1e-3) for n in sizes],
                                 case["prec"])
        if case["tune"]:
            s["plan"].autotune(reps=3)
        s["psi"] = [_psi((n, n, n), "srp", case["prec"], 1000 * int(seed) + i) for i, n in enumerate(sizes)]
    elif kind == "argle":
        s["plan"] = gp.Plan(case["n"], ARGLE_ALPHA, ARGLE_BETA, 1e-3, "c128")
        s["plan"].work()
        s["phi"], s["v"] = _argle_inputs(case, seed)
    elif kind == "adjoint":
        s["plan"] = gp.Plan(case["n"], *_coef(case["n"]), 1e-3, "c128")
        s["plan"].work()
        s["theta"] = _theta(case, seed)
    elif kind == "analysis":
        s["plan"] = _plan((case["n"],) * 3, case["prec"])
        s["plan"].work()
        s["psi"] = _psi((case["n"],) * 3, "waves", case["prec"], seed)
    elif kind == "helicity":
        xyz = (case["nx"], case["ny"], case["nz"])
        s["plan"] = _plan(xyz, case["prec"])
        s["psi"] = _psi(xyz[::-1], "tangle", case["prec"], seed)
    else:
        s["plan"] = _plan((case["n"],) * 3, case["prec"])
        s["pairs"], s["xi"] = _pairs(case, seed)
        s["psi"] = s["plan"].empty()
    return s


def _kept(values, prec):
    """Diagnostic arrays as a program keeps them: in the real type of the state they come from."""
    return np.asarray(values, dtype=np.float32 if prec == "c64" else np.float64)


def run(s):
    kind, plan = s["kind"], s["plan"]
    if kind == "evolve":
        out = {"psi": plan.step_n(s["psi"], s["steps"])}
        if s["diag"]:
            spec, out["energies"] = plan.spectra(s["psi"])
            out["spec"] = _kept(spec, s["prec"])
        return out
    if kind == "ensemble":
        return {"psi": plan.step_n(s["psi"], s["steps"]), "energies": _kept(plan.energies(s["psi"]), s["prec"])}
    if kind == "argle":
        report = plan.argle_run(s["phi"], s["v"], 1.6 / s["n"], s["steps"], s["check"], 0.0)
        return {"phi": s["phi"], "report": report}
    if kind == "adjoint":
        theta = s["theta"].detach().requires_grad_()
        psi = gp.evolve(theta, plan, s["steps"], s["ckpt"])
        J = gp.ekin_i_shells(psi, plan, s["smin"], s["smax"])
        J.backward()
        return {"J": J.detach(), "psi": psi.detach(), "grad": theta.grad}
    if kind == "analysis":
        spec, energies = plan.spectra(s["psi"])
        rho = plan.structure_fn(s["psi"])
        vel, mean_v2 = plan.structure_fn_velocity(s["psi"])
        mach = plan.mach(s["psi"])
        return {"spec": _kept(spec, s["prec"]), "energies": energies, "rho": _kept(rho, s["prec"]),
                "vel": _kept(vel, s["prec"]), "mean_v2": _kept(mean_v2, s["prec"]), "mach": list(mach)}
    if kind == "helicity":
        H, Hreg, spec = plan.helicity(s["psi"])
        return {"H": [H, Hreg], "spec": _kept(spec, s["prec"])}
    return plan.init_rvr(s["pairs"], s["xi"], out=s["psi"])


# ------------------------------------------------------------------ work
def _transform_flops(points):
    return 5.0 * points * math.log2(max(2.0, points))


def _diag_work(points, size):
    """Four packed transforms and three derivatives; the state is read, the report is small."""
    return points * size, 4 * _transform_flops(points) + 2 * _transform_flops(points) + 150.0 * points


def work(case):
    """Bytes and operations that one pass cannot do without.  A time step (and each half of
    a gradient's step) takes every point through a 3-D transform and back, so the state
    crosses memory once per step, read and written; the transforms are 5 N log2 N."""
    kind = case["kind"]
    size = 8 if case.get("prec") == "c64" else 16
    if kind == "evolve":
        pts = float(case["nx"] * case["ny"] * case["nz"])
        b = 2.0 * pts * size * case["steps"]
        f = case["steps"] * (2 * _transform_flops(pts) + 20.0 * pts)
        if case["diag"]:
            db, df = _diag_work(pts, size)
            b, f = b + db, f + df
        return {"bytes": b, "flops": f}
    if kind == "ensemble":
        b = f = 0.0
        for n in _runs(case):
            pts = float(n) ** 3
            db, df = _diag_work(pts, size)
            b += 2.0 * pts * size * case["steps"] + db
            f += case["steps"] * (2 * _transform_flops(pts) + 20.0 * pts) + df
        return {"bytes": b, "flops": f}
    pts = float(case["n"]) ** 3 if "n" in case else float(case["nx"] * case["ny"] * case["nz"])
    if kind == "argle":
        # the field read and written and the three velocity planes read once per step
        return {"bytes": case["steps"] * pts * (2 * 16 + 3 * 8),
                "flops": case["steps"] * (3 * _transform_flops(pts) + 60.0 * pts)}
    if kind == "adjoint":
        # forward steps, the same steps again into the tape, the backward steps with the tape read
        return {"bytes": case["steps"] * pts * 16 * (2 + 2 + 3) + 2 * pts * 8,
                "flops": case["steps"] * 3 * (2 * _transform_flops(pts) + 30.0 * pts)}
    if kind == "analysis":
        b, f = _diag_work(pts, size)
        return {"bytes": 4 * b, "flops": f + 3 * _transform_flops(pts) + 100.0 * pts}
    if kind == "helicity":
        return {"bytes": pts * size, "flops": 10 * _transform_flops(pts) + 250.0 * pts}
    return {"bytes": pts * size, "flops": pts * (case["pairs"] * 14 * 30.0)}


# ------------------------------------------------------------------ exact values
def _k(n, first=False):
    k = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEV).round()
    if first and n % 2 == 0:
        k[n // 2] = 0.0
    return k


def _ks(shape, first=False):
    return [_k(n, first).reshape([-1 if a == b else 1 for b in range(3)]) for a, n in enumerate(shape)]


def _linear(psi, phases):
    c = torch.fft.fftn(psi)
    for p in phases:
        c = c * p
    return torch.fft.ifftn(c)


def _evolved(psi, alpha, beta, dt, steps):
    """Strang steps with adjacent half steps joined: L(h) [N L(dt)]^(n-1) N L(h)."""
    def phases(tau):
        return [torch.exp(-1j * alpha * tau * k * k) for k in _ks(psi.shape)]
    half, full = phases(0.5 * dt), phases(dt)
    psi = _linear(psi, half)
    for s in range(steps):
        psi = psi * torch.exp(-1j * beta * dt * (psi.real ** 2 + psi.imag ** 2 - 1.0))
        psi = _linear(psi, full if s + 1 < steps else half)
    return psi


def _grad(f):
    """(d/dx, d/dy, d/dz) of f [z][y][x], the Nyquist entry of the wavenumber zero."""
    out = []
    for ax in (2, 1, 0):
        k = _k(f.shape[ax], True).reshape([-1 if a == ax else 1 for a in range(3)])
        d = torch.fft.ifft(1j * k * torch.fft.fft(f, dim=ax), dim=ax)
        out.append(d if f.is_complex() else d.real)
    return out


def _shells(shape):
    kz, ky, kx = _ks(shape)
    q = (4 * (kz * kz + ky * ky + kx * kx)).to(torch.int64)
    r = torch.floor(torch.sqrt(q.to(torch.float64))).to(torch.int64)
    r = torch.where(r * r > q, r - 1, r)
    r = torch.where((r + 1) * (r + 1) <= q, r + 1, r)
    return ((r + 1) // 2).reshape(-1)


def _nshell(shape):
    k2 = sum((n // 2) ** 2 for n in shape)
    return (math.isqrt(4 * k2) + 1) // 2 + 1


def _binned(dens, s, ns):
    return torch.bincount(s, weights=dens.reshape(-1), minlength=ns)


def _parts(w, k2, kd):
    """Incompressible and compressible parts of the transforms w = [x, y, z]."""
    c = sum(k * f for k, f in zip(kd, w)) / torch.where(k2 > 0, k2, torch.ones_like(k2))
    comp = [k * c for k in kd]
    return [f - g for f, g in zip(w, comp)], comp


def _sum2(fields):
    return sum(f.real ** 2 + f.imag ** 2 for f in fields)


def _diagnostics(psi, alpha, beta):
    shape, pts = psi.shape, psi.numel()
    kz, ky, kx = _ks(shape)
    k2 = kz * kz + ky * ky + kx * kx
    s, ns = _shells(shape), _nshell(shape)
    rho = psi.real ** 2 + psi.imag ** 2
    amp = torch.sqrt(rho)
    t = [psi.conj() * d * (2.0 * alpha) / amp for d in _grad(psi)]
    e = {"mass": float(rho.mean()), "e_kin": 0.5 * float(sum((f.imag ** 2).mean() for f in t)),
         "e_int": alpha * beta * float(((rho - 1.0) ** 2).mean())}
    c = torch.fft.fftn(psi) / pts
    e["energy"] = 2.0 * alpha ** 2 * float((k2 * (c.real ** 2 + c.imag ** 2)).sum()) + e["e_int"]
    del c
    wi, wc = _parts([torch.fft.fftn(f.imag) / pts for f in t], k2, (kx, ky, kz))
    rows = [_binned(0.5 * _sum2(wi), s, ns), _binned(0.5 * _sum2(wc), s, ns)]
    del wi, wc
    rows.append(_binned(0.5 * _sum2([torch.fft.fftn(f.real) / pts for f in t]), s, ns))
    rows.append(_binned(alpha * beta * _sum2([torch.fft.fftn(rho - 1.0) / pts]), s, ns))
    spec = torch.stack(rows).cpu().numpy()
    e["e_kin_i"], e["e_kin_c"], e["e_q"] = (float(spec[i].sum()) for i in range(3))
    return spec, e


def _lag_sums(f, ax):
    """<(f(x + m e) - f(x))^2> for m = 1 .. N/2 along array axis ax, from the correlation."""
    n = f.shape[ax]
    F = torch.fft.fft(f, dim=ax)
    p = (F.real ** 2 + F.imag ** 2).sum(dim=[a for a in range(3) if a != ax])
    c = torch.fft.ifft(p).real / f.numel()
    return 2.0 * (c[0] - c[1:n // 2 + 1]).cpu().numpy()


def _argle_exact(case, seed):
    phi, v = _argle_inputs(case, seed)
    a, b, dtau = ARGLE_ALPHA, ARGLE_BETA, 1.6 / case["n"]
    kz, ky, kx = _ks(phi.shape)
    k2 = kz * kz + ky * ky + kx * kx
    v2 = (v * v).sum(0)
    h = 0.5 * dtau * a

    def energy(f):
        g = sum(_sum2([d - 1j * v[j] * f / (2.0 * a)]) for j, d in enumerate(_grad(f)))
        return 2.0 * a * float((a * g + 0.5 * b * (_sum2([f]) - 1.0) ** 2).mean())

    def step(f):
        adv = sum(v[j] * d for j, d in enumerate(_grad(f)))
        n = -1j * adv + (b - v2 / (4.0 * a) - b * _sum2([f])) * f
        return torch.fft.ifftn(((1.0 - h * k2) * torch.fft.fftn(f) + dtau * torch.fft.fftn(n)) / (1.0 + h * k2))

    for s in range(1, case["steps"] + 1):
        check = s == case["steps"]                 # the report holds the last check
        if check:
            old, e_old = phi, energy(phi)
        phi = step(phi)
    e_new = energy(phi)
    return {"phi": phi, "report": {
        "steps": None, "converged": None, "crit_sup": float((phi - old).abs().max()) / dtau,
        "crit_energy": abs(e_new - e_old) / (dtau * e_old), "e_v": e_new}}


def _adjoint_exact(case, seed):
    alpha, beta = _coef(case["n"])
    theta = _theta(case, seed).requires_grad_()
    psi = _evolved(torch.polar(torch.ones_like(theta), theta), alpha, beta, 1e-3, case["steps"])
    kz, ky, kx = _ks(psi.shape)
    k2 = kz * kz + ky * ky + kx * kx
    amp = torch.sqrt(psi.real ** 2 + psi.imag ** 2)
    w = [torch.fft.fftn((psi.conj() * d).imag * (2.0 * alpha) / amp) / psi.numel() for d in _grad(psi)]
    wi, _ = _parts(w, k2, (kx, ky, kz))
    s = _shells(psi.shape).reshape(psi.shape)
    J = 0.5 * (_sum2(wi) * ((s >= case["smin"]) & (s <= case["smax"]))).sum()
    J.backward()
    return {"J": J.detach(), "psi": psi.detach(), "grad": theta.grad}


def _helicity_exact(psi, alpha):
    shape, pts = psi.shape, psi.numel()
    d = _grad(psi)
    rho = psi.real ** 2 + psi.imag ** 2
    v = [2.0 * alpha * (psi.conj() * f).imag / rho for f in d]
    dv = [_grad(f) for f in v]                     # dv[component][axis]
    om = [dv[2][1] - dv[1][2], dv[0][2] - dv[2][0], dv[1][0] - dv[0][1]]
    W = []
    for i in range(3):
        j, k = (i + 1) % 3, (i + 2) % 3
        W.append(4.0 * alpha * (d[j].real * d[k].imag - d[k].real * d[j].imag))
    g2 = _sum2(d)
    hess = [_grad(f) for f in d]                   # hess[j][i] = d_i d_j psi
    Jv = [sum((hess[j][i] * d[j].conj()).imag for j in range(3)) for i in range(3)]
    wn = torch.sqrt(sum(x * x for x in W))
    ok = (wn > 0) & (g2 > 1e-12 * g2.mean())
    one = torch.ones_like(wn)
    vpar = 2.0 * alpha * sum(a * b for a, b in zip(W, Jv)) / torch.where(ok, wn * g2, one)
    vr = [torch.where(ok, vpar * x / torch.where(ok, wn, one), 0.0 * one) for x in W]
    s, ns = _shells(shape), _nshell(shape)
    oh = [torch.fft.fftn(f) / pts for f in om]
    rows = []
    for u in (v, vr):
        rows.append(_binned(sum((torch.fft.fftn(f).conj() / pts * g).real for f, g in zip(u, oh)), s, ns))
    H = [float(sum((a * b).mean() for a, b in zip(u, om))) for u in (v, vr)]
    return {"H": H, "spec": torch.stack(rows).cpu().numpy()}


def _rvr_exact(case, seed):
    n = case["n"]
    pairs, xi = _pairs(case, seed)
    s201 = math.sqrt(201.0)
    a1, a2, b1 = (73.0 + 3.0 * s201) / 352.0, (6.0 + s201) / 528.0, (21.0 + s201) / 96.0
    g = (TWO_PI / n) * torch.arange(n, dtype=torch.float64, device=DEV)
    coords = (g[None, None, :], g[None, :, None], g[:, None, None])
    order = ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0))

    def ring(x, y, z, R):
        xt, yt, zt = x - math.pi, y - math.pi, z - math.pi
        dr = torch.sqrt(xt * xt + yt * yt) - R
        r2 = dr * dr + zt * zt
        e2 = r2 / (xi * xi)
        e4 = e2 * e2
        f = torch.sqrt((a1 * e2 + a2 * e4) / (1.0 + b1 * e2 + a2 * e4) / r2)
        return torch.complex(f * dr, f * zt)

    def pair(x, y, z, R, d):
        return ring(x, y, z - 0.5 * d, R) * ring(x, y, z + 0.5 * d, R).conj()

    psi = torch.ones((n, n, n), dtype=torch.complex128, device=DEV)
    L = 2.0 * TWO_PI
    for R, d, X, Y, Z, perm in pairs:
        o = order[perm]
        x, y, z = (torch.remainder(coords[o[i]] - c, TWO_PI) for i, c in enumerate((X, Y, Z)))
        psi = psi * pair(x, y, z, R, d)
        for im in ((L - x, y, z), (-x, y, z), (x, L - y, z), (x, -y, z), (x, y, L - z), (x, y, -z)):
            psi = psi * pair(*im, R, d).conj()
    return psi


def exact(case, seed):
    kind = case["kind"]
    if kind == "evolve":
        xyz = (case["nx"], case["ny"], case["nz"])
        alpha, beta = _coef(max(xyz))
        psi = _psi(xyz[::-1], case["ic"], case["prec"], seed).to(torch.complex128)
        psi = _evolved(psi, alpha, beta, _dt(max(xyz)), case["steps"])
        out = {"psi": psi}
        if case["diag"]:
            out["spec"], out["energies"] = _diagnostics(psi, alpha, beta)
        return out
    if kind == "ensemble":
        out = {"psi": [], "energies": []}
        for i, n in enumerate(_runs(case)):
            alpha, beta = _coef(n)
            psi = _psi((n, n, n), "srp", case["prec"], 1000 * int(seed) + i).to(torch.complex128)
            psi = _evolved(psi, alpha, beta, 1e-3, case["steps"])
            rho = psi.real ** 2 + psi.imag ** 2
            kz, ky, kx = _ks(psi.shape)
            c = torch.fft.fftn(psi) / psi.numel()
            e = 2.0 * alpha ** 2 * float(((kz * kz + ky * ky + kx * kx) * _sum2([c])).sum())
            out["psi"].append(psi)
            out["energies"].append([float(rho.mean()), e + alpha * beta * float(((rho - 1.0) ** 2).mean())])
        out["energies"] = np.array(out["energies"])
        return out
    if kind == "argle":
        return _argle_exact(case, seed)
    if kind == "adjoint":
        return _adjoint_exact(case, seed)
    if kind == "analysis":
        n = case["n"]
        alpha, beta = _coef(n)
        psi = _psi((n, n, n), "waves", case["prec"], seed).to(torch.complex128)
        spec, e = _diagnostics(psi, alpha, beta)
        rho = psi.real ** 2 + psi.imag ** 2
        S = sum(_lag_sums(rho - 1.0, ax) for ax in range(3)) / 3.0
        v = [2.0 * alpha * (psi.conj() * d).imag / rho for d in _grad(psi)]
        w2 = rho * sum(f * f for f in v)
        c = math.sqrt(2.0 * alpha * beta)
        return {"spec": spec, "energies": e, "rho": S,
                "vel": np.stack([_lag_sums(f, ax) for f, ax in zip(v, (2, 1, 0))]),
                "mean_v2": np.array([float((f * f).mean()) for f in v]),
                "mach": [math.sqrt(float(w2.max())) / c, math.sqrt(float(w2.mean())) / c]}
    if kind == "helicity":
        xyz = (case["nx"], case["ny"], case["nz"])
        psi = _psi(xyz[::-1], "tangle", case["prec"], seed).to(torch.complex128)
        return _helicity_exact(psi, _coef(max(xyz))[0])
    return _rvr_exact(case, seed)
