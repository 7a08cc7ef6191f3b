"""What the framework's speed is measured on: one call each of the public entry points, over the
range of sizes, filter lengths, velocity models and directions that a migration program has.

``listed`` names the cases, ``draw`` gives more of the same ranges, ``prepare`` makes the inputs on
the GPU from a seed, ``run`` is one call, ``work`` counts what the call cannot do without and
``exact`` is the same result in 64 bits from plain torch.
"""
from __future__ import annotations

import math
import random

import torch

from paper_1912_05529_amd import mig, synth

TWO_PI = 2.0 * math.pi
DX = DZ = 10.0
BAND_2D = (5.0, 55.0)          # Hz
BAND_3D = (5.0, 40.0)
PROP_2D = (750.0, 2400.0)      # propagation velocities the tables span, m/s
PROP_3D = (750.0, 2000.0)


def listed():
    return [
        # The smallest section of the benchmark (one scatterer under a constant velocity): one wave
        # per frequency, so the time is latency per depth step and launches.
        dict(name="section_small", kind="section", nx=128, nz=128, nw=64, ntaps=25, nk=512, vel="const"),
        # The benchmark's section: dipping layers and a body.
        dict(name="section_main", kind="section", nx=1024, nz=512, nw=200, ntaps=35, nk=2048, vel="layers"),
        # An odd-sized section in a smooth velocity (what tomography delivers): the filter differs
        # at every point and every depth.
        dict(name="section_smooth", kind="section", nx=601, nz=301, nw=97, ntaps=35, nk=2048, vel="smooth"),
        # A long line, past the widths that one workgroup holds at four points a thread.
        dict(name="section_long", kind="section", nx=3001, nz=300, nw=101, ntaps=35, nk=2048, vel="layers"),
        # A survey of uneven sections in one call (the benchmark's batch, fewer of them).
        dict(name="batch_uneven", kind="batch", nsec=16, nx_lo=256, nx_hi=2048, nz_lo=200, nz_hi=500,
             nw_lo=100, nw_hi=200, ntaps=35, nk=2048, vel="layers"),
        # The backward direction (demigration, gradients, least-squares migration) of the main section.
        dict(name="adjoint_main", kind="adjoint", nx=1024, nz=512, nw=200, ntaps=35, nk=2048, vel="layers"),
        # The backward direction of a longer line.
        dict(name="adjoint_long", kind="adjoint", nx=1501, nz=300, nw=101, ntaps=35, nk=2048, vel="layers"),
        # The benchmark's volume.
        dict(name="volume_main", kind="volume", nx=256, ny=256, nz=200, nw=128, ntaps=11, nk=1024, vel="layers"),
        # A small target volume of odd size: a few hundred microseconds' worth of small launches.
        dict(name="volume_small", kind="volume", nx=49, ny=75, nz=41, nw=25, ntaps=11, nk=256, vel="layers"),
        # A recorded t-x section to the migration frequencies (the benchmark's size).
        dict(name="transform_main", kind="transform", nx=1024, nt=1024, nw=200),
        # The filter table of the benchmark's section: once per survey and set of design options.
        dict(name="design_1d", kind="design", dims=1, ntaps=35, nk=2048),
        # The filter table of the benchmark's volume.
        dict(name="design_2d", kind="design", dims=2, ntaps=11, nk=1024),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["section", "section", "section", "batch", "adjoint", "adjoint", "volume", "volume",
                       "transform", "design"])
    if kind in ("section", "adjoint"):
        nx = _log_int(rng, 100, 4096 if kind == "section" else 2100)
        nz = _log_int(rng, 50, 512)
        most = 9.0e7 if kind == "section" else (9.0e7 if nx <= 1024 else 4.5e7)   # points x depths x frequencies
        nw = max(12, min(_log_int(rng, 16, 300), int(most / (nx * nz))))
        return dict(kind=kind, nx=nx, nz=nz, nw=nw, ntaps=rng.choice([19, 25, 35, 35, 45]),
                    nk=rng.choice([512, 2048]), vel=rng.choice(["const", "layers", "layers", "smooth"]))
    if kind == "batch":
        return dict(kind=kind, nsec=rng.randint(2, 12), nx_lo=rng.randint(100, 400), nx_hi=rng.randint(500, 2048),
                    nz_lo=rng.randint(50, 150), nz_hi=rng.randint(200, 400), nw_lo=rng.randint(20, 60),
                    nw_hi=rng.randint(80, 200), ntaps=rng.choice([25, 35]), nk=rng.choice([512, 2048]),
                    vel=rng.choice(["layers", "smooth"]))
    if kind == "volume":
        nx, ny = _log_int(rng, 24, 256), _log_int(rng, 24, 256)
        nz = _log_int(rng, 12, 150)
        nw = max(4, min(_log_int(rng, 8, 128), int(4.0e8 / (nx * ny * nz))))
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, nw=nw, ntaps=rng.choice([7, 9, 11, 11]), nk=rng.choice([256, 1024]),
                    vel=rng.choice(["const", "layers", "layers", "smooth"]))
    if kind == "transform":
        return dict(kind=kind, nx=_log_int(rng, 32, 3000), nt=_log_int(rng, 128, 4096), nw=_log_int(rng, 16, 300))
    if rng.random() < 0.5:
        return dict(kind=kind, dims=1, ntaps=rng.choice([19, 25, 35, 45]), nk=_log_int(rng, 64, 2048))
    return dict(kind=kind, dims=2, ntaps=rng.choice([7, 9, 11]), nk=_log_int(rng, 32, 1024))


# --------------------------------------------------------------------------- inputs
def _dev():
    return torch.device("cuda")


def _arange(n):
    return torch.arange(n, dtype=torch.float64, device=_dev())


def _gen(seed):
    return torch.Generator(device=_dev()).manual_seed(seed)


def _omega(nw, band):
    return torch.from_numpy(synth.omegas(nw, *band)).to(_dev())


def _layers(rng, x, z, y=None):
    """Medium velocity of 6-10 dipping interfaces and an elliptic body, z first."""
    X, Z = float(x[-1]) + DX, float(z[-1]) + DZ
    Y = float(y[-1]) + DX if y is not None else 0.0
    nl = rng.randint(6, 10)
    base = sorted(rng.uniform(0.05, 0.95) * Z for _ in range(nl))
    speeds = sorted(rng.uniform(1500.0, 4500.0 if y is None else 3500.0) for _ in range(nl + 1))
    zc = z[:, None] if y is None else z[:, None, None]
    xc = x[None, :] if y is None else x[None, :, None]
    layer = 0
    for b in base:
        depth = b + math.tan(math.radians(rng.uniform(-15.0, 15.0))) * (xc - X / 2)
        if y is not None:
            depth = depth + math.tan(math.radians(rng.uniform(-12.0, 12.0))) * (y[None, None, :] - Y / 2)
        layer = layer + (depth <= zc).long()
    v = torch.tensor(speeds, dtype=torch.float64, device=_dev())[layer]
    e = ((xc - rng.uniform(0.3, 0.7) * X) / (rng.uniform(0.08, 0.18) * X)) ** 2
    e = e + ((zc - rng.uniform(0.35, 0.65) * Z) / (rng.uniform(0.06, 0.15) * Z)) ** 2
    if y is not None:
        e = e + ((y[None, None, :] - rng.uniform(0.3, 0.7) * Y) / (rng.uniform(0.08, 0.18) * Y)) ** 2
    return torch.where(e <= 1.0, torch.full_like(v, 4800.0 if y is None else 4000.0), v)


def _smooth(rng, x, z, y=None):
    """Medium velocity growing with depth, with a few smooth anomalies."""
    X, Z = float(x[-1]) + DX, float(z[-1]) + DZ
    zc = z[:, None] if y is None else z[:, None, None]
    xc = x[None, :] if y is None else x[None, :, None]
    v = 1600.0 + (1600.0 / Z) * zc + 0.0 * xc
    if y is not None:
        v = v + 0.0 * y[None, None, :]
    for _ in range(5):
        r2 = ((xc - rng.uniform(0.0, 1.0) * X) / (rng.uniform(0.1, 0.3) * X)) ** 2
        r2 = r2 + ((zc - rng.uniform(0.0, 1.0) * Z) / (rng.uniform(0.1, 0.3) * Z)) ** 2
        if y is not None:
            Y = float(y[-1]) + DX
            r2 = r2 + ((y[None, None, :] - rng.uniform(0.0, 1.0) * Y) / (rng.uniform(0.1, 0.3) * Y)) ** 2
        v = v + rng.uniform(-120.0, 250.0) * torch.exp(-r2)
    return v.clamp(1500.0, 4000.0)


def _velocity(rng, kind, nx, nz, ny=None):
    """float32 propagation velocity (half the medium velocity)."""
    x, z = DX * _arange(nx), DZ * _arange(nz)
    y = None if ny is None else DX * _arange(ny)
    if kind == "const":
        v = torch.full((nz, nx) if ny is None else (nz, nx, ny), rng.uniform(1800.0, 2400.0), dtype=torch.float64, device=_dev())
    else:
        v = (_layers if kind == "layers" else _smooth)(rng, x, z, y)
    return (0.5 * v).float().contiguous()


def _amplitude(omega):
    """Amplitude spectrum of a 20 Hz Ricker wavelet, largest value 1."""
    f2 = (omega / TWO_PI / 20.0) ** 2
    return math.e * f2 * torch.exp(-f2)


def _surface(rng, gen, omega, nx, ny=None):
    """Surface wavefield: a dozen dipping arrivals and 5 % noise; [nx][nw], or [nw][nx][ny]."""
    nw = omega.numel()
    shape = (nx, nw) if ny is None else (nw, nx, ny)
    d = 0.05 * torch.randn(shape, dtype=torch.complex64, device=_dev(), generator=gen)
    amp = _amplitude(omega)
    for _ in range(12):
        px, t0 = rng.uniform(-4e-4, 4e-4), rng.uniform(0.0, 1.0)
        phase = amp * torch.exp(-1j * omega * t0) * rng.uniform(0.3, 1.0)
        ex = torch.exp(1j * (DX * px) * _arange(nx)[:, None] * omega[None, :])
        if ny is None:
            d += (ex * phase[None, :]).to(torch.complex64)
        else:
            py = rng.uniform(-4e-4, 4e-4)
            ey = torch.exp(1j * (DX * py) * omega[:, None] * _arange(ny)[None, :])
            d += (ex * phase[None, :]).t().to(torch.complex64)[:, :, None] * ey.to(torch.complex64)[:, None, :]
    return d.contiguous()


def _desc(case, jitter=None):
    dims = 2 if case["kind"] == "volume" or case.get("dims") == 2 else 1
    band, prop = (BAND_3D, PROP_3D) if dims == 2 else (BAND_2D, PROP_2D)
    step = DX if jitter is None else DX * jitter.uniform(0.95, 1.05)
    make = synth.table2d_for if dims == 2 else synth.table_for
    return make(case["ntaps"], case["nk"], band[0], band[1], prop[0], prop[1], step,
                DZ if jitter is None else DZ * jitter.uniform(0.95, 1.05))


def _section(case, rng, gen):
    omega = _omega(case["nw"], BAND_2D)
    return dict(vel=_velocity(rng, case["vel"], case["nx"], case["nz"]), omega=omega,
                data=_surface(rng, gen, omega, case["nx"]))


def _sections(case):
    """Sizes of a batch's sections: the case's own, whatever the seed."""
    rng = random.Random(3)
    return [dict(case, nx=rng.randint(case["nx_lo"], case["nx_hi"]), nz=rng.randint(case["nz_lo"], case["nz_hi"]),
                 nw=rng.randint(case["nw_lo"], case["nw_hi"])) for _ in range(case["nsec"])]


def _inputs(case, seed):
    rng, gen, kind = random.Random(seed), _gen(seed), case["kind"]
    if kind == "section":
        return _section(case, rng, gen)
    if kind == "batch":
        return [_section(c, rng, gen) for c in _sections(case)]
    if kind == "adjoint":
        vel = _velocity(rng, case["vel"], case["nx"], case["nz"])
        image = 0.02 * torch.randn(case["nz"], case["nx"], dtype=torch.float64, device=_dev(), generator=gen)
        image[1:] += (vel[1:] - vel[:-1]).double().sign()      # reflectors
        return dict(vel=vel, omega=_omega(case["nw"], BAND_2D), image=image)
    if kind == "volume":
        omega = _omega(case["nw"], BAND_3D)
        return dict(vel=_velocity(rng, case["vel"], case["nx"], case["nz"], case["ny"]), omega=omega,
                    data=_surface(rng, gen, omega, case["nx"], case["ny"]))
    if kind == "transform":
        nx, nt, dt = case["nx"], case["nt"], 0.004
        p = 0.05 * torch.randn(nx, nt, device=_dev(), generator=gen)
        t, x = dt * _arange(nt), DX * _arange(nx)
        for _ in range(8):
            t0 = torch.sqrt((rng.uniform(0.05, 0.9) * nt * dt) ** 2 + ((x - rng.uniform(0.0, 1.0) * nx * DX) / 1000.0) ** 2)
            a = (math.pi * 20.0 * (t[None, :] - t0[:, None])) ** 2
            p += ((1.0 - 2.0 * a) * torch.exp(-a)).float()
        return dict(section=p.contiguous(), dt=dt, omega=_omega(case["nw"], BAND_2D))
    return {}


def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind == "design":
        s.update(dims=case["dims"], desc=_desc(case, random.Random(seed)))
        return s
    x = _inputs(case, seed)
    if kind == "batch":
        s["batch"] = x
    else:
        s.update(x)
    if kind != "transform":
        s["desc"] = _desc(case)
        s["tab32"] = _table(s["desc"], 2 if kind == "volume" else 1)["tab64"].to(torch.complex64)
    return s


def run(s):
    kind = s["kind"]
    if kind == "section":
        return mig.migrate(s["data"], s["vel"], s["omega"], s["tab32"], s["desc"])
    if kind == "batch":
        return mig.migrate_batched(s["batch"], s["tab32"], s["desc"])
    if kind == "adjoint":
        return mig.demigrate(s["image"], s["vel"], s["omega"], s["tab32"], s["desc"])
    if kind == "volume":
        return mig.migrate3d(s["data"], s["vel"], s["omega"], s["tab32"], s["desc"])
    if kind == "transform":
        return mig.transform_t(s["section"], s["dt"], s["omega"])
    return (mig.design_table if s["dims"] == 1 else mig.design_table_2d)(s["desc"])


def work(case):
    """Inputs read once, outputs written once; the folded filters' operations."""
    kind = case["kind"]
    if kind == "batch":
        each = [work(dict(c, kind="section")) for c in _sections(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    if kind == "transform":
        nx, nt, nw = case["nx"], case["nt"], case["nw"]
        return {"bytes": 4 * nx * nt + 8 * nw + 8 * nx * nw, "flops": 4 * nx * nt * nw}
    M, nk = (case["ntaps"] - 1) // 2, case["nk"]
    flat = kind != "volume" and case.get("dims") != 2
    K = M + 1 if flat else (M + 1) * (M + 2) // 2
    if kind == "design":
        L, Lc = (1024, 8192) if flat else (48 * 48, 192 * 192)
        passes = 31      # one fit and 30 reweighted ones
        return {"bytes": nk * K * 24 + nk * 16,
                "flops": nk * (passes * (L * (K * (K + 1) + 4 * K) + K ** 3 / 3) + (passes - 1) * 4 * L * K + 4 * Lc * K)}
    points = case["nx"] * case.get("ny", 1)
    per = 8 * K + 2 * M if flat else 8 * K + 2 * (case["ntaps"] ** 2 - K)
    return {"bytes": 8 * points * case["nw"] + 12 * points * case["nz"] + 8 * case["nw"] + 8 * nk * K,
            "flops": points * case["nw"] * (case["nz"] - 1) * per}


# --------------------------------------------------------------------------- 64 bits
def _solve(G, B):
    """Symmetric positive definite systems, one per leading index: Gauss-Jordan elimination."""
    m = torch.cat([G, B], dim=2)
    for k in range(G.shape[1]):
        row = m[:, k, :] / m[:, k, k:k + 1]
        m = m - m[:, :, k:k + 1] * row[:, None, :]
        m[:, k, :] = row
    return m[:, :, G.shape[1]:]


def _basis(dims, M, *thetas):
    if dims == 1:
        n = _arange(M + 1)
        return torch.where(n == 0, 1.0, 2.0) * torch.cos(thetas[0][:, None] * n)
    n = _arange(M + 1)
    cx, cy = torch.cos(thetas[0][:, None] * n), torch.cos(thetas[1][:, None] * n)
    cols = []
    for a in range(M + 1):
        for b in range(a + 1):
            c = cx[:, a] * cy[:, b] if a == b else cx[:, a] * cy[:, b] + cx[:, b] * cy[:, a]
            cols.append((1.0 if a == 0 else 2.0 if b == 0 else 4.0) * c)
    return torch.stack(cols, 1)


def _table(d, dims):
    """The library's weighted least-squares design, for all entries at once."""
    M, nk, L = d.half, d.nk, d.ngrid
    grid = lambda n: (_arange(n) + 0.5) * math.pi / n  # noqa: E731
    if dims == 1:
        r2, A = grid(L) * grid(L), _basis(1, M, grid(L))
    else:
        tx, ty = grid(L).repeat_interleave(L), grid(L).repeat(L)
        r2, A = tx * tx + ty * ty, _basis(2, M, tx, ty)
    r, K = torch.sqrt(r2), A.shape[1]
    kappa = ((d.kmin + _arange(nk) * ((d.kmax - d.kmin) / (nk - 1))) * d.dx)[:, None]
    edge = kappa * math.sin(math.radians(d.theta_max_deg))
    zeta, q = d.dz / d.dx, kappa * kappa - r2
    root = zeta * torch.sqrt(q.abs())
    Dr, Di = torch.where(q >= 0, torch.cos(root), torch.exp(-root)), torch.where(q >= 0, torch.sin(root), 0.0)
    w = torch.where(r <= edge, d.w_pass, torch.where(r <= kappa, d.w_trans, d.w_evan)).double()
    pairs = (A[:, :, None] * A[:, None, :]).reshape(-1, K * K)
    eye = d.lam_value * torch.eye(K, dtype=torch.float64, device=_dev())
    for it in range(d.nreweight + 1):
        G = (w @ pairs).reshape(nk, K, K) + eye
        B = torch.stack([(w * Dr) @ A, (w * Di) @ A], 2)
        h = _solve(G, B)
        h = h + _solve(G, B - G @ h)
        if it < d.nreweight:
            over = torch.hypot(h[:, :, 0] @ A.t(), h[:, :, 1] @ A.t()) - 1.0
            w = torch.where(over > 0, w * (1.0 + d.beta * over / d.tau), w)
    c = math.cos(M * math.pi / (2.0 * d.ncheck))
    C = _basis(1, M, grid(d.ncheck)) if dims == 1 else None
    g = torch.empty(nk, dtype=torch.float64, device=_dev())
    if dims == 2:
        c, n = c * c, d.ncheck
        C = _basis(2, M, grid(n).repeat_interleave(n), grid(n).repeat(n))
    for j in range(0, nk, 256):
        hj = h[j:j + 256]
        g[j:j + 256] = torch.hypot(hj[:, :, 0] @ C.t(), hj[:, :, 1] @ C.t()).amax(1)
    lim = (1.0 - d.margin) * c
    s = torch.where(g > lim, lim / g, torch.ones_like(g))
    h = h * s[:, None, None]
    err = torch.hypot(h[:, :, 0] @ A.t() - Dr, h[:, :, 1] @ A.t() - Di)
    return {"tab64": torch.complex(h[:, :, 0], h[:, :, 1]).contiguous(), "maxgain": s * g,
            "passerr": torch.where(r <= edge, err, 0.0).amax(1)}


def _entries(omega, vel, d):
    """Table entry of every (frequency, point) of one depth row: nearest to omega / v."""
    dk = (d.kmax - d.kmin) / (d.nk - 1)
    u = (omega / dk)[:, None] * (1.0 / vel.double().reshape(-1))[None, :] - d.kmin / dk + 0.5
    return torch.floor(u).clamp(0, d.nk - 1).long()


def _exact_section(x, tab, d):
    M, nx = d.half, x["vel"].shape[1]
    P = x["data"].t().to(torch.complex128)
    rows = [P.real.sum(0)]
    fold = torch.arange(-M, M + 1, device=_dev()).abs()
    full = tab[:, fold]
    for k in range(x["vel"].shape[0] - 1):
        h = full[_entries(x["omega"], x["vel"][k], d)]                # [nw][nx][2M+1]
        P = (h * torch.nn.functional.pad(P, (M, M)).unfold(1, 2 * M + 1, 1)).sum(2)
        rows.append(P.real.sum(0))
    return torch.stack(rows).reshape(-1, nx)


def _exact_adjoint(x, tab, d):
    M, (nz, nx) = d.half, x["image"].shape
    Q = x["image"][nz - 1].to(torch.complex128)[None, :].repeat(x["omega"].numel(), 1)
    for k in range(nz - 2, -1, -1):
        h = tab[_entries(x["omega"], x["vel"][k], d)].conj()          # [nw][nx][M+1]
        g = torch.nn.functional.pad(h * Q[:, :, None], (0, 0, M, M))
        Q = x["image"][k].to(torch.complex128)[None, :] + g[:, M:M + nx, 0]
        for m in range(1, M + 1):
            Q = Q + g[:, M + m:M + m + nx, m] + g[:, M - m:M - m + nx, m]
    return Q.t().contiguous()


def _exact_volume(x, tab, d):
    M, (nz, nx, ny), nw = d.half, x["vel"].shape, x["omega"].numel()
    P = x["data"].to(torch.complex128)
    out = torch.empty(nz, nx, ny, dtype=torch.float64, device=_dev())
    out[0] = P.real.sum(0)
    for k in range(1, nz):
        j = _entries(x["omega"], x["vel"][k - 1], d)
        pad = torch.nn.functional.pad(P, (M, M, M, M))
        at = lambda p, q: pad[:, M + p:M + p + nx, M + q:M + q + ny]  # noqa: E731
        P = torch.zeros_like(P)
        u = 0
        for a in range(M + 1):
            for b in range(a + 1):
                taps = sorted({(s * p, t * q) for p, q in ((a, b), (b, a)) for s in (1, -1) for t in (1, -1)})
                S = at(*taps[0]).clone()
                for p, q in taps[1:]:
                    S += at(p, q)
                P += tab[:, u][j].reshape(nw, nx, ny) * S
                u += 1
        out[k] = P.real.sum(0)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "design":
        t = _table(_desc(case, random.Random(seed)), case["dims"])
        return dict(t, tab32=t["tab64"])
    x = _inputs(case, seed)
    if kind == "transform":
        a = x["dt"] * _arange(case["nt"])[:, None] * x["omega"][None, :]
        p = x["section"].double()
        return torch.complex(p @ torch.cos(a), -(p @ torch.sin(a)))
    d = _desc(case)
    tab = _table(d, 2 if kind == "volume" else 1)["tab64"].to(torch.complex64).to(torch.complex128)
    if kind == "batch":
        return [_exact_section(q, tab, d) for q in x]
    return {"section": _exact_section, "adjoint": _exact_adjoint, "volume": _exact_volume}[kind](x, tab, d)
