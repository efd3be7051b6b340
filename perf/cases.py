"""Performance cases of the advection library: one pass of each is a piece of work that a
program built on it does, through the package's public entry points.

A case is a dict of plain values; its ``kind`` says which program it stands for:

``hour``       an interactive loop on a small flat basin: one hour more, then the positions
``global2d``   a lon/lat eddy field with land, periodic in time: release, advect, read back
               (RK4, Euler, adaptive RKF45, Brownian, tracer sampling, 16-bit storage)
``ensemble``   many uneven flat runs with a Brownian term, advanced as one batch
``ocean3d``    a global 3D field streamed through the three-slot ring: advect a day while
               the next snapshot is converted
``footprint``  sinking, ageing, tracer-sampling particles traced backward in time
``train``      one optimiser step of the flow-map network on a host batch
``infer``      the flow-map network advancing particles with RK4 as the arbiter

Inputs are made on the GPU from the seed alone (random streamfunctions with the eddy sizes,
speeds and land fraction of the benchmark's workloads).  ``exact`` evaluates the same method
in plain torch in 64 bits.
"""

from __future__ import annotations

import math

import numpy as np
import torch

DAY = 86400.0
METRES = 111120.0  # metres per degree of arc
SIZES = (64, 256, 256, 256, 256, 2)


# ------------------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest call: a small basin in FP64, one hour at a time on a kept set
        dict(name="hour_10k", kind="hour", side=101, n=10_000, steps=60, dt=60.0),
        # the 0.25 degree global field, a million particles, ten days, records of every tenth
        dict(name="eddies_1m", kind="global2d", nx=1440, ny=720, nt=30, n=1_000_000, days=10,
             dt=300.0, dtype="f32", kernel="rk4", Kh=0.0, sample=False, cache=True, stride=10,
             sort_every=10),
        # a regional release: few particles, two days, an odd count, scaled FP16 storage
        dict(name="release_30k_f16s", kind="global2d", nx=721, ny=363, nt=10, n=30_011, days=2,
             dt=300.0, dtype="f16s", kernel="rk4", Kh=0.0, sample=False, cache=True, stride=1,
             sort_every=1),
        # adaptive steps, one millimetre a step, five days
        dict(name="adaptive_1m", kind="global2d", nx=1440, ny=720, nt=30, n=1_000_000, days=5,
             dt=300.0, dtype="f32", kernel="rkf45", Kh=0.0, sample=False, cache=False, stride=0,
             sort_every=1),
        # sub-grid diffusion on the sphere
        dict(name="diffusive_500k", kind="global2d", nx=1440, ny=720, nt=10, n=500_009, days=4,
             dt=300.0, dtype="f32", kernel="rk4", Kh=10.0, sample=False, cache=True, stride=0,
             sort_every=1),
        # temperature sampled along surface trajectories at every step
        dict(name="sampled_400k", kind="global2d", nx=1440, ny=720, nt=10, n=400_000, days=2,
             dt=600.0, dtype="f32", kernel="rk4", Kh=0.0, sample=True, cache=True, stride=4,
             sort_every=1),
        # uneven ensemble, 64 to 1024 cells a side, a thousand to a million particles a run,
        # three days
        dict(name="ensemble_24", kind="ensemble", runs=24, side_min=64, side_max=1024,
             n_min=1000, n_max=1_000_000, days=3, dt=300.0, Kh=10.0),
        # the 0.1 degree, 50-level global field, ten million particles, five days with
        # daily records of every hundredth, the positions of all of them at the end
        dict(name="ocean_10m", kind="ocean3d", nx=3600, ny=1800, nz=50, n=10_000_000, days=5,
             dt=600.0, dtype="f32", stride=100),
        # a 0.25 degree, 40-level field in bfloat16, odd sizes, two days
        dict(name="ocean_2m_bf16", kind="ocean3d", nx=1441, ny=719, nz=40, n=2_000_003, days=2,
             dt=600.0, dtype="bf16", stride=25),
        # the worked example: 54 levels, backward from the sea floor to the dwelling depth
        dict(name="footprint_200k", kind="footprint", nx=350, ny=300, nz=54, n=200_000,
             days=13, dt=300.0),
        # one optimiser step on the benchmark's batch
        dict(name="train_4096", kind="train", batch=4096),
        # half a day of two-hour network segments
        dict(name="infer_1m", kind="infer", nx=1440, ny=720, nt=10, n=1_000_000, segments=6,
             residual=50.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["hour", "global2d", "global2d", "global2d", "ensemble", "ocean3d",
                       "ocean3d", "footprint", "train", "infer"])
    if kind == "hour":
        return dict(kind=kind, side=_log_int(rng, 33, 801), n=_log_int(rng, 500, 200_000),
                    steps=rng.choice([1, 12, 60, 61, 240]), dt=60.0)
    if kind == "global2d":
        nx = _log_int(rng, 300, 1440)
        flavour = rng.choice(["plain", "plain", "rkf45", "euler", "brown", "sample"])
        n = _log_int(rng, 2_000, 400_000 if flavour in ("sample", "brown") else 1_000_000)
        return dict(kind=kind, nx=nx, ny=max(180, nx // 2 + rng.randint(-2, 2)),
                    nt=rng.choice([5, 10, 30]), n=n, days=rng.randint(1, 3),
                    dt=rng.choice([300.0, 600.0]),
                    dtype=rng.choice(["f32", "f32", "f64", "bf16", "f16s"])
                    if flavour in ("plain", "brown") else "f32",
                    kernel={"rkf45": "rkf45", "euler": "euler"}.get(flavour, "rk4"),
                    Kh=rng.choice([1.0, 10.0, 50.0]) if flavour == "brown" else 0.0,
                    sample=flavour == "sample", cache=flavour != "rkf45",
                    stride=0 if flavour == "rkf45" else rng.choice([0, 1, 7, 10]),
                    sort_every=rng.choice([0, 1, 10]))
    if kind == "ensemble":
        return dict(kind=kind, runs=rng.randint(2, 24), side_min=64,
                    side_max=_log_int(rng, 128, 1024), n_min=1000,
                    n_max=_log_int(rng, 20_000, 1_000_000), days=1, dt=300.0,
                    Kh=rng.choice([0.0, 1.0, 10.0]))
    if kind == "ocean3d":
        nx = _log_int(rng, 360, 3600)
        return dict(kind=kind, nx=nx, ny=nx // 2 + rng.randint(-1, 1), nz=rng.randint(10, 50),
                    n=_log_int(rng, 20_000, 6_000_000), days=1, dt=600.0,
                    dtype=rng.choice(["f32", "f32", "bf16", "f16s"]),
                    stride=rng.choice([10, 33, 100]))
    if kind == "footprint":
        return dict(kind=kind, nx=rng.randint(150, 350), ny=rng.randint(150, 300),
                    nz=rng.randint(30, 54), n=_log_int(rng, 5_000, 200_000),
                    days=rng.randint(3, 14), dt=300.0)
    if kind == "train":
        return dict(kind=kind, batch=128 * rng.randint(1, 64))
    nx = _log_int(rng, 400, 1440)
    return dict(kind=kind, nx=nx, ny=nx // 2, nt=rng.choice([5, 10]),
                n=_log_int(rng, 20_000, 1_000_000), segments=rng.randint(2, 6),
                residual=rng.choice([10.0, 50.0, 100.0]))


def work(case):
    """Bytes: positions in and out, records, the field values of the cells that particles can
    be in (each snapshot read once); flops: the method's own count in 64 bits (cosines
    excluded), or the network's products."""
    k = case["kind"]
    if k == "hour":
        n, s = case["n"], case["side"]
        return dict(bytes=40.0 * n + 16.0 * s * s, flops=194.0 * n * case["steps"])
    if k == "global2d":
        n, steps = case["n"], case["days"] * DAY / case["dt"]
        snaps = min(case["nt"], case["days"] + 1)
        node = {"f64": 16, "f32": 8}.get(case["dtype"], 4)
        rec = (case["days"] + 1) * 25.0 * (n // case["stride"]) if case["stride"] else 0.0
        flops = 230.0 if case["kernel"] == "rk4" else 60.0
        if case["kernel"] == "rkf45":  # about eleven attempts a day
            flops, steps = 448.0, 11.0 * case["days"]
        if case["Kh"] > 0:
            flops += 9.0
        if case["sample"]:
            flops += 20.0
        return dict(bytes=41.0 * n + rec + float(node) * case["nx"] * case["ny"] * snaps,
                    flops=flops * n * steps)
    if k == "ensemble":
        tot, cells = 0, 0
        for side, n in _ensemble_sizes(case):
            tot, cells = tot + n, cells + side * side
        steps = case["days"] * DAY / case["dt"]
        return dict(bytes=41.0 * tot + 16.0 * cells,
                    flops=(210.0 + (9.0 if case["Kh"] > 0 else 0.0)) * tot * steps)
    if k == "ocean3d":
        n, steps = case["n"], case["days"] * DAY / case["dt"]
        nodes = float(case["nx"]) * case["ny"] * case["nz"]
        node = 16 if case["dtype"] == "f32" else 8
        rec = (case["days"] + 1) * 37.0 * (n // case["stride"])
        # the pushed snapshots are read and their slots written; two are sampled a day
        return dict(bytes=60.0 * n + rec + nodes * (12 + node) * case["days"],
                    flops=567.0 * n * steps)
    if k == "footprint":
        n, steps = case["n"], case["days"] * DAY / case["dt"]
        return dict(bytes=92.0 * n * (case["days"] + 1), flops=607.0 * n * steps)
    mac = sum(a * b for a, b in zip(SIZES[:-1], SIZES[1:]))
    if k == "train":
        p = mac + sum(SIZES[1:])
        return dict(bytes=case["batch"] * 66 * 4.0 + 28.0 * p, flops=6.0 * mac * case["batch"])
    n, segs = case["n"], case["segments"]
    return dict(bytes=41.0 * n, flops=(2.0 * mac + 2 * 230.0 + 0.2 * 24 * 230.0) * n * segs)


# --------------------------------------------------------------------------- input fields
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, n, lo, hi):
    return torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (hi - lo) + lo


def _streamfunction(g, ny, nx, kappa0):
    """Random field with a kappa^-3 spectrum above kappa0 cycles per cell, unit maximum."""
    ky = torch.fft.fftfreq(ny, device="cuda", dtype=torch.float64)[:, None]
    kx = torch.fft.rfftfreq(nx, device="cuda", dtype=torch.float64)[None, :]
    k = torch.sqrt(kx * kx + ky * ky)
    amp = torch.where(k > 0, torch.clamp(k, min=1e-12) ** -3.0, torch.zeros_like(k))
    amp = torch.where((k > 0) & (k < kappa0), amp * (k / kappa0) ** 2, amp)
    ph = torch.rand(k.shape, generator=g, device="cuda", dtype=torch.float64) * (2 * math.pi)
    psi = torch.fft.irfft2(torch.polar(amp, ph), s=(ny, nx))
    return psi / psi.abs().max()


def _velocity(psi, lat=None):
    dy, dx = torch.gradient(psi)
    u, v = -dy, dx
    if lat is not None:
        c = torch.cos(torch.deg2rad(torch.from_numpy(lat).cuda()))[:, None]
        u, v = u * c, v * c
    return u, v


def _eddies(g, ny, nx, cell_m, lat=None, speed=1.0):
    """Two velocity fields of 200 km eddies, their cosine/sine mix at most `speed`."""
    out = []
    for _ in range(2):
        u, v = _velocity(_streamfunction(g, ny, nx, cell_m / 200e3), lat)
        s = speed / (math.sqrt(2.0) * torch.sqrt(u * u + v * v).max())
        out += [u * s, v * s]
    return out


def _global_axes(nx, ny):
    return (-180.0 + (np.arange(nx) + 0.5) * (360.0 / nx),
            -90.0 + (np.arange(ny) + 0.5) * (180.0 / ny))


def _land(g, ny, nx):
    """30% land in blobs of a few cells (node mask on the GPU)."""
    noise = torch.randn(ny, nx, generator=g, device="cuda", dtype=torch.float64)
    ky = torch.fft.fftfreq(ny, device="cuda", dtype=torch.float64)[:, None]
    kx = torch.fft.rfftfreq(nx, device="cuda", dtype=torch.float64)[None, :]
    f = torch.exp(-2.0 * (math.pi * 4.0) ** 2 * (kx * kx + ky * ky))
    sm = torch.fft.irfft2(torch.fft.rfft2(noise) * f, s=(ny, nx))
    thr = torch.sort(sm.reshape(-1)).values[int(0.7 * sm.numel())]
    return sm > thr


def _in_ocean(g, land, n, lon, lat):
    oc = ~(land[:-1, :-1] | land[:-1, 1:] | land[1:, :-1] | land[1:, 1:])
    cells = torch.nonzero(oc.reshape(-1)).reshape(-1)
    c = cells[torch.randint(cells.numel(), (n,), generator=g, device="cuda")]
    w = land.shape[1] - 1
    j, i = torch.div(c, w, rounding_mode="floor"), c % w
    lon, lat = torch.from_numpy(lon).cuda(), torch.from_numpy(lat).cuda()
    x = lon[i] + _uniform(g, n, 0.0, 1.0) * (lon[i + 1] - lon[i])
    y = lat[j] + _uniform(g, n, 0.0, 1.0) * (lat[j + 1] - lat[j])
    return x, y


def _inputs_hour(case, seed):
    g = _gen(seed)
    axis = 1000.0 * np.arange(case["side"], dtype=np.float64)
    mid = axis[-1] / 2
    x = torch.from_numpy(axis).cuda()
    U = (-1e-5 * (x - mid))[:, None].expand(x.numel(), x.numel())
    V = (1e-5 * (x - mid))[None, :].expand(x.numel(), x.numel())
    r = 0.8 * mid * torch.sqrt(_uniform(g, case["n"], 0.0, 1.0))
    ph = _uniform(g, case["n"], 0.0, 2 * math.pi)
    return dict(lon=axis, lat=axis.copy(), depth=None, land=None, spherical=False, period=0.0,
                times=[0.0], fields=[(U.contiguous(), V.contiguous(), None)],
                x=mid + r * torch.cos(ph), y=mid + r * torch.sin(ph), z=None, t0=0.0)


def _inputs_global2d(case, seed):
    g = _gen(seed)
    nx, ny, nt = case["nx"], case["ny"], case["nt"]
    lon, lat = _global_axes(nx, ny)
    ua, va, ub, vb = _eddies(g, ny, nx, 360.0 / nx * METRES, lat)
    land = _land(g, ny, nx)
    period, fields, tracer = nt * DAY, [], []
    for s in range(nt):
        c, sn = math.cos(2 * math.pi * s / nt), math.sin(2 * math.pi * s / nt)
        U, V = (c * ua + sn * ub).float(), (c * va + sn * vb).float()
        U[land], V[land] = 0.0, 0.0
        fields.append((U, V, None))
    if case.get("sample"):
        A = _streamfunction(g, ny, nx, 360.0 / nx * METRES / 200e3)
        base = 28.0 * torch.cos(torch.deg2rad(torch.from_numpy(lat).cuda()))[:, None]
        tracer = [(base + 2.0 * math.cos(2 * math.pi * s / nt) * A).float() for s in range(nt)]
    x, y = _in_ocean(g, land, case["n"], lon, lat)
    return dict(lon=lon, lat=lat, depth=None, land=land, spherical=True, period=period,
                times=[DAY * s for s in range(nt)], fields=fields, tracer=tracer, x=x, y=y,
                z=None, t0=0.0)


def _levels(nz, bottom):
    return 5.0 * (bottom / 5.0) ** (np.arange(nz) / (nz - 1.0))


def _stack3d(g, ny, nx, z, cell_m, lat, speed, wmax, days, tracer=False):
    """U, V, W (and a temperature) on the given days: eddies decaying and turning with depth."""
    ua, va, ub, vb = (a.float() for a in _eddies(g, ny, nx, cell_m, lat, speed))
    C = _streamfunction(g, ny, nx, cell_m / 200e3).float()
    fields, temps = [], []
    for t in days:
        wt = 2 * math.pi * t / 30.0
        U = torch.empty((z.size, ny, nx), dtype=torch.float32, device="cuda")
        V, W = torch.empty_like(U), torch.empty_like(U)
        T = torch.empty_like(U) if tracer else None
        for k in range(z.size):
            d = math.exp(-z[k] / 1500.0)
            c, s = d * math.cos(wt + z[k] / 800.0), d * math.sin(wt + z[k] / 800.0)
            torch.add(ua * c, ub, alpha=s, out=U[k])
            torch.add(va * c, vb, alpha=s, out=V[k])
            w = wmax * math.sin(math.pi * (z[k] - z[0]) / (z[-1] - z[0])) * math.cos(wt)
            torch.mul(C, w, out=W[k])
            if tracer:
                T[k] = (18.0 - 14.0 * (1 - math.exp(-z[k] / 600.0))
                        + 1.5 * math.exp(-z[k] / 300.0) * math.cos(wt) * C)
        fields.append((U, V, W))
        temps.append(T)
    return fields, temps


def _inputs_ocean3d(case, seed):
    g = _gen(seed)
    lon, lat = _global_axes(case["nx"], case["ny"])
    z = _levels(case["nz"], 5000.0)
    fields, _ = _stack3d(g, case["ny"], case["nx"], z, 360.0 / case["nx"] * METRES, lat, 1.0,
                         1e-4, [0, 1, 2])
    n = case["n"]
    return dict(lon=lon, lat=lat, depth=z, land=None, spherical=True, period=0.0,
                times=[0.0, DAY, 2 * DAY], fields=fields, x=_uniform(g, n, lon[0], lon[-1]),
                y=_uniform(g, n, lat[0], lat[-1]), z=_uniform(g, n, z[0], z[-1]), t0=0.0)


def _inputs_footprint(case, seed):
    g = _gen(seed)
    lon, lat = np.linspace(5.0, 40.0, case["nx"]), np.linspace(-50.0, -20.0, case["ny"])
    z = _levels(case["nz"], 5500.0)
    days = list(range(0, case["days"] + 3, 3))
    fields, temps = _stack3d(g, case["ny"], case["nx"], z, 35.0 / (case["nx"] - 1) * METRES, lat,
                             0.8, 5e-5, days, tracer=True)
    n = case["n"]
    return dict(lon=lon, lat=lat, depth=z, land=None, spherical=True, period=0.0,
                times=[DAY * d for d in days], fields=fields, tracer=temps,
                x=17.3 + _uniform(g, n, -0.05, 0.05), y=-34.7 + _uniform(g, n, -0.05, 0.05),
                z=torch.full((n,), 2440.0, device="cuda", dtype=torch.float64),
                t0=DAY * days[-1])


def _ensemble_sizes(case):
    """Sides and counts spread evenly in the logarithm, large grids not tied to large sets."""
    R = case["runs"]
    out = []
    for r in range(R):
        a, b = r / max(R - 1, 1), ((r * 7 + 3) % R) / max(R - 1, 1)
        out.append((int(round(case["side_min"] * (case["side_max"] / case["side_min"]) ** a)),
                    int(round(case["n_min"] * (case["n_max"] / case["n_min"]) ** b))))
    return out


def _inputs_ensemble(case, seed):
    g = _gen(seed)
    out = []
    for side, n in _ensemble_sizes(case):
        axis = 1e4 * np.arange(side, dtype=np.float64)
        ua, va, ub, vb = _eddies(g, side, side, 1e4)
        fields = []
        for s in range(5):
            c, sn = math.cos(2 * math.pi * s / 5), math.sin(2 * math.pi * s / 5)
            fields.append(((c * ua + sn * ub).float(), (c * va + sn * vb).float(), None))
        out.append(dict(lon=axis, lat=axis.copy(), depth=None, land=None, spherical=False,
                        period=5 * DAY, times=[DAY * s for s in range(5)], fields=fields,
                        x=_uniform(g, n, axis[0], axis[-1]), y=_uniform(g, n, axis[0], axis[-1]),
                        z=None, t0=0.0))
    return out


def _inputs_train(case, seed):
    """Feature-like rows (position, phase, a 5x5 velocity patch, offsets) and displacements."""
    r = np.random.default_rng(seed)
    B = case["batch"]
    X = np.zeros((B, 64), np.float32)
    X[:, 0:2] = r.uniform(-1, 1, (B, 2))
    X[:, 2], X[:, 3] = np.sin(0.7), np.cos(0.7)
    uv = r.normal(0.0, 0.2, (B, 2))
    X[:, 4:54] = np.tile(uv, 25) + r.normal(0.0, 0.05, (B, 50))
    X[:, 54:56] = r.uniform(-0.5, 0.5, (B, 2))
    X[:, 56:58] = uv
    X[:, 58:60] = r.uniform(0.3, 0.95, (B, 2))
    T = (uv * 0.98 + r.normal(0.0, 0.01, (B, 2))).astype(np.float32)
    params = [(r.normal(0.0, math.sqrt(2.0 / a), (a, b)).astype(np.float32),
               r.normal(0.0, 0.01, b).astype(np.float32))
              for a, b in zip(SIZES[:-1], SIZES[1:])]
    return X, T, params


def _passthrough_params(seed):
    """A network whose output is the velocity at the particle (features 56 and 57), carried
    through the layers as gelu(x) - gelu(-x) = x, with small random weights on every other
    unit: it agrees with RK4 to some tens of metres a segment, as a trained one does."""
    r = np.random.default_rng(seed)
    params = []
    for l, (a, b) in enumerate(zip(SIZES[:-1], SIZES[1:])):
        W = r.normal(0.0, 0.3 / math.sqrt(a), (a, b)).astype(np.float32)
        bias = r.normal(0.0, 0.01, b).astype(np.float32)
        if l < 4:
            W[:, 0:4] = 0.0
            bias[0:4] = 0.0
            for q in range(2):
                src = [56 + q] if l == 0 else [2 * q, 2 * q + 1]
                for s, sign in zip(src, (1.0, -1.0)):
                    W[s, 2 * q], W[s, 2 * q + 1] = sign, -sign
        else:
            W *= 0.005
            W[0:4, :] = 0.0
            bias[:] = 0.0
            for q in range(2):
                W[2 * q, q], W[2 * q + 1, q] = 1.0, -1.0
        params.append((W, bias))
    return params


# ----------------------------------------------------------------------- prepare and run
def _fieldset(inp, dtype, capacity=None):
    from paper_1707_05163_amd import FieldSet
    land = inp["land"]
    land = None if land is None else land.to(torch.uint8).cpu().numpy()
    cap = len(inp["times"]) if capacity is None else capacity
    fs = FieldSet(inp["lon"], inp["lat"], inp["depth"],
                  "spherical" if inp["spherical"] else "flat", dtype, cap, inp["period"], land)
    for s in range(min(cap, len(inp["times"])) if capacity is None else capacity - 1):
        U, V, W = inp["fields"][s]
        if dtype == "f64" and U.dtype == torch.float64:
            fs.push_snapshot(inp["times"][s], U.cpu().numpy(), V.cpu().numpy())
        else:
            fs.push_snapshot(inp["times"][s], U, V, W)
        if inp.get("tracer"):
            fs.push_tracer(inp["times"][s], inp["tracer"][s])
    torch.cuda.synchronize()
    return fs


def prepare(case, seed):
    from paper_1707_05163_amd import ParticleSet, Surrogate
    k = case["kind"]
    st = dict(case=case)
    if k == "hour":
        inp = _inputs_hour(case, seed)
        st["fs"] = _fieldset(inp, "f64")
        st["ps"] = ParticleSet(st["fs"], inp["x"], inp["y"])
        torch.cuda.synchronize()
    elif k in ("global2d", "infer"):
        inp = _inputs_global2d(case, seed)
        st["fs"] = _fieldset(inp, case.get("dtype", "f32"))
        st["x"], st["y"] = inp["x"], inp["y"]
        if k == "infer":
            st["model"] = Surrogate(seed=1)
            st["model"].set_params(_passthrough_params(seed))
    elif k == "ensemble":
        inps = _inputs_ensemble(case, seed)
        st["fs"] = [_fieldset(i, "f32") for i in inps]
        st["start"] = [(i["x"], i["y"]) for i in inps]
        st["opts"] = [ParticleSet.opts(Kh=case["Kh"], run_id=r) for r in range(len(inps))]
    elif k == "ocean3d":
        inp = _inputs_ocean3d(case, seed)
        st["fs"] = _fieldset(inp, case["dtype"], capacity=3)
        st["source"], st["day"] = inp["fields"], 0
        st["start"] = (inp["x"], inp["y"], inp["z"])
    elif k == "footprint":
        inp = _inputs_footprint(case, seed)
        st["fs"] = _fieldset(inp, "f32")
        st["start"], st["t0"] = (inp["x"], inp["y"], inp["z"]), inp["t0"]
    else:
        st["X"], st["T"], params = _inputs_train(case, seed)
        st["model"] = Surrogate(seed=1)
        st["model"].set_params(params)
    return st


def _result(ps, records):
    counts, status = ps.status()
    out = dict(final=ps.get(), status=status, steps=counts["particle_steps"])
    if records:
        out["records"] = ps.records()
    return out


def run(st):
    from paper_1707_05163_amd import ParticleSet, execute_batch
    c, k = st["case"], st["case"]["kind"]
    if k == "hour":
        st["ps"].execute(c["steps"] * c["dt"], c["dt"])
        return st["ps"].get()
    if k == "global2d":
        ps = ParticleSet(st["fs"], st["x"], st["y"])
        ps.execute(c["days"] * DAY, c["dt"], DAY, kernel=c["kernel"], Kh=c["Kh"], run_id=3,
                   tol=1e-3, min_exp=-6, max_exp=5, stencil_cache=c["cache"],
                   sample=c["sample"], output_stride=c["stride"], sort_every=c["sort_every"])
        out = _result(ps, c["stride"] > 0)
        if c["kernel"] == "rkf45":
            out["exponents"] = ps.step_exponents()
        ps.close()
        return out
    if k == "ensemble":
        sets = [ParticleSet(f, x, y) for f, (x, y) in zip(st["fs"], st["start"])]
        execute_batch(sets, c["days"] * DAY, c["dt"], DAY, st["opts"])
        out = [_result(p, False) for p in sets]
        for p in sets:
            p.close()
        # one array per quantity: the runs end to end
        return dict(lon=np.concatenate([o["final"]["lon"] for o in out]),
                    lat=np.concatenate([o["final"]["lat"] for o in out]),
                    ci=np.concatenate([o["final"]["ci"] for o in out]),
                    cj=np.concatenate([o["final"]["cj"] for o in out]),
                    status=np.concatenate([o["status"] for o in out]))
    if k == "ocean3d":
        x, y, z = st["start"]
        ps = ParticleSet(st["fs"], x, y, z, t0=st["day"] * DAY)
        for _ in range(c["days"]):
            ps.execute(DAY, c["dt"], DAY, output_stride=c["stride"], sort_every=0)
            d = st["day"] + 2  # the next time slice loads while this day is advected
            st["fs"].push_snapshot(d * DAY, *st["source"][d % 3], stream=0)
            st["day"] += 1
        out = _result(ps, True)
        ps.close()
        return out
    if k == "footprint":
        x, y, z = st["start"]
        ps = ParticleSet(st["fs"], x, y, z, t0=st["t0"])
        ps.execute(c["days"] * DAY, -c["dt"], DAY, output_stride=1, sink_speed=200.0 / DAY,
                   dwell_depth=50.0, maxage=30 * DAY, sample=True, sort_every=0)
        out = _result(ps, True)
        ps.close()
        return out
    if k == "train":
        loss = st["model"].train_step(st["X"], st["T"], 1e-3)
        return dict(loss=np.float32(loss), params=st["model"].get_params())
    ps = ParticleSet(st["fs"], st["x"], st["y"])
    stats = ps.execute_surrogate(st["model"], c["segments"] * 7200.0, 300.0, 24, c["residual"])
    out = dict(final=ps.get(), status=ps.status()[1], accepted=int(stats["accepted"]),
               fallback=int(stats["fallback"]))
    ps.close()
    return out


# ---------------------------------------------------------------------- exact: 64 bits
class _Reference:
    """The method in plain torch, FP64: cell search, multilinear interpolation, linear in
    time, metres to degrees on the sphere, RK4 / Euler / Fehlberg, status bits."""

    def __init__(self, inp, dtype="f32"):
        self.ax = [torch.from_numpy(np.asarray(a, np.float64)).cuda()
                   for a in (inp["lon"], inp["lat"], inp["depth"]) if a is not None]
        self.nd, self.spherical = len(self.ax), inp["spherical"]
        self.period, self.times = inp["period"], list(inp["times"])
        self.F = []
        for U, V, W in inp["fields"][:len(self.times)]:
            f = torch.stack([a for a in (U, V, W) if a is not None], dim=-1)
            self.F.append(self._stored(f, dtype).reshape(-1, f.shape[-1]))
        self.T = [t.reshape(-1) for t in inp.get("tracer") or []]
        L = inp["land"]
        self.land = None if L is None else (L[:-1, :-1] & L[:-1, 1:] & L[1:, :-1] & L[1:, 1:])

    @staticmethod
    def _stored(f, dtype):
        """The values that a 16-bit snapshot holds (a power-of-two scale per level in FP16)."""
        if dtype == "bf16":
            return f.bfloat16().float()
        if dtype == "f16s":
            dims = (0, 1) if f.dim() == 3 else (1, 2)
            m = f.abs().amax(dim=dims, keepdim=True).double()
            s = torch.where(m > 0, torch.exp2(torch.ceil(torch.log2(torch.clamp(m, min=1e-300)))
                                              - 14), torch.ones_like(m)).float()
            return (f / s).half().float() * s
        return f

    def bracket(self, t):
        T, P = self.times, self.period
        if len(T) == 1:
            return 0, 0, 0.0
        if P > 0:
            t = T[0] + math.fmod(math.fmod(t - T[0], P) + P, P)
            s = max(k for k in range(len(T)) if T[k] <= t)
            up = T[s + 1] if s + 1 < len(T) else T[0] + P
            return s, (s + 1) % len(T), (t - T[s]) / (up - T[s])
        s = max(k for k in range(len(T) - 1) if T[k] <= t)
        return s, s + 1, (t - T[s]) / (T[s + 1] - T[s])

    def locate(self, p):
        idx, frac, ok = [], [], None
        for a, x in zip(self.ax, p):
            i = torch.clamp(torch.searchsorted(a, x, right=True) - 1, 0, a.numel() - 2)
            good = (x >= a[0]) & (x <= a[-1])
            ok = good if ok is None else ok & good
            idx.append(i)
            frac.append((x - a[i]) / (a[i + 1] - a[i]))
        return idx, frac, ok

    def corners(self, idx, frac):
        nx, ny = self.ax[0].numel(), self.ax[1].numel()
        base = idx[1] * nx + idx[0]
        if self.nd == 3:
            base = base + idx[2] * (nx * ny)
        out = []
        for dk in range(2 if self.nd == 3 else 1):
            for dj in range(2):
                for di in range(2):
                    w = (frac[0] if di else 1 - frac[0]) * (frac[1] if dj else 1 - frac[1])
                    if self.nd == 3:
                        w = w * (frac[2] if dk else 1 - frac[2])
                    out.append((base + (dk * ny + dj) * nx + di, w))
        return out

    @staticmethod
    def blend(F, cs):
        """Corner values (float) times weights, summed in 64 bits."""
        tot = None
        for node, w in cs:
            v = F[node].double()
            v = v * (w[:, None] if v.dim() == 2 else w)
            tot = v if tot is None else tot + v
        return tot

    def sample(self, F, t, p, per_particle=None):
        idx, frac, ok = self.locate(p)
        cs = self.corners(idx, frac)
        if per_particle is None:
            a, b, tau = self.bracket(t)
            v = self.blend(F[a], cs)
            if a != b:
                v = (1 - tau) * v + tau * self.blend(F[b], cs)
            return v, ok
        sa, sb, tau = per_particle
        n = F.shape[0] // len(self.times)
        va = self.blend(F, [(c + sa * n, w) for c, w in cs])
        vb = self.blend(F, [(c + sb * n, w) for c, w in cs])
        return (1 - tau)[:, None] * va + tau[:, None] * vb, ok

    def slope(self, t, p, F=None, per_particle=None):
        v, ok = self.sample(self.F if F is None else F, t, p, per_particle)
        k = [v[:, q] for q in range(self.nd)]
        if self.spherical:
            k[0] = k[0] / (METRES * torch.cos(torch.deg2rad(p[1])))
            k[1] = k[1] / METRES
        return k, ok

    def on_land(self, p):
        idx, _, _ = self.locate(p[:2] if self.nd == 2 else p)
        return self.land[idx[1], idx[0]]

    def end(self, p, new, ok, status):
        """Commit a step: status 5 off the grid, 6 on land (deleted), else move."""
        act = status == 0
        _, _, inside = self.locate(new)
        bad = act & ~(ok & inside)
        status[bad] = 5
        good = act & ok & inside
        if self.land is not None:
            wet = ~self.on_land(new)
            status[good & ~wet] = 6
            good = good & wet
        for d in range(self.nd):
            p[d] = torch.where(good, new[d], p[d])
        return p

    def step(self, p, t, dt, status, euler=False, horizontal=None, kick=None):
        th, t1 = t + 0.5 * dt, t + dt
        k1, ok = self.slope(t, p)
        if euler:
            new = [x + k * dt for x, k in zip(p, k1)]
        else:
            k2, o2 = self.slope(th, [x + k * (0.5 * dt) for x, k in zip(p, k1)])
            k3, o3 = self.slope(th, [x + k * (0.5 * dt) for x, k in zip(p, k2)])
            k4, o4 = self.slope(t1, [x + k * dt for x, k in zip(p, k3)])
            ok = ok & o2 & o3 & o4
            new = [x + (a + 2 * b + 2 * c + d) * dt / 6
                   for x, a, b, c, d in zip(p, k1, k2, k3, k4)]
        if horizontal is not None:
            new[2] = torch.where(horizontal, p[2], new[2])
        if kick is not None:
            dx, dy = kick
            if self.spherical:
                dx = dx / (METRES * torch.cos(torch.deg2rad(new[1])))
                dy = dy / METRES
            new[0], new[1] = new[0] + dx, new[1] + dy
        return self.end(p, new, ok, status)


def _mulhilo(a, m):
    """High and low 32 bits of the 64-bit product of uint32 values held in int64."""
    lo, hi = a & 0xFFFF, a >> 16
    p0, p1 = lo * m, hi * m
    s = p0 + ((p1 & 0xFFFF) << 16)
    return (p1 >> 16) + (s >> 32), s & 0xFFFFFFFF


def _normals(n, step, run_id):
    """Philox4x32-10 (key run_id, 0x17070516; counter id, step, 0, 0) and Box-Muller."""
    c0 = torch.arange(n, device="cuda", dtype=torch.int64)
    c1 = torch.full_like(c0, step)
    c2, c3 = torch.zeros_like(c0), torch.zeros_like(c0)
    k0, k1 = run_id, 0x17070516
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        h0, l0 = _mulhilo(c0, 0xD2511F53)
        h1, l1 = _mulhilo(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
    u1 = ((c0 << 21) | (c1 >> 11)).double() * 2.0 ** -53 + 2.0 ** -54
    u2 = ((c2 << 21) | (c3 >> 11)).double() * 2.0 ** -53 + 2.0 ** -54
    r = torch.sqrt(-2.0 * torch.log(u1))
    return r * torch.cos(2 * math.pi * u2), r * torch.sin(2 * math.pi * u2)


def _diffuse(n, step, run_id, Kh, dt):
    s = math.sqrt(2.0 * Kh * abs(dt))
    a, b = _normals(n, step, run_id)
    return s * a, s * b


_C = (0.0, 1 / 4, 3 / 8, 12 / 13, 1.0, 1 / 2)
_A = ((), (1 / 4,), (3 / 32, 9 / 32), (1932 / 2197, -7200 / 2197, 7296 / 2197),
      (439 / 216, -8.0, 3680 / 513, -845 / 4104),
      (-8 / 27, 2.0, -3544 / 2565, 1859 / 4104, -11 / 40))
_B4 = (25 / 216, 0.0, 1408 / 2565, 2197 / 4104, -1 / 5, 0.0)
_B5 = (16 / 135, 0.0, 6656 / 12825, 28561 / 56430, -9 / 50, 2 / 55)


def _adaptive(ref, case, p, status):
    """Every particle by |dt| 2^e with its own e, one day at a time."""
    n, dt = p[0].numel(), case["dt"]
    T = torch.tensor(ref.times, device="cuda", dtype=torch.float64)
    F = torch.cat(ref.F)
    e = torch.zeros(n, device="cuda", dtype=torch.int64)

    def bracket(t):
        tp = T[0] + torch.remainder(t - T[0], ref.period)
        s = torch.searchsorted(T, tp, right=True) - 1
        up = torch.where(s + 1 < T.numel(), T[torch.clamp(s + 1, max=T.numel() - 1)],
                         T[0] + ref.period)
        return s, (s + 1) % T.numel(), (tp - T[s]) / (up - T[s])

    for day in range(case["days"]):
        t_end = (day + 1) * DAY
        t = torch.full((n,), day * DAY, device="cuda", dtype=torch.float64)
        while True:
            live = torch.nonzero((status == 0) & (t < t_end)).reshape(-1)
            if not live.numel():
                break
            q, tl, el = [x[live] for x in p], t[live], e[live]
            h = dt * torch.exp2(el.double())
            cut = h >= t_end - tl
            h = torch.where(cut, t_end - tl, h)
            ks, ok = [], torch.ones_like(cut)
            for i in range(6):
                pt = [x + h * sum(a * k[d] for a, k in zip(_A[i], ks)) if i else x
                      for d, x in enumerate(q)]
                k, o = ref.slope(None, pt, F, bracket(tl + _C[i] * h))
                ks.append(k)
                ok = ok & o
            new = [x + h * sum(b * k[d] for b, k in zip(_B4, ks)) for d, x in enumerate(q)]
            ev = [h * sum((b - a) * k[d] for a, b, k in zip(_B4, _B5, ks)) for d in range(2)]
            ex = ev[0] * METRES * torch.cos(torch.deg2rad(q[1]))
            err = torch.sqrt(ex * ex + (ev[1] * METRES) ** 2)
            retry = ok & (err > 1e-3) & (el > -6)
            s = status[live].clone()
            s[retry] = 1  # held back from the commit
            q = ref.end(q, new, ok, s)
            s[retry] = 0
            moved = ~retry & (s == 0)
            t[live] = torch.where(moved, torch.where(cut, torch.full_like(tl, t_end), tl + h), tl)
            up = moved & ~cut & (err <= 1e-3 / 32) & (el < 5)
            e[live] = el - retry.long() + up.long()
            for d in range(2):
                p[d][live] = q[d]
            status[live] = s
    return p


def _advect(ref, case, inp, run_id=0, behave=False, euler=False):
    """Positions at every day, and the tracer sample and age where the case has them."""
    p = [a.clone() for a in (inp["x"], inp["y"], inp["z"]) if a is not None]
    n = p[0].numel()
    status = torch.zeros(n, device="cuda", dtype=torch.uint8)
    temp = torch.full((n,), math.nan, device="cuda", dtype=torch.float64)
    age = torch.zeros(n, device="cuda", dtype=torch.float64)
    dt = -case["dt"] if behave else case["dt"]
    per, t0, Kh = int(round(DAY / case["dt"])), inp["t0"], case.get("Kh", 0.0)
    recs = [([x.clone() for x in p], temp.clone(), age.clone())]
    for day in range(case["days"]):
        for s in range(day * per, (day + 1) * per):
            t, act, flat = t0 + s * dt, status == 0, None
            if behave:
                sink = act & (p[2] > 50.0)
                p[2] = torch.where(sink, torch.clamp(p[2] + 200.0 / DAY * dt, min=50.0), p[2])
                flat = p[2] <= 50.0
                age = torch.where(act & flat, age + abs(dt), age)
                status[act & flat & (age >= 30 * DAY)] = 12
                act = status == 0
            if ref.T:
                v, ok = ref.sample(ref.T, t, p)
                temp = torch.where(act & ok, v, temp)
            kick = _diffuse(n, s, run_id, Kh, dt) if Kh > 0 else None
            p = ref.step(p, t, dt, status, euler, flat, kick)
        recs.append(([x.clone() for x in p], temp.clone(), age.clone()))
    return recs


def _laid_out(recs, stride, behave):
    names = ("lon", "lat", "depth")
    h = lambda a: a.cpu().numpy()  # noqa: E731
    final = {k: h(a) for k, a in zip(names, recs[-1][0])}
    out = dict(final=final, status=None, steps=None)
    if stride:
        out["records"] = {k: np.stack([h(r[0][q][::stride]) for r in recs])
                          for q, k in enumerate(names[:len(recs[0][0])])}
        if behave:
            out["records"]["temp"] = np.stack([h(r[1][::stride]) for r in recs])
            out["records"]["age"] = np.stack([h(r[2][::stride]) for r in recs])
    return out


def exact(case, seed):
    k = case["kind"]
    if k == "infer":
        return None  # the network rounds to bfloat16 and thresholds: no 64-bit counterpart
    if (k == "ocean3d" and case["n"] * case["days"] > 12_000_000) or \
            (k == "ensemble" and case["runs"] * case["days"] > 30):
        return None  # takes too long in plain torch
    if k == "hour":
        inp = _inputs_hour(case, seed)
        ref = _Reference(inp)
        p = [inp["x"].clone(), inp["y"].clone()]
        status = torch.zeros(case["n"], device="cuda", dtype=torch.uint8)
        for s in range(case["steps"]):
            p = ref.step(p, s * case["dt"], case["dt"], status)
        return dict(lon=p[0].cpu().numpy(), lat=p[1].cpu().numpy(), ci=None, cj=None)
    if k == "global2d":
        inp = _inputs_global2d(case, seed)
        ref = _Reference(inp, case["dtype"])
        if case["kernel"] == "rkf45":
            p = [inp["x"].clone(), inp["y"].clone()]
            status = torch.zeros(case["n"], device="cuda", dtype=torch.uint8)
            p = _adaptive(ref, case, p, status)
            out = _laid_out([(p, None, None)], 0, False)
            out["exponents"] = None
            return out
        recs = _advect(ref, case, inp, 3, euler=case["kernel"] == "euler")
        return _laid_out(recs, case["stride"], case["sample"])
    if k == "ensemble":
        lon, lat = [], []
        for r, inp in enumerate(_inputs_ensemble(case, seed)):
            p = _advect(_Reference(inp), case, inp, r)[-1][0]
            lon.append(p[0].cpu().numpy())
            lat.append(p[1].cpu().numpy())
        return dict(lon=np.concatenate(lon), lat=np.concatenate(lat), ci=None, cj=None,
                    status=None)
    if k == "ocean3d":
        inp = _inputs_ocean3d(case, seed)
        return _laid_out(_advect(_Reference(inp, case["dtype"]), case, inp), case["stride"],
                         False)
    if k == "footprint":
        inp = _inputs_footprint(case, seed)
        return _laid_out(_advect(_Reference(inp), case, inp, behave=True), 1, True)
    X, T, params = _inputs_train(case, seed)
    X, T = torch.from_numpy(X).cuda().double(), torch.from_numpy(T).cuda().double()
    W = [torch.from_numpy(w).cuda().double().requires_grad_() for w, _ in params]
    b = [torch.from_numpy(v).cuda().double().requires_grad_() for _, v in params]
    h = X
    for l in range(5):
        h = h @ W[l] + b[l]
        if l < 4:
            h = torch.nn.functional.gelu(h, approximate="tanh")
    loss = 0.5 * ((h - T) ** 2).sum() / X.shape[0]
    loss.backward()

    def stepped(a):  # Adam's first step: both moments corrected to the gradient itself
        return (a - 1e-3 * a.grad / (a.grad.abs() + 1e-8)).detach().cpu().numpy()

    return dict(loss=np.float64(loss.item()), params=[(stepped(w), stepped(v))
                                                      for w, v in zip(W, b)])
