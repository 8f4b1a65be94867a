"""Performance cases of the particle library and of the field producer.

Each case is one call pattern of a program that uses this package, at one
size: stepping particles through held or streamed velocity levels, stepping
the field producer, the coupled loop of both, gradients through a
checkpointed run, and finite-time Lyapunov exponents.

``listed()`` gives the named cases, ``draw(rng)`` one more of the same
ranges, ``prepare(case, seed)`` what a program holds before the call,
``run(state)`` one pass through the public entry points, ``work(case)`` the
bytes and operations a pass cannot do without, and ``exact(case, seed)`` the
same outputs in 64-bit torch, without the package's kernels.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_17836_amd import autotune, coupled, lpt, ns2d, workloads

L = 2.0 * math.pi
DEV = "cuda"
MASK64 = (1 << 64) - 1

# the eight Stokes numbers and schemes of the package's batching workload
_BATCH = ",".join(f"{kind}:{st}:{sch}:{count}" for kind, st, sch, count, _ in
                  workloads.C4_BATCH.species)


def listed():
    return [
        # The smallest call a user makes: a few thousand tracers on a 64^2
        # steady Taylor-Green cell, 100 steps a call, statistics every 10
        # (the package's tg64 benchmark).
        dict(name="advect_64_taylor_green", kind="advect", n=64, precision="fp64",
             flow="taylor_green", k0=1.0, dt=0.01, mode="bracket", levels="held",
             species="tracer:0.0:bilinear:4096", steps=100, stats_every=10, sort_interval=0),
        # The paper's own size: about a thousand particles carried by a 256^2
        # decaying flow, ten coupled steps a call.
        dict(name="coupled_256_paper", kind="coupled", n=256, precision="fp64", dt=2e-3,
             species="tracer:0.0:bspline:1000,inertial:0.5:bilinear:1000", steps=10,
             stats_every=10, sort_interval=0),
        # Velocity frames that arrive coarser than the particle step (files, or
        # another solver), on a grid that is no power of two with ragged
        # counts: ingest the bracket's two levels, then eight steps inside it.
        dict(name="stream_1000_ragged", kind="advect", n=1000, precision="fp64",
             flow="spectrum", k0=10.0, dt=0.004, mode="bracket", levels="streamed",
             species="tracer:0.0:bspline:300007,inertial:0.1:bilinear:200003", steps=8,
             stats_every=8, sort_interval=16),
        # Turbulence-sized ensemble in FP64 with the bicubic scheme (the
        # package's spec1024 benchmark): tracers and inertial particles.
        dict(name="advect_1024_catmull_rom", kind="advect", n=1024, precision="fp64",
             flow="spectrum", k0=10.0, dt=0.005, mode="pingpong", levels="held",
             species="tracer:0.0:catmull_rom:1048576,inertial:0.1:catmull_rom:1048576", steps=10,
             stats_every=10, sort_interval=20),
        # The headline: 2^24 split-precision tracers on 4096^2, sixteen steps
        # (one re-sort interval) a call.
        dict(name="advect_4096_split", kind="advect", n=4096, precision="fp32_split",
             flow="spectrum", k0=20.0, dt=1e-3, mode="pingpong", levels="held",
             species="tracer:0.0:bilinear:16777216", steps=16, stats_every=100,
             sort_interval=16),
        # A parameter sweep in one context: eight Stokes numbers, three
        # schemes, 65 thousand to 8 million particles each.
        dict(name="advect_2048_batch", kind="advect", n=2048, precision="fp32_split",
             flow="spectrum", k0=10.0, dt=1e-3, mode="pingpong", levels="held",
             species=_BATCH, steps=10, stats_every=100, sort_interval=20),
        # The field producer alone, from a size where launches count to the
        # largest grid of the built-in transforms.
        dict(name="field_512", kind="field", n=512, dt=1e-3, steps=10),
        dict(name="field_2048", kind="field", n=2048, dt=1e-3, steps=4),
        dict(name="field_4096", kind="field", n=4096, dt=5e-4, steps=2),
        # The coupled loop at the package's benchmark size: 2048^2 field, a
        # million FP64 tracers.
        dict(name="coupled_2048", kind="coupled", n=2048, precision="fp64", dt=1e-3,
             species="tracer:0.0:bilinear:1048576", steps=4, stats_every=100, sort_interval=20),
        # Gradient of a loss of the final positions with respect to the
        # initial positions and to the velocity grid (flow reconstruction):
        # the checkpointed run and its reverse sweep.
        dict(name="gradient_2048", kind="gradient", n=2048, flow="cells", k0=10.0, dt=0.01,
             scheme="bilinear", count=2048 * 2048, seeding="lattice", steps=40, every=20,
             sort_interval=20),
        # Finite-time Lyapunov exponents of a lattice of tracers.
        dict(name="ftle_1024", kind="ftle", n=1024, flow="cells", k0=10.0, dt=0.01,
             scheme="catmull_rom", count=512 * 512, seeding="lattice", steps=40, every=20,
             sort_interval=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["advect", "advect", "advect", "field", "coupled", "gradient", "ftle"])
    scheme = rng.choice(["bilinear", "catmull_rom", "bspline"])
    if kind == "field":
        n = 1 << rng.randint(6, 12)
        return dict(kind=kind, n=n, dt=5e-4 if n == 4096 else 1e-3,
                    steps=rng.randint(1, 10 if n <= 1024 else 4))
    if kind in ("gradient", "ftle"):
        n = _log_int(rng, 64, 2048)
        seeding = rng.choice(["lattice", "uniform"])
        count = _log_int(rng, 1000, (1 << 21) if kind == "gradient" else (1 << 18))
        if seeding == "lattice":
            count = int(math.isqrt(count)) ** 2
        steps = rng.randint(8, 40)
        return dict(kind=kind, n=n, flow="cells", k0=min(10.0, n / 10),
                    dt=rng.uniform(0.2, 3.0) * L / n, scheme=scheme, count=count,
                    seeding=seeding, steps=steps, every=rng.randint(4, 20),
                    sort_interval=20 if count > 20000 else 0)

    def species(total, most):
        k = rng.randint(1, most)
        out = []
        for _ in range(k):
            count = max(1, int(total * rng.uniform(0.5, 1.0) / k))
            st = rng.choice([0.0, 0.05, 0.5, 5.0])
            out.append(f"{'inertial' if st else 'tracer'}:{st}:"
                       f"{rng.choice(['bilinear', 'catmull_rom', 'bspline'])}:{count}")
        return ",".join(out)

    if kind == "coupled":
        n = 1 << rng.randint(6, 11)
        total = _log_int(rng, 100, 1 << 20)
        steps = rng.randint(1, 10 if n <= 1024 else 4)
        return dict(kind=kind, n=n, precision=rng.choice(["fp64", "fp32_split"]), dt=1e-3,
                    species=species(total, 2), steps=steps, stats_every=steps,
                    sort_interval=20 if total > 20000 else 0)
    n = _log_int(rng, 64, 4096)
    total = _log_int(rng, 500, 1 << 22)
    steps = _log_int(rng, 1, 40)
    return dict(kind="advect", n=n, precision=rng.choice(["fp64", "fp32_split"]),
                flow="spectrum", k0=min(20.0, n / 12), dt=rng.uniform(0.1, 0.9) * L / n,
                mode=rng.choice(["pingpong", "bracket"]),
                levels=rng.choice(["held", "streamed"]), species=species(total, 3), steps=steps,
                stats_every=rng.choice([0, steps]), sort_interval=16 if total > 20000 else 0)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _modes(n):
    ky = torch.fft.fftfreq(n, d=1.0 / n, device=DEV, dtype=torch.float64)[:, None]
    kx = torch.fft.rfftfreq(n, d=1.0 / n, device=DEV, dtype=torch.float64)[None, :]
    return kx, ky, torch.sqrt(kx * kx + ky * ky)


def _spectrum(n, k0, seed, gap):
    """Two velocity levels [2, n, n] of a random-phase stream function, the
    phases advanced by |k| gap in the second; rms 1 a component."""
    kx, ky, km = _modes(n)
    amp = torch.sqrt(km * torch.exp(-(km / k0) ** 2))
    phase = torch.rand(amp.shape, generator=_generator(seed), device=DEV,
                       dtype=torch.float64) * L

    def level(ph):
        psi = torch.polar(amp, ph)
        return torch.stack([torch.fft.irfft2(1j * ky * psi, s=(n, n)),
                            torch.fft.irfft2(-1j * kx * psi, s=(n, n))])

    a, b = level(phase), level(phase - km * gap)
    scale = 1.0 / torch.sqrt((a * a).mean())
    return (a * scale).contiguous(), (b * scale).contiguous()


def _taylor_green(n):
    x = torch.arange(n, device=DEV, dtype=torch.float64) * (L / n)
    s, c = torch.sin(x), torch.cos(x)
    return torch.stack([s[None, :] * c[:, None], -c[None, :] * s[:, None]]).contiguous()


def _levels(case, seed):
    n = case["n"]
    if case["flow"] == "taylor_green":
        a = _taylor_green(n)
        return a, a
    gap = case["dt"] * (case["steps"] if case.get("mode") == "bracket" else 1)
    a, b = _spectrum(n, case["k0"], seed, gap)
    if case["flow"] == "cells":   # Taylor-Green cells with a weak random part
        tg = _taylor_green(n)
        return tg + 0.1 * a, tg + 0.1 * b
    return a, b


def _vorticity(n, seed):
    """Random-phase initial vorticity of rms 3 (energy peak at mode 10, or
    n / 10 on small grids)."""
    k0 = min(10.0, n / 10)
    _, _, km = _modes(n)
    amp = torch.sqrt(km ** 5 * torch.exp(-(km / k0) ** 2))
    ph = torch.rand(amp.shape, generator=_generator(seed), device=DEV, dtype=torch.float64) * L
    w = torch.fft.irfft2(torch.polar(amp, ph), s=(n, n))
    return (w * (3.0 / torch.sqrt((w * w).mean()))).contiguous()


NU = 1e-4


def _species(text):
    out = []
    for part in text.split(","):
        kind, st, scheme, count = part.split(":")
        out.append((kind, float(st), scheme, int(count)))
    return out


def _signed(z):
    z &= MASK64
    return z - (1 << 64) if z >> 63 else z


def _init_seed(seed, k):
    return (1000003 * seed + 7919 * k + 1) & MASK64


def _shr(z, s):
    return (z >> s) & ((1 << (64 - s)) - 1)


def _uniform(count, seed):
    """The positions Tracker.init_uniform documents: outputs 2p and 2p + 1 of
    the SplitMix64 stream, top 53 bits as a fraction of L."""
    k = torch.arange(2 * count, device=DEV, dtype=torch.int64) + 1
    z = _signed(seed) + k * _signed(0x9E3779B97F4A7C15)
    z = (z ^ _shr(z, 30)) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _signed(0x94D049BB133111EB)
    z = z ^ _shr(z, 31)
    u = _shr(z, 11).to(torch.float64) * 2.0 ** -53 * L
    u = torch.where(u >= L, u - L, u)
    return u[0::2].contiguous(), u[1::2].contiguous()


def _points(case, seed):
    if case["seeding"] == "uniform":
        p = torch.rand((2, case["count"]), generator=_generator(seed + 17), device=DEV,
                       dtype=torch.float64) * L
        return p[0].contiguous(), p[1].contiguous()
    side = math.isqrt(case["count"])
    c = (torch.arange(side, device=DEV, dtype=torch.float64) + 0.5) * (L / side)
    return c.repeat(side).contiguous(), c.repeat_interleave(side).contiguous()


def _cotangents(case, seed):
    g = torch.randn((2, case["count"]), generator=_generator(seed + 29), device=DEV,
                    dtype=torch.float64)
    return g[0].contiguous(), g[1].contiguous()


# ---------------------------------------------------------------------------
# prepare
# ---------------------------------------------------------------------------
def _shipped_tuning(case):
    """The launch shape the package ships for this workload, if it has one."""
    sp = tuple((k, st, sch, c, 0) for k, st, sch, c in _species(case["species"]))
    w = workloads.Workload("case", case["n"], case["precision"], case["flow"], dt=case["dt"],
                           time_mode=case["mode"], stats_every=case["stats_every"], species=sp)
    key = autotune.workload_key(w, autotune.device_key(0))
    entry = autotune.load_cache(autotune.SHIPPED).get(key)
    return entry["tuning"] if entry else None


def _add(tracker, case, seed, shift=0):
    """The case's species and the tensors that receive their state."""
    outs = []
    for k, (kind, st, scheme, count) in enumerate(_species(case["species"])):
        zeros = torch.zeros(count, device=DEV, dtype=torch.float64)
        sid = tracker.add_species(kind, st, scheme, zeros, zeros)
        tracker.init_uniform(sid, _init_seed(seed, k + shift))
        pos = tuple(torch.empty_like(zeros) for _ in range(4))
        vel = tuple(torch.empty_like(zeros) for _ in range(2)) if st > 0.0 else ()
        outs.append((sid, pos, vel))
    return outs


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    st = dict(case=case)
    if kind == "field":
        st["field"] = ns2d.Ns2d(n, NU, case["dt"])
        st["field"].set_vorticity(_vorticity(n, seed))
        st["uv"] = _buffers(n)
    elif kind == "coupled":
        st["loop"] = coupled.CoupledLoop(n, NU, case["dt"], _vorticity(n, seed),
                                         precision=case["precision"],
                                         sort_interval=case["sort_interval"])
        st["outs"] = _add(st["loop"].tracker, case, seed)
        st["uv"] = _buffers(n)
    elif kind == "advect":
        a, b = _levels(case, seed)
        tr = lpt.Tracker(n, case["precision"], sort_interval=case["sort_interval"])
        tr.set_time_mode(case["mode"])
        # a held bracket covers the whole run; ping-pong levels are one step apart
        tb = case["dt"] * (1 if case["mode"] == "pingpong" else
                           case["steps"] * (1 if case["levels"] == "streamed" else 1 << 20))
        tr.set_snapshot(0, 0.0, a[0], a[1])
        tr.set_snapshot(1, tb, b[0], b[1])
        st["outs"] = _add(tr, case, seed)
        tuning = _shipped_tuning(case)
        if tuning:
            tr.set_tuning(**tuning)
        st.update(tracker=tr, a=a, b=b)
    else:
        a, b = _levels(case, seed)
        x0, y0 = _points(case, seed)
        tr = lpt.Tracker(n, "fp64", sort_interval=case["sort_interval"])
        tr.set_snapshot(0, 0.0, a[0], a[1])
        tr.set_snapshot(1, case["steps"] * case["dt"], b[0], b[1])
        tr.add_species("tracer", 0.0, case["scheme"], x0, y0)
        st.update(tracker=tr, a=a, b=b, pos=tuple(torch.empty_like(x0) for _ in range(4)))
        if kind == "gradient":
            st["gx"], st["gy"] = _cotangents(case, seed)
    return st


def _buffers(n):
    return tuple(torch.empty((n, n), device=DEV, dtype=torch.float64) for _ in range(2))


# ---------------------------------------------------------------------------
# run
# ---------------------------------------------------------------------------
def _read(tracker, outs):
    """Positions (and velocities) of every species into the program's tensors."""
    res = []
    for sid, pos, vel in outs:
        tracker.get_positions(sid, out=pos)
        if vel:
            st = lpt.load().lpt_get_velocities(tracker.handle, sid, vel[0].data_ptr(),
                                               vel[1].data_ptr(), 1)
            if st != lpt.OK:
                raise RuntimeError(f"lpt_get_velocities: status {st}")
        res.extend(pos + vel)
    return res


def _grid_velocity(field, uv):
    """The producer's current velocity into the program's tensors."""
    st = ns2d.load().ns2d_get_fields(field._h, uv[0].data_ptr(), uv[1].data_ptr(), None, None, 1)
    if st != ns2d.OK:
        raise RuntimeError(f"ns2d_get_fields: status {st}")
    return list(uv)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "field":
        state["field"].step(case["steps"])
        return _grid_velocity(state["field"], state["uv"])
    if kind == "coupled":
        state["loop"].step(case["steps"], case["stats_every"])
        return (_read(state["loop"].tracker, state["outs"]) +
                _grid_velocity(state["loop"].field, state["uv"]))
    tr = state["tracker"]
    if kind == "advect":
        if case["levels"] == "streamed":
            _stream(tr, case, state["a"], state["b"])
        tr.step(case["steps"], case["dt"], case["stats_every"])
        res = _read(tr, state["outs"])
        if case["stats_every"] and case["steps"] % case["stats_every"] == 0:
            for sid, _, _ in state["outs"]:   # the transport statistics so far
                rec = tr.get_stats(sid)
                res.append(np.stack([rec[f] for f in ("t", "msd_x", "msd_y", "msd", "sem")]))
        return res
    _stream(tr, case, state["a"], state["b"])
    tr.forward_checkpointed(case["steps"], case["dt"], case["every"])
    tr.get_positions(0, out=state["pos"])
    if kind == "gradient":
        return list(state["pos"]) + list(tr.adjoint(state["gx"], state["gy"]))
    return list(state["pos"]) + [tr.ftle()]


def _stream(tr, case, a, b):
    """The next pair of levels: ping-pong keeps the step's parity, a bracket
    starts at the present time."""
    if case.get("mode") == "pingpong":
        tr.set_snapshot(0, 0.0, a[0], a[1])
        tr.set_snapshot(1, case["dt"], b[0], b[1])
    else:
        t = tr.get_time()[1]
        tr.set_snapshot(0, t, a[0], a[1])
        tr.set_snapshot(1, t + case["steps"] * case["dt"], b[0], b[1])


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
def _flops(kind, st, scheme):
    """Operations of one particle-step: four interpolations of two levels and
    the Runge-Kutta combination (a fused multiply-add counts two)."""
    f = 208 if scheme == "bilinear" else 824
    return f + (46 if kind == "inertial" and st > 0.0 else 0)


def _field_work(n, steps):
    spec = n * ((n - 1) // 3 + 1) * 16
    # state and previous right-hand side in and out, velocity out
    return dict(bytes=4 * spec + 2 * 8 * n * n,
                flops=steps * 5 * 2.5 * n * n * 2 * math.log2(n))


def work(case):
    n, kind = case["n"], case["kind"]
    if kind == "field":
        return _field_work(n, case["steps"])
    if kind in ("gradient", "ftle"):
        grid = 2 * 2 * n * n * 8
        per = _flops("tracer", 0.0, case["scheme"])
        # positions in and out; cotangents and gradients, or the exponent
        extra = 4 * 8 if kind == "gradient" else 8
        return dict(bytes=grid + case["count"] * (16 + 32 + extra) +
                    (grid if kind == "gradient" else 0),
                    flops=case["count"] * case["steps"] * 3 * per)
    fp64 = case["precision"] == "fp64"
    b = f = 0
    for k, st, scheme, count in _species(case["species"]):
        inert = st > 0.0
        b += count * (2 * ((32 + 16 * inert) if fp64 else (16 + 8 * inert)) + 32 + 16 * inert)
        f += count * case["steps"] * _flops(k, st, scheme)
    if kind == "coupled":
        w = _field_work(n, case["steps"])
        return dict(bytes=b + w["bytes"], flops=f + w["flops"])
    b += 2 * 2 * n * n * (8 if fp64 or case["levels"] == "streamed" else 4)
    return dict(bytes=b, flops=f)


# ---------------------------------------------------------------------------
# exact: plain torch in 64 bits
# ---------------------------------------------------------------------------
def _weights(scheme, s):
    if scheme == "bilinear":
        return 0, [1.0 - s, s]
    if scheme == "catmull_rom":
        return -1, [0.5 * (-s + 2 * s ** 2 - s ** 3), 0.5 * (2 - 5 * s ** 2 + 3 * s ** 3),
                    0.5 * (s + 4 * s ** 2 - 3 * s ** 3), 0.5 * (s ** 3 - s ** 2)]
    return -1, [(1 - s) ** 3 / 6, (4 - 6 * s ** 2 + 3 * s ** 3) / 6,
                (1 + 3 * s + 3 * s ** 2 - 3 * s ** 3) / 6, s ** 3 / 6]


def _velocity(F, n, scheme, x, y):
    """Interpolated (u, v) of the grid F [n * n, 2] at (x, y)."""
    sx, sy = x * (n / L), y * (n / L)
    fx, fy = torch.floor(sx.detach()), torch.floor(sy.detach())
    o, wx = _weights(scheme, sx - fx)
    _, wy = _weights(scheme, sy - fy)
    i, j = fx.to(torch.int64), fy.to(torch.int64)
    u = v = 0.0
    for b, wb in enumerate(wy):
        row = torch.remainder(j + (o + b), n) * n
        for a, wa in enumerate(wx):
            f = F.index_select(0, row + torch.remainder(i + (o + a), n))
            w = wa * wb
            u = u + w * f[:, 0]
            v = v + w * f[:, 1]
    return u, v


def _nodes(level):
    return level.reshape(2, -1).t().contiguous()


def _stage_weights(mode, k, steps, held, dt):
    """Weights of the first level at the four stages of step k."""
    if mode == "pingpong":
        th = [0.0, 0.5, 0.5, 1.0]
        return [1.0 - t for t in th] if k % 2 == 0 else th
    span = steps if not held else steps * (1 << 20)
    return [1.0 - (k + c) / span for c in (0.0, 0.5, 0.5, 1.0)]


def _rk4(F, n, scheme, dt, st, x, y, vx, vy):
    """One step through the four stage grids F; st > 0: Stokes drag."""
    def vel(q, a, b):
        return _velocity(F[q], n, scheme, a, b)
    c = (0.0, 0.5 * dt, 0.5 * dt, dt)
    if st == 0.0:
        kx, ky = [], []
        for q in range(4):
            u, v = vel(q, x + c[q] * kx[-1], y + c[q] * ky[-1]) if q else vel(0, x, y)
            kx.append(u)
            ky.append(v)
        return (x + dt / 6 * (kx[0] + 2 * kx[1] + 2 * kx[2] + kx[3]),
                y + dt / 6 * (ky[0] + 2 * ky[1] + 2 * ky[2] + ky[3]), vx, vy)
    V, A = [], []
    for q in range(4):
        px = (x + c[q] * V[-1][0], y + c[q] * V[-1][1]) if q else (x, y)
        w = (vx + c[q] * A[-1][0], vy + c[q] * A[-1][1]) if q else (vx, vy)
        u, v = vel(q, *px)
        V.append(w)
        A.append(((u - w[0]) / st, (v - w[1]) / st))

    def comb(S, m):
        return dt / 6 * (S[0][m] + 2 * S[1][m] + 2 * S[2][m] + S[3][m])
    return x + comb(V, 0), y + comb(V, 1), vx + comb(A, 0), vy + comb(A, 1)


def _wrap(x):
    w = x - L * torch.floor(x / L)
    return torch.where(w >= L, w - L, w)


def _stats_row(t, dx, dy):
    mx, my = (dx * dx).mean(), (dy * dy).mean()
    r2 = dx * dx + dy * dy
    sem = torch.sqrt(r2.var(unbiased=True) / r2.numel()) if r2.numel() > 1 else r2.sum() * 0.0
    return [t, float(mx), float(my), float(mx + my), float(sem)]


def _advance(case, seed, grids):
    """Every species through case["steps"] steps; grids(k) gives the four
    stage grids of step k.  Yields (x0, y0, x, y, vx, vy, record rows)."""
    n, dt, every = case["n"], case["dt"], case["stats_every"]
    sp = _species(case["species"])
    parts = []
    for k, (kind, st, scheme, count) in enumerate(sp):
        x0, y0 = _uniform(count, _init_seed(seed, k))
        vx = vy = None
        if st > 0.0:
            vx, vy = _velocity(grids(0)[0], n, scheme, x0, y0)
        parts.append([x0, y0, x0, y0, vx, vy, []])
    chunk = 1 << 21
    for s in range(case["steps"]):
        F = grids(s)
        for (kind, st, scheme, count), p in zip(sp, parts):
            res = [_rk4(F, n, scheme, dt, st, *(None if a is None else a[c:c + chunk]
                                                for a in p[2:6]))
                   for c in range(0, count, chunk)]
            for m in range(2, 6):
                if p[m] is not None:
                    p[m] = torch.cat([r[m - 2] for r in res])
            if every and (s + 1) % every == 0:
                p[6].append(_stats_row((s + 1) * dt, p[2] - p[0], p[3] - p[1]))
    return parts


def _state_outputs(case, parts):
    out = []
    for (kind, st, scheme, count), p in zip(_species(case["species"]), parts):
        out += [_wrap(p[2]), _wrap(p[3]), p[2], p[3]]
        if st > 0.0:
            out += [p[4], p[5]]
    return out


class _Field:
    """Pseudospectral vorticity with second-order Adams-Bashforth steps."""

    def __init__(self, n, dt, omega):
        self.n, self.dt, self.prev = n, dt, None
        self.kx, self.ky, km = _modes(n)
        self.k2 = km * km
        self.band = (3 * self.kx.abs() < n) & (3 * self.ky.abs() < n)
        self.w = torch.fft.rfft2(omega) * self.band
        self.ik2 = torch.where(self.k2 > 0, 1.0 / self.k2.clamp(min=1.0), 0.0)

    def back(self, z):
        return torch.fft.irfft2(z, s=(self.n, self.n))

    def velocity(self):
        psi = self.w * self.ik2
        return torch.stack([self.back(1j * self.ky * psi), self.back(-1j * self.kx * psi)])

    def step(self):
        u, v = self.velocity()
        adv = u * self.back(1j * self.kx * self.w) + v * self.back(1j * self.ky * self.w)
        r = -torch.fft.rfft2(adv) * self.band - NU * self.k2 * self.w
        old = r if self.prev is None else self.prev
        self.w = self.w + self.dt * (1.5 * r - 0.5 * old)
        self.prev = r


def exact(case, seed):
    kind, n, dt, steps = case["kind"], case["n"], case["dt"], case["steps"]
    if kind == "field":
        f = _Field(n, dt, _vorticity(n, seed))
        for _ in range(steps):
            f.step()
        return list(f.velocity())
    if kind == "coupled":
        f = _Field(n, dt, _vorticity(n, seed))
        levels = [f.velocity()]
        for _ in range(steps + 1):
            f.step()
            levels.append(f.velocity())

        def grids(k):
            a, b = _nodes(levels[k]), _nodes(levels[k + 1])
            m = 0.5 * (a + b)
            return [a, m, m, b]
        parts = _advance(case, seed, grids)
        return _state_outputs(case, parts) + list(levels[-1])
    a, b = _levels(case, seed)
    if kind == "advect":
        A, B = _nodes(a), _nodes(b)
        held = case["levels"] == "held"

        def grids(k):
            w = _stage_weights(case["mode"], k, steps, held, dt)
            g = [w[0] * A + (1.0 - w[0]) * B, w[1] * A + (1.0 - w[1]) * B, None,
                 w[3] * A + (1.0 - w[3]) * B]
            g[2] = g[1]
            return g
        parts = _advance(case, seed, grids)
        out = _state_outputs(case, parts)
        if case["stats_every"] and steps % case["stats_every"] == 0:
            out += [np.array(p[6]).T for p in parts]
        return out
    return _exact_derivatives(case, seed, a, b)


def _exact_derivatives(case, seed, a, b):
    kind, n, dt, steps = case["kind"], case["n"], case["dt"], case["steps"]
    x0, y0 = _points(case, seed)
    bilinear = case["scheme"] == "bilinear"
    chunk = (1 << 20) if bilinear else (1 << 17)
    grad = kind == "gradient"
    if grad:
        gx, gy = _cotangents(case, seed)
        chunk = min(chunk, 1 << 19)
    A = _nodes(a).requires_grad_(grad)
    B = _nodes(b).requires_grad_(grad)
    xs, ys, gxs, gys, sig = [], [], [], [], []
    gA = torch.zeros_like(A)
    gB = torch.zeros_like(B)
    for c in range(0, case["count"], chunk):
        px = x0[c:c + chunk].clone().requires_grad_(True)
        py = y0[c:c + chunk].clone().requires_grad_(True)
        x, y = px, py
        for k in range(steps):
            w = _stage_weights("bracket", k, steps, False, dt)
            F = [w[0] * A + (1.0 - w[0]) * B, w[1] * A + (1.0 - w[1]) * B, None,
                 w[3] * A + (1.0 - w[3]) * B]
            F[2] = F[1]
            x, y, _, _ = _rk4(F, n, case["scheme"], dt, 0.0, x, y, None, None)
        xs.append(x.detach())
        ys.append(y.detach())
        if grad:
            loss = (gx[c:c + chunk] * x).sum() + (gy[c:c + chunk] * y).sum()
            dx, dy, dA, dB = torch.autograd.grad(loss, (px, py, A, B))
            gxs.append(dx)
            gys.append(dy)
            gA += dA
            gB += dB
        else:
            p, q = torch.autograd.grad(x.sum(), (px, py), retain_graph=True)
            r, s = torch.autograd.grad(y.sum(), (px, py))
            m, o, t = p * p + r * r, q * q + s * s, p * q + r * s
            lam = 0.5 * (m + o) + torch.sqrt((0.5 * (m - o)) ** 2 + t * t)
            sig.append(0.5 * torch.log(lam) / (steps * dt))
        del x, y, F
    x, y = torch.cat(xs), torch.cat(ys)
    out = [_wrap(x), _wrap(y), x, y]
    if grad:
        gU = torch.stack([gA.t().reshape(2, n, n), gB.t().reshape(2, n, n)])
        return out + [torch.cat(gxs), torch.cat(gys), gU]
    return out + [torch.cat(sig).cpu().numpy()]
