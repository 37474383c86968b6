"""Workloads the library is timed on: time stepping of a single lattice in every
storage format and streaming scheme, the benchmark's snapshot interval, batched
serving, and the diagnostics the studies take of a state.

listed() gives the cases, draw() more of the same ranges, prepare() what a
program holds before the call (a lattice with its start flow), run() one pass
through the public entry points, work() the bytes and operations of a pass, and
exact() the same results from plain FP64 torch, written from the equations.

The start flow is a seeded sum of solenoidal Fourier modes (wavenumbers up to 6,
rms velocity about U0 = 0.043, amplitudes falling as in an inertial range) plus
the 1e-3 velocity noise of the forced-HIT workload, so that every run meets
turbulence-like gradients; the force is 16 solenoidal modes on |k| <= 2.
"""
import math
import random

import numpy as np
import torch

from paper_2512_23116_amd import lbm, serving

U0 = 0.043
RE = 2.0e4
BYTES = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}
DTYPE = {"fp64": torch.float64, "fp32": torch.float32, "fp16": torch.float16,
         "bf16": torch.bfloat16}
SCALE = {"fp64": 1.0, "fp32": 1.0, "fp16": 32768.0, "bf16": 1.0}


# ------------------------------------------------------------------ cases ---
def _step(name, n, precision, streaming, steps, tb=0, C=0.1, smag_form=1, tau_mode=0, forced=True,
          spg=64):
    nx, ny, nz = n
    return dict(name=name, kind="step", nx=nx, ny=ny, nz=nz, precision=precision,
                streaming=streaming, steps=steps, tb=tb, C=C, smag_form=smag_form,
                tau_mode=tau_mode, forced=forced, spg=spg)


def listed():
    return [
        # The 32^3 FP64 decaying-flow parity case, a few steps at a time: the
        # smallest calls, where launches and host latency count.
        _step("decay_32_fp64_aa", (32, 32, 32), "fp64", "aa", 4, C=0.1, smag_form=0,
              forced=False),
        # A ragged lattice with odd extents and the self-consistent relaxation
        # time, plain launches (no graph).
        _step("ragged_130x127x129_fp32_aa", (129, 127, 130), "fp32", "aa", 16, C=0.13,
              tau_mode=1, spg=0),
        # The 256^3 precision study: the FP64 reference run and FP16 storage.
        _step("hit_256_fp64_ab", (256, 256, 256), "fp64", "ab", 16),
        _step("hit_256_fp16_aa", (256, 256, 256), "fp16", "aa", 64),
        # BF16 storage on a lattice well beyond the cache.
        _step("hit_400_bf16_aa", (400, 400, 400), "bf16", "aa", 16),
        # The 512^3 reference DNS of the Smagorinsky-constant study: FP32, two
        # steps per pass, no closure.
        _step("dns_512_fp32_two_step", (512, 512, 512), "fp32", "ab", 16, tb=2, C=0.0),
        # The 800^3 DNS of the iso-Reynolds pair in FP16, two steps per pass:
        # the largest lattice.
        _step("dns_800_fp16_two_step", (800, 800, 800), "fp16", "ab", 4, tb=2, C=0.0),
        # The benchmark's headline lattice with its snapshot (statistics, K_t map
        # of the mid plane, spectrum); a fifth of its 500-step interval per pass,
        # one graph replay.
        dict(name="hit_100_fp32_ab_interval", kind="interval", nx=100, ny=100, nz=100,
             precision="fp32", streaming="ab", steps=100, C=0.1),
        # One batched call of the serving loop: 16 slots of its request sizes.
        dict(name="serving_16_slots", kind="batch",
             sizes="128,96,64,48,32,128,64,48,96,32,64,96,48,128,32,64", steps=64),
        # A snapshot of the regime study: K_t field to the host, theta histogram
        # of 400 bins, domain statistics.
        dict(name="regime_snapshot_100_fp32", kind="regime", nx=100, ny=100, nz=100,
             precision="fp32", streaming="aa", bins=400),
        # A snapshot of the energy-balance study: turbulence scales,
        # one-dimensional spectra, shell spectrum.
        dict(name="energy_balance_128_fp32", kind="spectra", nx=128, ny=128, nz=128,
             precision="fp32", streaming="aa"),
        # A snapshot of the intermittency study: structure functions at 16
        # geometrically spaced separations.
        dict(name="intermittency_256_fp32", kind="structure", nx=256, ny=256, nz=256,
             precision="fp32", streaming="aa", nr=16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _extents(rng, lo, hi):
    """Three extents around a log-uniform size, ragged half of the time."""
    n = _log_int(rng, lo, hi)
    if rng.random() < 0.5:
        return n, n, n
    return tuple(max(4, int(n * rng.uniform(0.75, 1.0))) for _ in range(3))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "interval", "batch", "regime", "spectra",
                       "structure"])
    if kind == "step":
        precision = rng.choice(["fp64", "fp32", "fp32", "fp16", "bf16"])
        nx, ny, nz = _extents(rng, 24, 320 if precision == "fp64" else 512)
        streaming = rng.choice(["aa", "ab"])
        tb = 2 if streaming == "ab" and precision != "fp64" and rng.random() < 0.5 else 0
        # passes of about 20 ms at most on the larger lattices
        most = max(4, min(64, int(4e8 / (nx * ny * nz))))
        steps = rng.choice([s for s in (4, 8, 16, 32, 64) if s <= most])
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, precision=precision, streaming=streaming,
                    steps=steps, tb=tb, C=rng.choice([0.0, 0.1, 0.13]),
                    smag_form=rng.choice([0, 1]), tau_mode=rng.choice([0, 0, 1]),
                    forced=rng.random() < 0.8, spg=rng.choice([0, 64]))
    if kind == "interval":
        nx, ny, nz = _extents(rng, 48, 160)
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, precision=rng.choice(["fp64", "fp32"]),
                    streaming=rng.choice(["aa", "ab"]), steps=rng.choice([20, 64, 100]),
                    C=rng.choice([0.1, 0.13]))
    if kind == "batch":
        slots = rng.randint(2, 16)
        sizes = [str(rng.choice([32, 48, 64, 96, 128])) for _ in range(slots)]
        return dict(kind=kind, sizes=",".join(sizes), steps=64)
    nx, ny, nz = _extents(rng, 32, 240)
    if kind == "regime":
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, precision=rng.choice(["fp64", "fp32"]),
                    streaming=rng.choice(["aa", "ab"]), bins=_log_int(rng, 40, 4000))
    if kind == "spectra":
        n = min(nx, 180)
        return dict(kind=kind, nx=n, ny=n, nz=n, precision=rng.choice(["fp64", "fp32"]),
                    streaming=rng.choice(["aa", "ab"]))
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, precision=rng.choice(["fp64", "fp32"]),
                streaming=rng.choice(["aa", "ab"]), nr=rng.randint(4, 16))


# ----------------------------------------------------------------- inputs ---
def _force_modes(n, seed):
    """16 solenoidal modes on 1 <= |k|^2 <= 4 with seeded phases: (k, amp, phase)."""
    r = random.Random(seed * 7919 + 1)
    F0 = 0.2 * U0 * U0 / n
    out = []
    for kx in range(0, 3):
        for ky in range(-2, 3):
            for kz in range(-2, 3):
                k2 = kx * kx + ky * ky + kz * kz
                if 1 <= k2 <= 4 and (kx, ky, kz) > (0, 0, 0):
                    out.append(((kx, ky, kz), _perpendicular((kx, ky, kz), F0 * 0.43, r),
                                r.uniform(0.0, 2.0 * math.pi)))
    return out


def _perpendicular(k, size, r):
    """A vector of length `size` at a random angle in the plane perpendicular to k."""
    kv = np.array(k, dtype=np.float64)
    v = np.array([r.gauss(0.0, 1.0) for _ in range(3)])
    v -= kv * (v @ kv) / (kv @ kv)
    return tuple(float(x) for x in size * v / np.linalg.norm(v))


def _flow_modes(seed, n=18):
    r = random.Random(seed * 104729 + 2)
    out = []
    while len(out) < n:
        k = tuple(r.randint(-6, 6) for _ in range(3))
        k2 = sum(c * c for c in k)
        if 1 <= k2 <= 36:
            out.append((k, _perpendicular(k, 0.028 * k2 ** (-5.0 / 12.0), r),
                        r.uniform(0.0, 2.0 * math.pi)))
    return out


def _axes(nx, ny, nz):
    x, y, z = (torch.arange(n, device="cuda", dtype=torch.float64) for n in (nx, ny, nz))
    return x.view(1, 1, nx), y.view(1, ny, 1), z.view(nz, 1, 1)


def _phase(k, phi, nx, ny, nz):
    x, y, z = _axes(nx, ny, nz)
    w = 2.0 * math.pi
    return (w * k[0] / nx) * x + (w * k[1] / ny) * y + ((w * k[2] / nz) * z + phi)


def _velocity(nx, ny, nz, seed, noise=1e-3):
    """u of shape (3, nz, ny, nx), FP64."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.empty((3, nz, ny, nx), dtype=torch.float64, device="cuda")
    for a in range(3):
        torch.rand((nz, ny, nx), generator=g, dtype=torch.float64, device="cuda", out=u[a])
        u[a].mul_(2.0 * noise).sub_(noise)
    for k, amp, phi in _flow_modes(seed):
        s = _phase(k, phi, nx, ny, nz).sin_()
        for a in range(3):
            u[a].add_(s, alpha=amp[a])
    return u


def _strain(nx, ny, nz, seed):
    """S_ab = (d_a u_b + d_b u_a) / 2 of the smooth part of the flow (xx, yy, zz, xy, xz, yz)."""
    S = torch.zeros((6, nz, ny, nx), dtype=torch.float64, device="cuda")
    for k, amp, phi in _flow_modes(seed):
        c = _phase(k, phi, nx, ny, nz).cos_()
        w = [2.0 * math.pi * q / n for q, n in zip(k, (nx, ny, nz))]
        for j, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
            S[j].add_(c, alpha=0.5 * (w[a] * amp[b] + w[b] * amp[a]))
    return S


def _developed(case, seed):
    """Full populations f (19 planes) of a developed flow: f_eq plus the first-order
    non-equilibrium part -3 w tau0 (c c - 1/3) : S."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    S = _strain(nx, ny, nz, seed)
    f = _equilibrium(_velocity(nx, ny, nz, seed))
    tr = (S[0] + S[1] + S[2]) / 3.0
    for i in range(19):
        c = [float(v) for v in _C[i]]
        q = (c[0] * c[0] * S[0] + c[1] * c[1] * S[1] + c[2] * c[2] * S[2] - tr
             + 2.0 * (c[0] * c[1] * S[3] + c[0] * c[2] * S[4] + c[1] * c[2] * S[5]))
        f[i].sub_(q, alpha=3.0 * float(_W[i]) * _tau0(case)).add_(float(_W[i]))
    return f


def _tau0(case):
    if "tau0" in case:
        return case["tau0"]
    return 0.51 if case.get("forced") is False else 0.5 + 3.0 * U0 * case["nx"] / RE


def _stream():
    """One stream for every lattice here, as a program that steps them in turn has."""
    global _shared
    if _shared is None:
        _shared = torch.cuda.Stream()
    return _shared


_shared = None


def _lattice(case, seed, stream=None):
    forced = case.get("forced", True)
    modes = _force_modes(case["nx"], seed) if forced else ()
    steps = case.get("steps", 64)
    spg = case.get("spg", steps if steps % 4 == 0 else 64)
    return lbm.Lattice((case["nz"], case["ny"], case["nx"]), _tau0(case), case.get("C", 0.13),
                       modes, precision=case["precision"], streaming=case["streaming"],
                       smag_form=case.get("smag_form", 1), steps_per_graph=spg,
                       temporal_block=case.get("tb", 0), tau_mode=case.get("tau_mode", 0),
                       stream=stream or _stream())


def _populations(lat, case):
    """The lattice's population planes (19, ncell), views of its buffer (one by one on
    lattices of more than 2^31 populations).  Every pass
    takes an even number of steps (a multiple of four of launches that alternate two
    arrays), so the current planes are the first array's."""
    n = case["nx"] * case["ny"] * case["nz"]
    b = BYTES[case["precision"]]
    arrays = 2 if case["streaming"] == "ab" else 1
    size = lbm.lbm_required_bytes(lat.cfg)
    off = lat.cfg.device_buffer - lat.buffer.data_ptr()
    plane = size // (arrays * 19)
    dtype = DTYPE[case["precision"]]
    if n * 19 <= 1 << 31:
        return lat.buffer[off:off + 19 * plane].view(dtype).view(19, plane // b)[:, :n]
    return [lat.buffer[off + i * plane:off + i * plane + n * b].view(dtype) for i in range(19)]


def _slots(case, seed):
    """The lattices of a batch: C in [0.08, 0.18], tau0 in [0.505, 0.55], each with its
    own flow and force."""
    out = []
    for i, n in enumerate(int(s) for s in case["sizes"].split(",")):
        out.append(dict(nx=n, ny=n, nz=n, precision="fp32", streaming="aa", steps=case["steps"],
                        C=0.08 + 0.1 * ((i * 7 + seed) % 16) / 15.0,
                        tau0=0.505 + 0.045 * ((i * 5 + seed) % 16) / 15.0, seed=seed * 100 + i))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        eng = serving.GpuEngine(max_slots=16, steps_per_graph=64)
        reqs = []
        for i, slot in enumerate(_slots(case, seed)):
            n = slot["nx"]
            reqs.append(serving.Request(rid=i, N=n, C=slot["C"], tau0=slot["tau0"], force_seed=i,
                                        init_seed=i, arrival=0.0, steps=1 << 30))
            eng.lat[i] = _lattice(slot, slot["seed"], eng.stream)
            eng.lat[i].init_velocity(_velocity(n, n, n, slot["seed"]))
        return dict(case=case, eng=eng, reqs=reqs)
    lat = _lattice(case, seed)
    if kind in ("regime", "spectra"):
        lat.set_populations(torch.stack(_developed(case, seed)).cpu().numpy())
    else:
        lat.init_velocity(_velocity(case["nx"], case["ny"], case["nz"], seed))
    state = dict(case=case, lat=lat)
    if kind == "structure":
        top = min(case["nx"], case["ny"], case["nz"]) // 2
        state["rs"] = sorted(set(int(r) for r in np.round(np.geomspace(1, top, case["nr"]))))
    return state


# -------------------------------------------------------------------- run ---
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        eng, reqs = state["eng"], state["reqs"]
        eng.calls.clear()
        eng.wait(eng.step(reqs, [case["steps"]] * len(reqs)))
        return [_populations(eng.lat[r.rid], dict(nx=r.N, ny=r.N, nz=r.N, precision="fp32",
                                                  streaming="aa")) for r in reqs]
    lat = state["lat"]
    if kind == "step":
        lat.step(case["steps"])
        return _populations(lat, case)
    if kind == "interval":
        kmax = min(case["nx"], case["ny"], case["nz"]) // 2
        lat.step(case["steps"])
        lat.snapshot_begin(kmax, case["nz"] // 2)
        st, E, plane = lat.snapshot_end()
        # statistics of a state in the storage's precision, in that precision
        real = np.float64 if case["precision"] == "fp64" else np.float32
        return dict(f=_populations(lat, case), E=E.astype(real), plane=plane,
                    kt_mean=real(st["kt_mean"]), kt_var=real(st["kt_var"]),
                    theta_mean=real(st["theta_mean"]), energy=real(st["energy"]))
    if kind == "regime":
        return dict(kt=lat.kt_field(), hist=lat.theta_histogram(0.0, 4e-3, case["bins"]),
                    stats=lat.stats())
    if kind == "spectra":
        n = case["nx"]
        turb = lat.turbulence()
        E1, ic = lat.spectra_1d(n // 4 + 1)
        return dict(turb=turb, E1=E1, ic=ic, E=lat.spectrum(n // 2))
    return lat.structure_functions(state["rs"])


def work(case):
    """Per time step every population is read once and written once (two steps per
    pass: once per pair), with about 300 operations per cell; a diagnostic reads the
    state once."""
    if case["kind"] == "batch":
        cells = sum(int(s) ** 3 for s in case["sizes"].split(","))
        return dict(bytes=2 * 19 * 4 * cells * case["steps"], flops=300 * cells * case["steps"])
    n = case["nx"] * case["ny"] * case["nz"]
    b = BYTES[case["precision"]]
    if case["kind"] == "step":
        passes = case["steps"] // (2 if case["tb"] == 2 else 1)
        return dict(bytes=2 * 19 * b * n * passes, flops=300 * n * case["steps"])
    log2n = math.log2(max(n, 2))
    fft = 3 * 2.5 * n * log2n
    if case["kind"] == "interval":
        return dict(bytes=19 * b * n * (2 * case["steps"] + 1),
                    flops=300 * n * (case["steps"] + 1) + fft)
    if case["kind"] == "regime":
        return dict(bytes=(19 * b + 4) * n, flops=200 * n)
    if case["kind"] == "spectra":
        return dict(bytes=19 * b * n, flops=200 * n + fft)
    return dict(bytes=19 * b * n, flops=(100 + 3 * 12 * case["nr"]) * n)


# ------------------------------------------------------- the same in 64 bits ---
# Velocities c_i in opposite pairs, rest last; weights by speed.
_C = np.array([(1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
               (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0),
               (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1),
               (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 0, 0)])
_W = np.array([1 / 18] * 6 + [1 / 36] * 12 + [1 / 3])
_RATES = dict(e=1.19, eps=1.4, q=1.2, pi=1.4, m=1.98)


def _moment_matrix():
    """The D3Q19 moments as polynomials of c, evaluated on the velocity set."""
    cx, cy, cz = (_C[:, a].astype(np.float64) for a in range(3))
    c2 = cx * cx + cy * cy + cz * cz
    rows = [np.ones(19), 19 * c2 - 30, (21 * c2 * c2 - 53 * c2 + 24) / 2,
            cx, (5 * c2 - 9) * cx, cy, (5 * c2 - 9) * cy, cz, (5 * c2 - 9) * cz,
            3 * cx * cx - c2, (3 * c2 - 5) * (3 * cx * cx - c2),
            cy * cy - cz * cz, (3 * c2 - 5) * (cy * cy - cz * cz),
            cx * cy, cy * cz, cx * cz,
            (cy * cy - cz * cz) * cx, (cz * cz - cx * cx) * cy, (cx * cx - cy * cy) * cz]
    return torch.tensor(np.stack(rows), dtype=torch.float64, device="cuda")


def _equilibrium(u):
    """f_eq - w at rho = 1: 19 planes shaped like u[0]."""
    uu = (u * u).sum(0)
    out = []
    for i in range(19):
        cu = sum(float(_C[i, a]) * u[a] for a in range(3))
        out.append(float(_W[i]) * (3.0 * cu + 4.5 * cu * cu - 1.5 * uu))
    return out


def _force(case, modes, lo, hi):
    """F (3, cells of planes lo..hi-1)."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    F = torch.zeros((3, hi - lo, ny, nx), dtype=torch.float64, device="cuda")
    x, y, z = _axes(nx, ny, nz)
    w = 2.0 * math.pi
    for k, amp, phi in modes:
        s = torch.sin((w * k[0] / nx) * x + (w * k[1] / ny) * y + ((w * k[2] / nz) * z[lo:hi] + phi))
        for a in range(3):
            F[a].add_(s, alpha=amp[a])
    return F.view(3, -1)


def _moments_of(g, F, case, M):
    """Deviation moments, velocity, non-equilibrium moments and tau_e of cells g (19, n)."""
    m = M @ g
    rho = 1.0 + m[0]
    ru = torch.stack([m[3], m[5], m[7]]) + 0.5 * F
    u = ru / rho
    xx, yy, zz = ru[0] * u[0], ru[1] * u[1], ru[2] * u[2]
    r2 = xx + yy + zz
    meq = torch.zeros_like(m)
    meq[0] = m[0]
    meq[1] = -11.0 * m[0] + 19.0 * r2
    meq[2] = -475.0 / 63.0 * r2
    for a, (j, q) in enumerate(((3, 4), (5, 6), (7, 8))):
        meq[j] = ru[a]
        meq[q] = -2.0 / 3.0 * ru[a]
    meq[9] = 2.0 * xx - yy - zz
    meq[11] = yy - zz
    meq[13], meq[14], meq[15] = ru[0] * u[1], ru[1] * u[2], ru[0] * u[2]
    neq = m - meq
    tau0, tm = _tau0(case), case.get("tau_mode", 0)
    C = case.get("C", 0.13)
    c3 = 3.0 * (C * C if case.get("smag_form", 1) == 1 else C)
    s1, s9 = (_RATES["e"], 1.0 / tau0) if tm == 0 else (0.0, 1.0)
    Sxx = -(s1 * neq[1] + 19.0 * s9 * neq[9]) / 38.0
    Syy = -(2.0 * s1 * neq[1] - 19.0 * s9 * (neq[9] - 3.0 * neq[11])) / 76.0
    Szz = -(2.0 * s1 * neq[1] - 19.0 * s9 * (neq[9] + 3.0 * neq[11])) / 76.0
    d2 = (1.5 * s9) ** 2 * (neq[13] ** 2 + neq[14] ** 2 + neq[15] ** 2)
    S2 = 2.0 * (Sxx * Sxx + Syy * Syy + Szz * Szz + 2.0 * d2)
    if tm == 0:
        tau_t = c3 * S2.sqrt()
    else:
        X = c3 * S2.sqrt()
        tau_t = 2.0 * X / (tau0 + torch.sqrt(tau0 * tau0 + 4.0 * X))
        S2 = S2 / (tau0 + tau_t) ** 2
    return m, u, neq, tau_t, S2, rho


def _slabs(case, most=1 << 24):
    per = max(1, most // (case["nx"] * case["ny"]))
    return [(lo, min(lo + per, case["nz"])) for lo in range(0, case["nz"], per)]


def _advance(g, case, modes, steps):
    """`steps` collide-and-stream steps of the deviations g (19 planes (nz, ny, nx)), in place."""
    M = _moment_matrix()
    Minv = torch.linalg.inv(M)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    r = _RATES
    for _ in range(steps):
        for lo, hi in _slabs(case):
            F = _force(case, modes, lo, hi)
            cells = torch.stack([q[lo:hi].reshape(-1) for q in g])
            m, u, neq, tau_t, _, _ = _moments_of(cells, F, case, M)
            s_nu = 1.0 / (_tau0(case) + tau_t)
            uF = (u * F).sum(0)
            P = 2.0 * u[0] * F[0] - u[1] * F[1] - u[2] * F[2]
            Q = u[1] * F[1] - u[2] * F[2]
            force = {1: 38.0 * uF, 2: -11.0 * uF, 9: 2.0 * P, 10: -P, 11: 2.0 * Q, 12: -Q,
                     13: u[0] * F[1] + u[1] * F[0], 14: u[1] * F[2] + u[2] * F[1],
                     15: u[0] * F[2] + u[2] * F[0]}
            for a, (j, q) in enumerate(((3, 4), (5, 6), (7, 8))):
                force[j], force[q] = F[a], -2.0 / 3.0 * F[a]
            rate = {1: r["e"], 2: r["eps"], 4: r["q"], 6: r["q"], 8: r["q"], 10: r["pi"],
                    12: r["pi"], 16: r["m"], 17: r["m"], 18: r["m"], 3: 1.0, 5: 1.0, 7: 1.0,
                    9: s_nu, 11: s_nu, 13: s_nu, 14: s_nu, 15: s_nu}
            for k, s in rate.items():
                m[k] -= s * neq[k]
                if k in force:
                    m[k] += (1.0 - 0.5 * s) * force[k]
            m = Minv @ m
            for q, v in zip(g, m):
                q[lo:hi] = v.view(hi - lo, ny, nx)
        for i in range(18):
            cx, cy, cz = (int(v) for v in _C[i])
            g[i] = torch.roll(g[i], shifts=(cz, cy, cx), dims=(0, 1, 2))
    return g


def _fields(g, case, modes):
    """theta, u, |S|^2, rho, F of the deviations g (19 planes (nz, ny, nx))."""
    M = _moment_matrix()
    shape = (case["nz"], case["ny"], case["nx"])
    theta, s2, rho = (torch.empty(shape, dtype=torch.float64, device="cuda") for _ in range(3))
    u, F = (torch.empty((3,) + shape, dtype=torch.float64, device="cuda") for _ in range(2))
    for lo, hi in _slabs(case):
        Fs = _force(case, modes, lo, hi)
        _, us, _, tau_t, S2, rs = _moments_of(torch.stack([q[lo:hi].reshape(-1) for q in g]), Fs,
                                            case, M)
        theta[lo:hi] = (_tau0(case) - 0.5 + tau_t).view(hi - lo, *shape[1:])
        s2[lo:hi] = S2.view(hi - lo, *shape[1:])
        rho[lo:hi] = rs.view(hi - lo, *shape[1:])
        u[:, lo:hi] = us.view(3, hi - lo, *shape[1:])
        F[:, lo:hi] = Fs.view(3, hi - lo, *shape[1:])
    return theta, u, s2, rho, F


def _stored(g, case):
    """g as the population planes hold it: at its own cell (AA after an even number of
    steps) or at the cell it came from (A/B), in units of the storage scale."""
    if case["streaming"] == "ab":
        for i in range(18):
            cx, cy, cz = (int(v) for v in _C[i])
            g[i] = torch.roll(g[i], shifts=(-cz, -cy, -cx), dims=(0, 1, 2))
    if SCALE[case["precision"]] != 1.0:
        for q in g:
            q *= SCALE[case["precision"]]
    g = [q.view(-1) for q in g]
    return torch.stack(g) if 19 * g[0].numel() <= 1 << 31 else g


def _shells(u, kmax):
    """E[0..kmax] = 1/2 sum |u_hat|^2 over k - 1/2 <= |q| < k + 1/2."""
    nz, ny, nx = u.shape[1:]
    q = [torch.fft.fftfreq(n, 1.0 / n, device="cuda", dtype=torch.float64) for n in (nx, ny, nz)]
    mag = torch.sqrt(q[2].view(nz, 1, 1) ** 2 + q[1].view(1, ny, 1) ** 2 + q[0].view(1, 1, nx) ** 2)
    shell = torch.floor(mag + 0.5).long().view(-1)
    e = sum(torch.fft.fftn(u[a]).abs().square() for a in range(3)).view(-1)
    e *= 0.5 / float(nx * ny * nz) ** 2
    E = torch.bincount(shell, weights=e, minlength=kmax + 1)
    return E[:kmax + 1].cpu().numpy()


def _field_stats(case, theta, u, s2, rho, F):
    n = theta.numel()
    d = theta - theta.mean()
    var = (d * d).mean()
    root3 = math.sqrt(3.0)
    skew, flat = (d ** 3).mean() / var ** 1.5, (d ** 4).mean() / var ** 2
    uu = u.square().sum(0)
    th = [float(v) for v in (theta.mean(), var, skew, flat, theta.min(), theta.max())]
    prod = [float((u[a] * u[b]).mean()) for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))]
    return dict(n_cells=n, steps=0, theta_mean=th[0], theta_var=th[1], theta_skew=th[2],
                theta_flat=th[3], theta_min=th[4], theta_max=th[5], kt_mean=root3 * th[0],
                kt_var=3.0 * th[1], kt_skew=th[2], kt_flat=th[3], kt_min=root3 * th[4],
                kt_max=root3 * th[5], mass=float(rho.sum()),
                momentum=[float((rho * u[a]).sum()) for a in range(3)],
                energy=float(0.5 * uu.mean()), energy_rho=float(0.5 * (rho * uu).mean()),
                n_nonfinite=0, strain2=float(s2.mean()),
                nut_strain2=float(((theta - (_tau0(case) - 0.5)) / 3.0 * s2).mean()),
                injection=float((F * u).sum(0).mean()),
                u_mean=[float(u[a].mean()) for a in range(3)], uu=prod)


def _turbulence(case, st, E):
    N = case["nx"]
    k = np.arange(1, E.size)
    kap = 2.0 * np.pi * k / N
    nu0 = (_tau0(case) - 0.5) / 3.0
    e = E[1:].sum()
    eps = 2.0 * nu0 * (kap * kap * E[1:]).sum()
    u_rms = math.sqrt(2.0 * e / 3.0)
    taylor = math.sqrt(15.0 * nu0 * u_rms ** 2 / eps)
    m = np.array(st["u_mean"])
    q = st["uu"]
    R = np.array([[q[0], q[3], q[4]], [q[3], q[1], q[5]], [q[4], q[5], q[2]]]) - np.outer(m, m)
    tr = np.trace(R)
    b = R / tr - np.eye(3) / 3.0
    II, III = -0.5 * np.trace(b @ b), np.trace(b @ b @ b) / 3.0
    return dict(kmax=int(E.size - 1), energy=st["energy"], energy_spec=float(e), u_rms=u_rms,
                integral_scale=float(0.75 * np.pi * (E[1:] / kap).sum() / e), eps_spec=float(eps),
                eps_strain=nu0 * st["strain2"], eps_sgs=st["nut_strain2"],
                injection=st["injection"], eta=float((nu0 ** 3 / eps) ** 0.25), taylor=taylor,
                re_lambda=u_rms * taylor / nu0, energy_frac=[float(R[i, i] / tr) for i in range(3)],
                b=[float(b[i, j]) for i, j in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))],
                II_b=float(II), III_b=float(III), lumley_xi=float(np.cbrt(III / 2.0)),
                lumley_eta=float(np.sqrt(-II / 3.0)))


def _spectra_1d(u, kmax):
    n = u.shape[1]
    E = np.zeros((3, 3, kmax + 1))
    k = torch.fft.fftfreq(n, 1.0 / n, device="cuda").abs().round().long()
    for c in range(3):
        p = torch.fft.fftn(u[c]).abs().square() / float(n) ** 6
        for a, dims in enumerate(((0, 1), (0, 2), (1, 2))):
            line = torch.bincount(k, weights=p.sum(dims), minlength=kmax + 1)
            E[c, a] = line[:kmax + 1].cpu().numpy()
    EL = (E[0, 0] + E[1, 1] + E[2, 2]) / 3.0
    ET = (E[1, 0] + E[2, 0] + E[0, 1] + E[2, 1] + E[0, 2] + E[1, 2]) / 6.0
    ic = np.full(kmax + 1, np.nan)
    for j in range(2, kmax):
        slope = (math.log(EL[j + 1]) - math.log(EL[j - 1])) / (math.log(j + 1) - math.log(j - 1))
        ic[j] = (EL[j] - EL[j] * slope) / (2.0 * ET[j])
    return E, ic


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return [exact(dict(slot, kind="step"), slot["seed"]) for slot in _slots(case, seed)]
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    modes = _force_modes(nx, seed) if case.get("forced", True) else []
    if kind in ("step", "interval"):
        g = _equilibrium(_velocity(nx, ny, nz, seed))
        _advance(g, case, modes, case["steps"])
        if kind == "step":
            return _stored(g, case)
        theta, u, s2, rho, F = _fields(g, case, modes)
        st = _field_stats(case, theta, u, s2, rho, F)
        return dict(E=_shells(u, min(nx, ny, nz) // 2),
                    plane=(math.sqrt(3.0) * theta[nz // 2]).clone(), kt_mean=st["kt_mean"],
                    kt_var=st["kt_var"], theta_mean=st["theta_mean"], energy=st["energy"],
                    f=_stored(g, case))
    if kind == "structure":
        # the velocity of f_eq(u) with the half-force shift
        u = _velocity(nx, ny, nz, seed)
        u += 0.5 * _force(case, modes, 0, nz).view(3, nz, ny, nx)
        top = min(nx, ny, nz) // 2
        rs = sorted(set(int(r) for r in np.round(np.geomspace(1, top, case["nr"]))))
        out = np.zeros((len(rs), 6))
        for j, r in enumerate(rs):
            for a, dim in enumerate((2, 1, 0)):
                d = torch.roll(u[a], -r, dim) - u[a]
                d2, ad = d * d, d.abs()
                for m, v in enumerate((d2, d2 * d, d2 * ad, d2 * d2, d2 * d2 * ad, d2 * d2 * d2)):
                    out[j, m] += float(v.mean()) / 3.0
        return out
    g = [q - float(w) for q, w in zip(_developed(case, seed), _W)]
    theta, u, s2, rho, F = _fields(g, case, modes)
    st = _field_stats(case, theta, u, s2, rho, F)
    if kind == "regime":
        return dict(kt=math.sqrt(3.0) * theta, hist=None, stats=st)
    E = _shells(u, int(0.5 * math.sqrt(3.0) * nx + 1.0))
    E1, ic = _spectra_1d(u, nx // 4 + 1)
    return dict(turb=_turbulence(case, st, E), E1=E1, ic=ic, E=E[:nx // 2 + 1])
