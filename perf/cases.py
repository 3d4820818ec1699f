"""The workloads whose speed is followed from change to change: whole PIC steps
through the library's handle (``hpic.Sim``), over the geometries, sizes, particle
shapes and precisions that runs of this framework use.

A pass advances every run of a handle by ``steps`` steps and then reads what a
program looks at after such a stretch: the six fields of each run (Cartesian
runs, into device tensors), with ``particles`` also the momenta in loading order,
and for quasi-3D runs the accelerating field (E_z, mode 0) and the laser's
(E_r, mode 1) on the host, the only place that geometry delivers fields to.

``exact`` advances the same inputs with the method written out in torch FP64:
spline gather, Boris rotation, Esirkepov deposit, Eq. (11), the filter and the
hybrid update of Eqs. (12)-(17) (per azimuthal mode in quasi-3D).
"""
import math
import random

import numpy as np
import torch

from paper_1502_01376_amd import hpic

# Every key a case may set, with the value it has otherwise.
DEFAULTS = dict(geom="2d", n1=64, n2=32, n3=0, modes=0, precision="fp32", shape=2, interp=0, kmod=0,
                dx1=0.2, dx2=0.2, dt=0.05, gamma=50.0, sigma=1e-4, sub1=2, sub2=2, ppc=0,
                spread=0.0, density=1.0, laser=0.0, antenna=False, runs=1, mix=0, tile1=0, tile2=0,
                sort=0, steps=16, particles=False)


def _case(**kw):
    return {k: v for k, v in kw.items()}


def listed():
    return [
        # One step and a look at the fields on the smallest grid in use: what a
        # program that couples to the run every step waits for (launches).
        _case(name="small_step", ppc=4, steps=1),
        # Four independent 256 x 256 drifts in one handle, as the instability
        # study runs its variants, between two diagnostics.
        _case(name="drift_256_x4", n1=256, n2=256, runs=4, dt=0.08, density=100.0, ppc=4, steps=16),
        # The flagship run: laser against a drifting plasma, 8.4M particles,
        # at the tiling the autotuner picks for it.
        _case(name="laser_2d", n1=2048, n2=512, dx1=0.1, dt=0.045, gamma=20.0, sigma=0.0, sub1=4,
              sub2=2, laser=2.0, tile1=16, tile2=16, sort=64, steps=16, particles=True),
        # The same physics in the FP64 form that precision studies use.
        _case(name="laser_2d_fp64", n1=1024, n2=512, dx1=0.1, dt=0.045, gamma=20.0, sigma=0.0,
              sub1=4, sub2=2, laser=2.0, precision="fp64", steps=8),
        # A parameter scan: 24 uneven runs batched in one handle, particles at
        # random positions, default tiling.
        _case(name="scan_24", runs=24, mix=4, steps=16),
        # Boosted-frame wakefield grid: few particles per cell on very long
        # rows, laser from the moving antenna.
        _case(name="lwfa_antenna", n1=8192, n2=512, dx1=2.746, dx2=2.746, dt=0.618, gamma=-14.0,
              density=1.607e-2, ppc=2, antenna=True, steps=8),
        # Cubic shape with the modified symbol (the long instability runs).
        _case(name="cubic_2d", n1=1024, n2=300, shape=3, kmod=1, dt=0.08, ppc=4, steps=16),
        # 3D drift, 16.8M particles with varying weights, at its usual tiling.
        _case(name="drift_3d", geom="3d", n1=512, n2=128, n3=128, sigma=0.0, sub1=2, sub2=1,
              spread=0.05, tile1=8, tile2=4, sort=64, steps=4),
        # A 3D run on odd transverse sizes, energy-conserving gather, momenta
        # read back.
        _case(name="ragged_3d", geom="3d", n1=128, n2=37, n3=45, interp=1, ppc=3, gamma=20.0,
              steps=8, particles=True),
        # 3D in the FP64 form.
        _case(name="drift_3d_fp64", geom="3d", n1=128, n2=64, n3=64, precision="fp64", ppc=2, steps=4),
        # Quasi-3D column with a seed pulse, three modes.
        _case(name="quasi_3d", geom="q3d", n1=2048, n2=256, modes=3, dx1=0.1, dt=0.04, gamma=20.0,
              sigma=0.0, laser=1.0, steps=16),
        # Quasi-3D in the FP64 form, two modes, odd radial size.
        _case(name="quasi_3d_fp64", geom="q3d", n1=256, n2=61, modes=2, dx1=0.1, dt=0.04, gamma=20.0,
              sigma=0.0, laser=1.0, precision="fp64", steps=8),
    ]


def draw(rng):
    def log2int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    precision = "fp64" if rng.random() < 0.25 else "fp32"
    kind = rng.choice(("2d", "2d", "2d", "batch", "3d", "3d", "q3d"))
    gamma = round(rng.uniform(5.0, 100.0), 3)
    steps = rng.choice((1, 2, 4, 8, 16))
    if kind == "batch":
        return _case(runs=rng.randint(2, 16), mix=rng.randint(0, 999), steps=rng.choice((4, 8, 16)),
                     precision=precision, shape=rng.choice((2, 2, 3)))
    if kind == "2d":
        n1 = 2 ** rng.randint(6, 12)
        n2 = log2int(16, max(17, min(1024, 2 ** 21 // n1)))
        return _case(n1=n1, n2=n2, ppc=rng.randint(2, 12 if n1 * n2 < 2 ** 19 else 8), gamma=gamma,
                     shape=rng.choice((2, 2, 2, 3)), interp=rng.choice((0, 0, 1)),
                     kmod=rng.choice((0, 0, 1)), spread=rng.choice((0.0, 0.0, 0.05)),
                     laser=rng.choice((0.0, 2.0)) if n1 >= 256 and n2 >= 64 else 0.0,
                     precision=precision, steps=steps, particles=rng.random() < 0.5)
    if kind == "3d":
        n1 = 2 ** rng.randint(5, 8)
        return _case(geom="3d", n1=n1, n2=log2int(8, 96), n3=log2int(8, 96), ppc=rng.randint(1, 6),
                     gamma=gamma, interp=rng.choice((0, 0, 1)), spread=rng.choice((0.0, 0.05)),
                     precision=precision, steps=min(steps, 8), particles=rng.random() < 0.5)
    return _case(geom="q3d", n1=2 ** rng.randint(6, 10), n2=log2int(24, 192), modes=rng.randint(1, 4),
                 dx1=0.1, dt=0.04, gamma=gamma, sigma=0.0, laser=1.0, precision=precision,
                 interp=rng.choice((0, 0, 1)), steps=steps)


# ------------------------------------------------------------------ inputs
def _runs(case):
    """The runs of a case's handle, each a case of its own with every key set.
    A batch with ``mix`` draws sizes, drift, density and particle count per run
    as the parameter scan does."""
    c = dict(DEFAULTS, **case)
    if c["runs"] == 1:
        return [c]
    if not c["mix"]:
        return [dict(c, runs=1) for _ in range(c["runs"])]
    r = random.Random(c["mix"])
    return [dict(c, runs=1, n1=r.choice((256, 512, 1024, 2048)), n2=r.choice((64, 128, 256, 512)),
                 gamma=r.uniform(5.0, 100.0), density=r.uniform(0.5, 2.0), ppc=r.randint(4, 16))
            for _ in range(c["runs"])]


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _antenna(c):
    """At the peak of its envelope from the first step on."""
    L1, L2 = c["n1"] * c["dx1"], c["n2"] * c["dx2"]
    beta = math.sqrt(1.0 - 1.0 / c["gamma"] ** 2)
    omega = (1.0 + beta) / (abs(c["gamma"]) * (1.0 + beta))
    T = 400.0 * c["dt"]
    return dict(x0=0.125 * L1, v=-beta, t0=-0.5 * T, T=T, K0=2.0 * 4.0 * omega, omega=omega, phase=0.3,
                x2c=0.5 * L2, waist=0.08 * L2)


def _inputs(c, seed):
    """Particles and fields of one run in FP64 on the device: positions x in
    cell units (quasi-3D: physical z, x, y), u, w, E, B, background current."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    f8 = dict(dtype=torch.float64, device=dev)
    n = [c["n1"], c["n2"]] + ([c["n3"]] if c["geom"] == "3d" else [])
    if c["geom"] == "q3d":
        return _inputs_q3d(c, g, f8)
    dim, cells = len(n), math.prod(n)
    ppc = c["ppc"] or c["sub1"] * c["sub2"]
    idx = torch.arange(cells, device=dev)
    pos = []
    for d in range(dim):
        at = (idx // math.prod(n[:d])) % n[d]
        if c["ppc"]:  # uniformly random in each cell
            off = torch.rand((cells, ppc), generator=g, **f8)
        else:  # a jittered sub-lattice
            sub = (c["sub1"], c["sub2"], 1)[d]
            k = torch.arange(ppc, device=dev)
            k = k % c["sub1"] if d == 0 else (k // c["sub1"]) % sub
            off = (k + torch.rand((cells, ppc), generator=g, **f8)) / sub
        pos.append(torch.remainder(at[:, None] + off, n[d]).reshape(-1))
    x = torch.stack(pos)
    np_ = x.shape[1]
    u = c["sigma"] * torch.randn((3, np_), generator=g, **f8)
    u[0] += math.copysign(math.sqrt(c["gamma"] ** 2 - 1.0), c["gamma"])
    w = torch.full((cells, ppc), c["density"] / ppc, **f8)
    if c["spread"]:
        w *= 1.0 + c["spread"] * (2.0 * torch.rand((cells, 1), generator=g, **f8) - 1.0)
    w = w.reshape(-1).contiguous()
    gam = torch.sqrt(1.0 + (u * u).sum(0))
    jbg = (w * u / gam).sum(1) / cells  # q = -1: minus the electrons' mean current
    E = torch.zeros([3] + n[::-1], **f8)
    B = torch.zeros_like(E)
    if c["laser"] and dim == 2:
        E, B = _laser(c, E, B, f8)
    return dict(x=x, u=u, w=w, E=E, B=B, jbg=jbg)


def _laser(c, E, B, f8):
    """Gaussian pulse polarised along x3 moving in -x1, from its vector
    potential, at the Yee nodes."""
    a0, k0 = c["laser"], 1.0 / c["dx1"]
    L1, L2 = c["n1"] * c["dx1"], c["n2"] * c["dx2"]
    length, waist = L1 / 50.0, L2 / 12.0

    def grad(s1, s2):
        p = ((torch.arange(c["n1"], **f8) + s1) * c["dx1"] - 0.75 * L1)[None, :]
        q = ((torch.arange(c["n2"], **f8) + s2) * c["dx2"] - 0.5 * L2)[:, None]
        A = a0 * torch.exp(-(p / length) ** 2 - (q / waist) ** 2)
        return (A * (-2.0 * p / length ** 2 * torch.cos(k0 * p) - k0 * torch.sin(k0 * p)),
                A * torch.cos(k0 * p) * (-2.0 * q / waist ** 2))

    E[2] = -grad(0.0, 0.0)[0]
    B[0] = grad(0.0, 0.5)[1]
    B[1] = -grad(0.5, 0.0)[0]
    return E, B


def _inputs_q3d(c, g, f8):
    n1, n2, M, dz, dr = c["n1"], c["n2"], c["modes"], c["dx1"], c["dx2"]
    fill, nt = n2 - 10, 4  # the rest stays empty: particles may not reach the wall
    i = torch.arange(n1, **f8)[:, None, None, None] + (torch.arange(2, **f8)[:, None] + 0.5) / 2
    j = torch.arange(fill, **f8)[None, :, None, None] + 0.5
    th = 2.0 * math.pi * (torch.rand((n1, fill, 1, 1), generator=g, **f8) + torch.arange(nt, **f8) / nt)
    shape = (n1, fill, 2, nt)
    r = (j * dr).expand(shape)
    # a jitter inside the cell gives the column the field noise of a real load
    r = r + dr * (torch.rand(shape, generator=g, **f8) - 0.5)
    z = i + 0.5 * (torch.rand(shape, generator=g, **f8) - 0.5)
    x = torch.stack([torch.remainder(z, n1).reshape(-1) * dz, (r * torch.cos(th)).reshape(-1),
                     (r * torch.sin(th)).reshape(-1)])
    u = torch.zeros((3, x.shape[1]), **f8)
    u[0] = math.sqrt(c["gamma"] ** 2 - 1.0)
    w = (c["density"] * 2.0 * math.pi * r * dr * dz / (2 * nt)).reshape(-1)
    E = torch.zeros((M, 3, n2 + 1, n1), dtype=torch.complex128, device=f8["device"])
    B = torch.zeros_like(E)
    if M > 1 and c["laser"]:
        def pulse(sz, sr):
            p = ((torch.arange(n1, **f8) + sz) * dz - 0.75 * n1 * dz)[None, :]
            q = ((torch.arange(n2 + 1, **f8) + sr) * dr)[:, None]
            return c["laser"] * torch.exp(-(p / (n1 * dz / 50.0)) ** 2 - (q / (n2 * dr / 7.0)) ** 2) * \
                torch.cos(10.0 * p)
        E[1, 1], E[1, 2] = pulse(0.0, 0.5), 1j * pulse(0.0, 0.0)
        B[1, 1], B[1, 2] = 1j * pulse(0.5, 0.0), -pulse(0.5, 0.5)
        E[1, :, n2] = 0.0
        B[1, :, n2] = 0.0
    return dict(x=x, u=u, w=w, E=E, B=B)


# ------------------------------------------------------------------ the framework
def prepare(case, seed):
    runs = _runs(case)
    cfg = [hpic.config(c["n1"], c["n2"], c["dx1"], c["dx2"], c["dt"], precision=c["precision"],
                       n3=c["n3"], dx3=c["dx2"] if c["n3"] else 0.0, kmod=c["kmod"], modes=c["modes"],
                       interp=c["interp"], shape=c["shape"]) for c in runs]
    sim = hpic.Sim(cfg, stream=torch.cuda.current_stream())
    state = dict(sim=sim, case=runs[0], n=len(runs))
    for r, c in enumerate(runs):
        d = _inputs(c, seed * 1000 + r)
        if c["geom"] == "q3d":
            E, B = d["E"].cpu().numpy(), d["B"].cpu().numpy()
            for m in range(c["modes"]):
                sim.set_fields_mode(r, m, E[m], B[m])
            sim.set_particles(r, d["x"].cpu().numpy(), d["u"].cpu().numpy(), d["w"].cpu().numpy())
            sim.set_background(r, 2)
            continue
        dx = torch.tensor([c["dx1"], c["dx2"], c["dx2"]][: d["x"].shape[0]], dtype=torch.float64,
                          device=d["x"].device)
        sim.set_particles_device(r, (d["x"] * dx[:, None]).contiguous(), d["u"], d["w"])
        if c["laser"]:
            sim.set_fields(r, d["E"].cpu().numpy(), d["B"].cpu().numpy())
        sim.set_background(r, True, d["jbg"].cpu().numpy())
        if c["antenna"]:
            sim.set_antenna(r, **_antenna(c))
    c = runs[0]
    if c["sort"]:
        sim.set_tiling(c["tile1"], c["tile2"], c["sort"])
    if c["geom"] != "q3d":
        real = torch.float32 if c["precision"] == "fp32" else torch.float64
        state["fields"] = [torch.empty((6,) + sim.shape(r), dtype=real, device="cuda")
                           for r in range(len(runs))]
        if c["particles"]:
            state["u"] = [torch.empty((3, sim.count(r)), dtype=real, device="cuda")
                          for r in range(len(runs))]
            state["id"] = [torch.empty(sim.count(r), dtype=torch.int32, device="cuda")
                           for r in range(len(runs))]
    return state


def run(state):
    sim, c = state["sim"], state["case"]
    sim.step(c["steps"])
    if c["geom"] == "q3d":
        # the FP32 form's fields are FP32 values: kept as such
        kind = np.complex64 if c["precision"] == "fp32" else np.complex128
        out = {"Ez0": sim.field_mode(0, 0, 0).astype(kind, copy=False)}
        if c["modes"] > 1:
            out["Er1"] = sim.field_mode(0, 1, 1).astype(kind, copy=False)
        return out
    for r, F in enumerate(state["fields"]):
        for k in range(6):
            sim.field_device(r, k, F[k])
    out = {"fields": state["fields"]}
    if c["particles"]:
        out["u"] = []
        for r in range(state["n"]):
            sim.particles_device(r, u=state["u"][r], pid=state["id"][r])
            out["u"].append(torch.empty_like(state["u"][r]).index_copy_(1, state["id"][r].long(),
                                                                        state["u"][r]))
    return out


def work(case):
    """Per step: every particle's state read and written once, the fields of
    every node (and the master copy the next step starts from) read and written
    once; operations of gather, push, deposit and the row transforms."""
    total = {"bytes": 0.0, "flops": 0.0}
    for c in _runs(case):
        real = 4 if c["precision"] == "fp32" else 8
        if c["geom"] == "q3d":
            nodes = c["n1"] * (c["n2"] + 1) * c["modes"]
            parts = c["n1"] * (c["n2"] - 10) * 8
            pbytes = parts * (2 * (3 * 4 + 6 * real) + real)
            cbytes = nodes * (2 * 6 * 16 + 6 * 2 * real)
            pflops = parts * (400 + c["modes"] * (6 * 9 * 4 + 40 * 6))
            cflops = nodes * (9 * 5 * math.log2(c["n1"]) + 150)
        else:
            dim = 3 if c["n3"] else 2
            nodes = c["n1"] * c["n2"] * max(c["n3"], 1)
            parts = nodes * (c["ppc"] or c["sub1"] * c["sub2"])
            pbytes = parts * (2 * (4 + (dim + 3) * real) + real)
            cbytes = nodes * (2 * 6 * 8 + 6 * real)
            pflops = parts * (200 + 12 * (c["shape"] + 1) ** dim + 6 * (c["shape"] + 2) ** dim)
            cflops = nodes * (9 * 2.5 * math.log2(c["n1"]) + 75)
        total["bytes"] += c["steps"] * (pbytes + cbytes)
        total["flops"] += c["steps"] * (pflops + cflops)
    return total


# ------------------------------------------------------------------ the method in FP64
def _spline(order, d):
    a = d.abs()
    if order == 1:
        return (1.0 - a).clamp(min=0.0)
    if order == 2:
        return torch.where(a < 0.5, 0.75 - a * a, 0.5 * (1.5 - a).clamp(min=0.0) ** 2)
    return torch.where(a < 1.0, (4.0 - 6.0 * a * a + 3.0 * a ** 3) / 6.0, (2.0 - a).clamp(min=0.0) ** 3 / 6.0)


def _base(order, e):
    """First node of a spline's support around coordinate e."""
    return torch.floor(e + (0.5 if order % 2 == 0 else 0.0)) - order // 2


STAGGER = ((1, 0, 0), (0, 1, 0), (0, 0, 1), (0, 1, 1), (1, 0, 1), (1, 1, 0))  # E1 E2 E3 B1 B2 B3


def _boris(h, E, B, u):
    m = [u[k] + h * E[k] for k in range(3)]
    g = torch.sqrt(1.0 + m[0] ** 2 + m[1] ** 2 + m[2] ** 2)
    t = [h * B[k] / g for k in range(3)]
    s = [2.0 * v / (1.0 + t[0] ** 2 + t[1] ** 2 + t[2] ** 2) for v in t]

    def cross(a, b):
        return [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]

    p = [m[k] + v for k, v in enumerate(cross(m, t))]
    return torch.stack([m[k] + v + h * E[k] for k, v in enumerate(cross(p, s))])


def _symbols(c, n1, dx, dev, full):
    """i [k]1 xi+, i [k]1 xi-, the factor of Eq. (11) and the filter along the
    transform axis (``full``: complex transform, signed k1)."""
    kappa = torch.fft.fftfreq(n1, 1.0 / n1, dtype=torch.float64, device=dev) if full else \
        torch.arange(n1 // 2 + 1, dtype=torch.float64, device=dev)
    if full:
        kappa[n1 // 2] = n1 // 2
    a = kappa.abs()
    k1 = 2.0 * math.pi * a / (n1 * dx)
    kk = k1.clone()
    if c["kmod"]:
        kg = 2.0 * math.pi / dx
        kl, ku, km = 0.15 * kg, 0.26 * kg, 0.205 * kg
        bump = 0.01 * kg * torch.cos((k1 - km) / (kl - km) * math.pi / 2.0) ** 2
        kk = kk + torch.where((k1 >= kl) & (k1 <= ku), bump, torch.zeros_like(bump))
    h = 0.5 * k1 * dx
    dp = 1j * kk * torch.exp(1j * h)
    dm = 1j * kk * torch.exp(-1j * h)
    corr = torch.where(a > 0, torch.sin(h) / (0.5 * dx) / torch.where(a > 0, kk, torch.ones_like(kk)),
                       torch.ones_like(kk))
    neg = kappa < 0
    dp, dm = torch.where(neg, dp.conj(), dp), torch.where(neg, dm.conj(), dm)
    return dp, dm, corr, (a <= 0.25 * n1).to(torch.float64)


def _exact_cartesian(c, d):
    x, u, E, B, dt = d["x"].clone(), d["u"].clone(), d["E"].clone(), d["B"].clone(), c["dt"]
    dim = x.shape[0]
    n = [c["n1"], c["n2"], c["n3"]][:dim]
    dx = [c["dx1"], c["dx2"], c["dx2"]][:dim]
    stride = [math.prod(n[:k]) for k in range(dim)]
    qw, order, cells = -d["w"], c["shape"], math.prod(n)
    dev = x.device
    dp, dm, corr, filt = _symbols(c, n[0], dx[0], dev, False)
    up = [lambda f, k=k: (torch.roll(f, -1, -1 - k) - f) / dx[k] for k in range(dim)]
    dn = [lambda f, k=k: (f - torch.roll(f, 1, -1 - k)) / dx[k] for k in range(dim)]
    up[0], dn[0] = (lambda f: dp * f), (lambda f: dm * f)
    if dim == 2:
        up.append(lambda f: 0.0 * f)
        dn.append(lambda f: 0.0 * f)

    def curl(f, D):
        return torch.stack([D[1](f[2]) - D[2](f[1]), D[2](f[0]) - D[0](f[2]), D[0](f[1]) - D[1](f[0])])

    Ek, Bk = torch.fft.rfft(E), torch.fft.rfft(B)
    for step in range(c["steps"]):
        # gather
        w, at = {}, {}
        for k in range(dim):
            for s in (0, 1):
                o = order - 1 if (s and c["interp"]) else order
                e = x[k] - 0.5 * s
                b = _base(o, e)
                w[k, s] = [_spline(o, e - b - j) for j in range(o + 1)]
                at[k, s] = [torch.remainder(b.long() + j, n[k]) * stride[k] for j in range(o + 1)]
        got = []
        for comp, F in enumerate(list(E) + list(B)):
            F, st, acc = F.reshape(-1), STAGGER[comp], torch.zeros_like(x[0])
            for j2, w2 in enumerate(w[1, st[1]]):
                for j3 in range(len(w[2, st[2]]) if dim == 3 else 1):
                    row = at[1, st[1]][j2]
                    wr = w2
                    if dim == 3:
                        row, wr = row + at[2, st[2]][j3], wr * w[2, st[2]][j3]
                    for j1, w1 in enumerate(w[0, st[0]]):
                        acc += w1 * wr * F[row + at[0, st[0]][j1]]
            got.append(acc)
        u = _boris(-0.5 * dt, got[:3], got[3:], u)
        v = u / torch.sqrt(1.0 + (u * u).sum(0))
        new = torch.stack([x[k] + dt / dx[k] * v[k] for k in range(dim)])
        # deposit on windows that hold both stencils
        S0, S1, node = [], [], []
        for k in range(dim):
            b = torch.minimum(_base(order, x[k]), _base(order, new[k]))
            S0.append([_spline(order, x[k] - b - j) for j in range(order + 2)])
            S1.append([_spline(order, new[k] - b - j) for j in range(order + 2)])
            node.append([torch.remainder(b.long() + j, n[k]) * stride[k] for j in range(order + 2)])
        J = torch.zeros((3, cells), dtype=torch.float64, device=dev)
        R = range(order + 2)
        for k in range(dim):
            others = [(k + j) % dim for j in range(1, dim)]
            e, f = others[0], others[-1]
            g = -qw * dx[k] / dt
            for a in R:
                for b in (R if dim == 3 else (0,)):
                    if dim == 3:
                        T = (S0[e][a] * (2.0 * S0[f][b] + S1[f][b]) + S1[e][a] * (S0[f][b] + 2.0 * S1[f][b])) / 6.0
                        o = node[e][a] + node[f][b]
                    else:
                        T, o = 0.5 * (S0[e][a] + S1[e][a]), node[e][a]
                    acc = torch.zeros_like(qw)
                    for i in R[:-1]:
                        acc = acc + (S1[k][i] - S0[k][i])
                        J[k].index_add_(0, o + node[k][i], g * acc * T)
        if dim == 2:
            for a in R:
                for b in R:
                    W = (S0[0][a] * (2.0 * S0[1][b] + S1[1][b]) + S1[0][a] * (S0[1][b] + 2.0 * S1[1][b])) / 6.0
                    J[2].index_add_(0, node[0][a] + node[1][b], qw * v[2] * W)
        x = torch.stack([torch.remainder(new[k], n[k]) for k in range(dim)])
        J = J.reshape(E.shape)
        if c["antenna"]:
            J[2] += _antenna_current(c, (step + 0.5) * dt, dev)
        J += d["jbg"].reshape([3] + [1] * dim)
        Jk = torch.fft.rfft(J) * filt
        Jk[0] *= corr
        Bk = Bk - 0.5 * dt * curl(Ek, up)
        Ek = Ek + dt * (curl(Bk, dn) - Jk)
        Bk = Bk - 0.5 * dt * curl(Ek, up)
        E, B = torch.fft.irfft(Ek, n[0]), torch.fft.irfft(Bk, n[0])
    return torch.cat([E, B]), u


def _antenna_current(c, t, dev):
    a = _antenna(c)
    f8 = dict(dtype=torch.float64, device=dev)
    s = t - a["t0"]
    K = a["K0"] * math.sin(math.pi * s / a["T"]) ** 2 * math.sin(a["omega"] * s + a["phase"])
    K = K if 0.0 <= s <= a["T"] else 0.0
    L2 = c["n2"] * c["dx2"]
    y = torch.arange(c["n2"], **f8) * c["dx2"] - a["x2c"]
    y = y - L2 * torch.round(y / L2)
    e = torch.arange(c["n1"], **f8) - (a["x0"] + a["v"] * t) / c["dx1"]
    e = e - c["n1"] * torch.round(e / c["n1"])
    return K / c["dx1"] * torch.exp(-(y / a["waist"]) ** 2)[:, None] * _spline(2, e)[None, :]


def _exact_q3d(c, d):
    n1, n2, M, dz, dr, dt = c["n1"], c["n2"], c["modes"], c["dx1"], c["dx2"], c["dt"]
    x, u, qw = d["x"].clone(), d["u"].clone(), -d["w"]
    dev, pi = x.device, math.pi
    dp, dm, corr, filt = _symbols(c, n1, dz, dev, True)
    rows = torch.arange(n2 + 1, dtype=torch.float64, device=dev)
    area = 2.0 * pi * rows * dr * dr
    area[0] = 0.25 * pi * dr * dr
    F = torch.cat([d["E"], d["B"]], 1)  # [M][6][n2+1][n1]
    Fk = torch.fft.fft(F)

    def polar(p):
        r = torch.sqrt(p[1] ** 2 + p[2] ** 2)
        safe = torch.where(r > 0, r, torch.ones_like(r))
        ct = torch.where(r > 0, p[1] / safe, torch.ones_like(r))
        st = torch.where(r > 0, p[2] / safe, torch.zeros_like(r))
        return r / dr, ct, st

    # the co-drifting background: minus the z average of the electrons' current
    rho, _, _ = polar(x)
    vz = u[0] / torch.sqrt(1.0 + (u * u).sum(0))
    jbg = torch.zeros(n2 + 1, dtype=torch.float64, device=dev)
    b = _base(2, rho)
    for j in range(3):
        row = (b.long() + j).abs()
        jbg.index_add_(0, row, -qw * vz * _spline(2, rho - b - j) / (n1 * dz * area[row]))

    def faraday(Fk):
        Fk = Fk.clone()
        m = torch.arange(M, dtype=torch.float64, device=dev)[:, None, None]
        Ez, Er, Et = Fk[:, 0], Fk[:, 1], Fk[:, 2]
        j = rows[:n2, None]
        cz = ((j + 1) * Et[:, 1:] - j * Et[:, :n2]) / ((j + 0.5) * dr) - 1j * m / ((j + 0.5) * dr) * Er[:, :n2]
        ct = dp * Er[:, :n2] - (Ez[:, 1:] - Ez[:, :n2]) / dr
        cr = torch.zeros_like(cz)
        cr[:, 1:] = 1j * m / (j[1:] * dr) * Ez[:, 1:n2] - dp * Et[:, 1:n2]
        if M > 1:
            cr[1, 0] = 1j * Ez[1, 1] / dr - dp * Et[1, 0]
        Fk[:, 3, :n2] -= 0.5 * dt * cz
        Fk[:, 4, :n2] -= 0.5 * dt * cr
        Fk[:, 5, :n2] -= 0.5 * dt * ct
        return Fk

    def ampere(Fk, Jk):
        Fk = Fk.clone()
        m = torch.arange(M, dtype=torch.float64, device=dev)[:, None, None]
        Bz, Br, Bt = Fk[:, 3], Fk[:, 4], Fk[:, 5]
        j = rows[:n2, None]
        Fk[:, 1, :n2] += dt * (1j * m / ((j + 0.5) * dr) * Bz[:, :n2] - dm * Bt[:, :n2] - Jk[:, 1, :n2])
        j = j[1:]
        cz = ((j + 0.5) * Bt[:, 1:n2] - (j - 0.5) * Bt[:, : n2 - 1]) / (j * dr) - 1j * m / (j * dr) * Br[:, 1:n2]
        ct = dm * Br[:, 1:n2] - (Bz[:, 1:n2] - Bz[:, : n2 - 1]) / dr
        Fk[:, 0, 1:n2] += dt * (cz - Jk[:, 0, 1:n2])
        Fk[:, 2, 1:n2] += dt * (ct - Jk[:, 2, 1:n2])
        Fk[0, 0, 0] += dt * (4.0 * Bt[0, 0] / dr - Jk[0, 0, 0])
        if M > 1:
            Fk[1, 2, 0] += dt * (dm * Br[1, 0] - 2.0 * Bz[1, 0] / dr - Jk[1, 2, 0])
        return Fk

    for _ in range(c["steps"]):
        rho, ct, st = polar(x)
        w, at = {}, {}
        for k, e0 in enumerate((x[0] / dz, rho)):
            for s in (0, 1):
                o = 1 if (s and c["interp"]) else 2
                e = e0 - 0.5 * s
                b = _base(o, e)
                w[k, s] = [_spline(o, e - b - j) for j in range(o + 1)]
                at[k, s] = [b.long() + j for j in range(o + 1)]
        got = []
        for comp in range(6):
            sz, sr, _ = STAGGER[comp]
            acc = torch.zeros_like(qw)
            P = torch.ones_like(qw, dtype=torch.complex128)
            for m in range(M):
                v = torch.zeros_like(P)
                for jr, wr in enumerate(w[1, sr]):
                    row = at[1, sr][jr]
                    ghost = row < 0
                    sign = (-1.0) ** m * (1.0 if comp in (0, 3) else -1.0)
                    wr = torch.where(ghost, sign * wr, wr)
                    row = torch.where(ghost, -row - 1 if sr else -row, row)
                    for jz, wz in enumerate(w[0, sz]):
                        v += wz * wr * F[m, comp].reshape(-1)[row * n1 + torch.remainder(at[0, sz][jz], n1)]
                acc += (v * P.conj()).real
                P = P * (ct - 1j * st)
            got.append(acc)
        Ec = [got[0], got[1] * ct - got[2] * st, got[1] * st + got[2] * ct]
        Bc = [got[3], got[4] * ct - got[5] * st, got[4] * st + got[5] * ct]
        u = _boris(-0.5 * dt, Ec, Bc, u)
        new = x + dt * u / torch.sqrt(1.0 + (u * u).sum(0))
        rhob, ctb, stb = polar(new)
        S, base = [], []
        for e0, e1 in ((x[0] / dz, new[0] / dz), (rho, rhob)):
            b = torch.minimum(_base(2, e0), _base(2, e1))
            S.append([[_spline(2, e - b - j) for j in range(4)] for e in (e0, e1)])
            base.append(b.long())
        (Z0, Z1), (R0, R1) = S
        col = [torch.remainder(base[0] + a, n1) for a in range(4)]
        mid = 0.5 * (x + new)
        rm = torch.sqrt(mid[1] ** 2 + mid[2] ** 2)
        vth = torch.where(rm > 0, (mid[1] * (new[2] - x[2]) - mid[2] * (new[1] - x[1])) /
                          torch.where(rm > 0, rm * dt, torch.ones_like(rm)), torch.zeros_like(rm))
        J = torch.zeros((M, 3, (n2 + 1) * n1, 2), dtype=torch.float64, device=dev)

        def add(m, comp, at_, val):
            J[m, comp].index_add_(0, at_, torch.view_as_real(val))

        P0 = torch.ones_like(qw, dtype=torch.complex128)
        P1 = P0.clone()
        for m in range(M):
            cm, sm = (1.0, 1.0) if m == 0 else (2.0, (-1.0) ** m)
            Pm = 0.5 * (P0 + P1)
            q = -cm * qw * Pm
            for b in range(4):
                row = base[1] + b
                ghost = row < 0
                arow = row.abs()
                one = torch.ones_like(qw)
                f = torch.where(ghost, sm * one, one)
                acc = torch.zeros_like(qw)
                for a in range(3):
                    acc = acc + (Z1[a] - Z0[a]) * 0.5 * (R0[b] + R1[b])
                    add(m, 0, arow * n1 + col[a], q * (f * acc / (area[arow] * dt)))
                face = row.clamp(min=0)
                run_r = sum(R1[j] - R0[j] for j in range(b + 1))
                if b < 3:
                    ff = torch.where(ghost, -sm * one, one) / (2.0 * pi * (face + 0.5) * dr * dz * dt)
                    for a in range(4):
                        add(m, 1, face * n1 + col[a], q * (ff * run_r * 0.5 * (Z0[a] + Z1[a])))
                for a in range(4):
                    W3 = (Z0[a] * (2.0 * R0[b] + R1[b]) + Z1[a] * (R0[b] + 2.0 * R1[b])) / 6.0
                    direct = torch.where(ghost, -sm * one, one) * cm * qw * W3 * vth / (area[arow] * dz) * Pm
                    if m == 0:
                        val = direct
                    else:
                        Wb = 0.5 * (Z0[a] * R0[b] + Z1[a] * R1[b])
                        flux = 1j * cm * qw * Wb * (P1 - P0) / (m * dt) * f / (2.0 * pi * dr * dz)
                        axis = direct if m == 1 else torch.zeros_like(flux)
                        val = torch.where(row == 0, axis, flux)
                    add(m, 2, arow * n1 + col[a], val)
            P0, P1 = P0 * (ct - 1j * st), P1 * (ctb - 1j * stb)
        Jc = torch.view_as_complex(J).reshape(M, 3, n2 + 1, n1)
        Jc[0, 0] += jbg[:, None]
        Jk = torch.fft.fft(Jc) * filt
        Jk[:, 0] *= corr
        Fk = faraday(ampere(faraday(Fk), Jk))
        F = torch.fft.ifft(Fk)
        x = new
        x[0] = torch.remainder(x[0], n1 * dz)
    return F


def exact(case, seed):
    out = {"fields": [], "u": []}
    for r, c in enumerate(_runs(case)):
        d = _inputs(c, seed * 1000 + r)
        if c["geom"] == "q3d":
            F = _exact_q3d(c, d)
            got = {"Ez0": F[0, 0].cpu().numpy()}
            if c["modes"] > 1:
                got["Er1"] = F[1, 1].cpu().numpy()
            return got
        F, u = _exact_cartesian(c, d)
        out["fields"].append(F)
        out["u"].append(u)
    if not c["particles"]:
        del out["u"]
    return out
