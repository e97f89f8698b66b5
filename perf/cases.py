"""The work that users of lib_llgdisk have it do, as timed cases.

Every case goes through the package's public entry points the way the studies
in `experiments/`, the tests and `bench.py` call them: field evaluations, the
two integrators on a lone disk, on ragged ensembles and on thermal replicas,
their observable series, sampled observables, the adjoint of a trajectory
loss, constrained relaxation and power spectra.  Permalloy on a = 2 nm cells.

* `listed()`: the named cases; `draw(rng)`: one more of the same ranges;
* `prepare(case, seed)`: handle, launch plan, parameters and inputs;
* `run(state)`: one pass; the integrators step the state in place;
* `work(case)`: bytes and floating point operations a pass cannot do without;
* `exact(case, seed)`: what `run` returns, from the formulas in float64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1207_2192_amd as llg
from paper_1207_2192_amd.adjoint import core_trajectory

A_NM = 2.0
C_PY = 0.14298555               # a^2 / lambda_ex^2 of Permalloy on 2 nm cells
LAMBDA_NM = A_NM / math.sqrt(C_PY)
A_EX = 13e-12                   # exchange stiffness, J/m
KB = 1.380649e-23
DESCENT = 3e-4                  # step length of the fit of (alpha, c)
CUTOFF = 4.0 * LAMBDA_NM / A_NM  # radius of the core-position weights, cells


def listed():
    return [
        # the smallest call: the field of one small disk, on the plan a new handle has (latency)
        dict(name="field_small", kind="field", n=1, d_min=30, d_max=30, lor="0.333"),
        # right-hand side of a lone disk with an odd box, the last row pair half empty
        dict(name="rhs_odd", kind="rhs", n=1, d_min=125, d_max=125, lor="0.16"),
        # T = 0 dynamics of one small disk between two samples (R = 30 nm, L = 10 nm)
        dict(name="rk4_small", kind="rk4", n=1, d_min=30, d_max=30, lor="0.333", steps=100, alpha=0.01),
        # gyrotropic run of one disk, undamped (R = 100 nm, L = 20 nm)
        dict(name="rk4_lone", kind="rk4", n=1, d_min=100, d_max=100, lor="0.2", steps=100, alpha=0.0),
        # ragged ensemble, R = 30 .. 120 nm at three aspect ratios, one launch
        dict(name="rk4_ragged", kind="rk4", n=256, d_min=30, d_max=120, lor="0.1,0.2,0.3", steps=20, alpha=0.02),
        # thermal replicas of a large disk (R = 250 nm, L = 20 nm, 300 K): the most memory and cells
        dict(name="heun_replicas", kind="heun", n=64, d_min=250, d_max=250, lor="0.08", steps=20, alpha=0.1,
             kelvin=300.0, dtau=0.0266, renorm=True),
        # thermal campaign of small disks with the <m>, E series every 50 steps (R = 30 nm, L = 5 and 10 nm)
        dict(name="series_thermal", kind="heun_series", n=64, d_min=30, d_max=30, lor="0.167,0.333", steps=250,
             every=50, alpha=0.02, kelvin=300.0, dtau=0.04, renorm=True),
        # resonance sweep: one small disk per drive frequency, series every 50 steps
        dict(name="series_driven", kind="rk4_series", n=16, d_min=30, d_max=30, lor="0.333", steps=250, every=50,
             alpha=0.05, drive=0.004),
        # observables of the replicas between launches: core position, energy, <m>
        dict(name="observe_replicas", kind="observe", n=64, d_min=250, d_max=250, lor="0.08"),
        # trajectory loss, its gradient in m_0 and a descent step in (alpha, c) (R = 80 nm, L = 10 nm), two segments
        dict(name="adjoint_rk4", kind="adjoint", n=1, d_min=80, d_max=80, lor="0.125", segments=2, steps=50,
             alpha=0.01, noise=False),
        # stiffness sweep: R in 30 .. 120 nm at three thicknesses, three targets each, a fixed number of sweeps
        dict(name="relax_sweep", kind="relax", n=36, d_min=30, d_max=120, lor="0.1,0.2,0.3", sweeps=500),
        # spectra of the recorded <m_x> of a campaign: segments of 4096 samples
        dict(name="spectra", kind="spectrum", n=96, length=4096, window="none", mean=True),
    ]


def draw(rng):
    """A case of the listed ranges: sizes over their logarithm, odd boxes among them."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def box(lo=12, hi=250):
        return log_int(lo, hi)

    def copies(d, most, cells):      # as many disks as stay within a number of cells
        return log_int(1, max(1, min(most, cells // (d * d))))

    lor = "%.3f" % rng.uniform(0.05, 0.3)
    kind = rng.choice(["field", "rhs", "rk4", "ragged", "heun", "heun_series", "rk4_series", "observe", "adjoint",
                       "relax", "spectrum"])
    if kind in ("field", "rhs", "observe"):
        d = box()
        return dict(kind=kind, n=copies(d, 64, 4_000_000), d_min=d, d_max=d, lor=lor)
    if kind == "rk4":
        d = box()
        return dict(kind="rk4", n=1, d_min=d, d_max=d, lor=lor, steps=log_int(8, 100), alpha=rng.choice([0.0, 0.02]))
    if kind == "ragged":
        lo = box(16, 60)
        hi = rng.randint(lo + 5, 120)
        return dict(kind="rk4", n=log_int(12, 256), d_min=lo, d_max=hi, lor="0.1,%s" % lor, steps=log_int(4, 20),
                    alpha=0.02)
    if kind == "heun":
        d = box()
        return dict(kind="heun", n=copies(d, 64, 4_000_000), d_min=d, d_max=d, lor=lor, steps=log_int(4, 20),
                    alpha=rng.choice([0.02, 0.1]), kelvin=rng.choice([150.0, 300.0]), dtau=rng.choice([0.0266, 0.04]),
                    renorm=rng.random() < 0.7)
    if kind == "heun_series":
        d = box(20, 120)
        every = rng.choice([10, 25, 50])
        return dict(kind="heun_series", n=copies(d, 64, 60_000), d_min=d, d_max=d, lor=lor, every=every,
                    steps=every * rng.randint(1, 4) + rng.randint(0, 3), alpha=0.02, kelvin=300.0, dtau=0.04,
                    renorm=True)
    if kind == "rk4_series":
        d = box(20, 120)
        every = rng.choice([10, 25, 50])
        return dict(kind="rk4_series", n=copies(d, 16, 60_000), d_min=d, d_max=d, lor=lor, every=every,
                    steps=every * rng.randint(1, 4) + rng.randint(0, 3), alpha=0.05, drive=0.004)
    if kind == "adjoint":
        d = box(24, 100)
        return dict(kind="adjoint", n=1, d_min=d, d_max=d, lor="%.3f" % rng.uniform(0.1, 0.3),
                    segments=rng.randint(1, 3), steps=log_int(6, 30), alpha=rng.choice([0.01, 0.05]),
                    noise=rng.random() < 0.4)
    if kind == "relax":
        lo = box(24, 60)
        return dict(kind="relax", n=log_int(1, 36), d_min=lo, d_max=rng.randint(lo, 120), lor="0.15,%s" % lor,
                    sweeps=log_int(200, 340))
    length = 2 ** rng.randint(8, 16)
    return dict(kind="spectrum", n=log_int(1, max(2, min(96, 400_000 // length))), length=length,
                window=rng.choice(["none", "hann"]), mean=rng.random() < 0.8)


# ---------------------------------------------------------------- inputs
def shapes(case):
    """(D, L in nm) of every disk of a case: box sizes over [d_min, d_max] in up to
    ten steps, each at the case's aspect ratios L/R; equal geometries repeat."""
    lo, hi, ratios = case["d_min"], case["d_max"], [float(x) for x in case["lor"].split(",")]
    boxes = sorted({lo + round(k * (hi - lo) / 9) for k in range(10)})
    out = []
    for k in range(case["n"]):
        d = boxes[(7 * k) % len(boxes)]
        out.append((d, round(ratios[(k // len(boxes)) % len(ratios)] * d * A_NM / 2.0, 2)))
    return out


def start_states(case, seed):
    """One float32 [3, D, D] vortex per disk: seeded displacement, polarity and
    chirality; thermal cases (and fields) carry a seeded tilt of every cell."""
    rng = np.random.default_rng(seed)
    rough = 0.1 if case["kind"] in ("heun", "heun_series", "observe", "field", "rhs") else 0.0
    out = []
    for k, (d, _) in enumerate(shapes(case)):
        c = np.arange(d, dtype=np.float64) - (d - 1) / 2.0
        y, x = np.meshgrid(c, c, indexing="ij")
        reach = min(rng.uniform(1.0, 5.0), 0.12 * d)
        ang, x0, y0 = rng.uniform(0.0, 2.0 * math.pi), 0.013, 0.017
        if case["kind"] == "relax":                     # next to the target position
            reach *= 0.02
            x0, y0 = targets(case)[k][0] / A_NM, 0.0
        dx, dy = x - x0 - reach * math.cos(ang), y - y0 - reach * math.sin(ang)
        phi = np.arctan2(dy, dx) + rng.choice([-1.0, 1.0]) * math.pi / 2.0
        mz = rng.choice([-1.0, 1.0]) * np.exp(-(dx * dx + dy * dy) / (2.0 * 2.5 ** 2))
        s = np.sqrt(1.0 - mz * mz)
        v = np.stack([s * np.cos(phi), s * np.sin(phi), mz])
        if rough:
            v += rough * rng.standard_normal(v.shape, dtype=np.float32)
        v /= np.linalg.norm(v, axis=0, keepdims=True)
        out.append(torch.from_numpy(v.astype(np.float32)))
    return out


def temperature(case, L):
    return KB * case.get("kelvin", 0.0) / (2.0 * A_EX * L * 1e-9)


def drive_frequency(k):
    return 0.0004 + 0.00006 * k      # cycles per unit of tau, around the gyration of small disks


def params(case):
    out = []
    for k, (_, L) in enumerate(shapes(case)):
        p = llg.LLGParams(alpha=case.get("alpha", 0.0), c=C_PY, dtau=case.get("dtau", 0.04),
                          temp=temperature(case, L), renorm=case.get("renorm", False))
        if case.get("drive"):
            p.hac, p.freq = (case["drive"], 0.0, 0.0), drive_frequency(k)
        out.append(p)
    return out


def targets(case):
    """Target positions (nm) of a relaxation: 0, one and two cells off the centre."""
    return [((k % 3) * A_NM, 0.0) for k in range(case["n"])]


def noise_of(case, seed):
    return (1000 + seed, 0, 0) if case["noise"] else None


def signals(case, seed):
    """Recorded <m_x>: a slow line, a doublet and noise, [n, length] float64."""
    rng = np.random.default_rng(seed)
    t = np.arange(case["length"], dtype=np.float64)
    f = rng.uniform(0.001, 0.4, size=(case["n"], 3, 1))
    a = rng.uniform(0.002, 0.05, size=(case["n"], 3, 1))
    x = (a * np.sin(2.0 * math.pi * f * t + rng.uniform(0.0, 6.28, size=(case["n"], 3, 1)))).sum(axis=1)
    return torch.from_numpy(x + 0.01 + 0.003 * rng.standard_normal(x.shape))


def adjoint_params(case):
    d, L = shapes(case)[0]
    return llg.LLGParams(c=C_PY, dtau=0.04, temp=KB * 300.0 / (2.0 * A_EX * L * 1e-9) if case["noise"] else 0.0,
                         renorm=case["noise"])


def target_path(case, seed, like):
    """Core positions (nm) to be reached: an inward spiral on one side of the start."""
    rng = np.random.default_rng(seed + 77)
    r0, a0 = rng.uniform(14.0, 18.0), rng.uniform(0.0, 2.0 * math.pi)
    k = np.arange(case["segments"] + 1)
    path = np.stack([r0 * 0.98 ** k * np.cos(a0 + 0.05 * k), r0 * 0.98 ** k * np.sin(a0 + 0.05 * k)], axis=1)
    return torch.tensor(path, dtype=torch.float32).to(like.device)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "spectrum":
        return dict(case=case, x=signals(case, seed).cuda())
    geo = shapes(case)
    R, L = [d * A_NM / 2.0 for d, _ in geo], [t for _, t in geo]
    disk = llg.Disk.batch(R, L, A_NM) if case["n"] > 1 else llg.Disk.build(R[0], L[0], A_NM)
    m = disk.pack(start_states(case, seed)).cuda()
    state = dict(case=case, disk=disk, m=m, seed=seed)
    if kind == "adjoint":
        state["params"] = adjoint_params(case)
        state["target"] = target_path(case, seed, m)
        state["theta"] = torch.tensor([case["alpha"], C_PY], requires_grad=True)     # fitted parameters: alpha, c
        state["m"] = m.requires_grad_(True)
        return state
    state["params"] = params(case)
    if kind.endswith("series"):      # the campaign's record: as many digits as the float32 states behind it have
        state["record"] = torch.empty(-(-case["steps"] // case["every"]), case["n"], 4, device=m.device)
    if kind in ("rk4", "rk4_series"):
        disk.autotune(m, state["params"], "rk4", probe_steps=10)
    if kind in ("heun", "heun_series"):
        disk.autotune(m, state["params"], "heun", probe_steps=10)
        disk.set_step(0)
    if kind == "relax":
        state["X"] = targets(case)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "spectrum":
        return llg.power_spectrum(state["x"], case["mean"], case["window"])
    disk, m, prm = state["disk"], state["m"], state["params"]
    if kind == "field":
        return disk.demag_field(m)
    if kind == "rhs":
        return disk.rhs(m, prm)
    if kind == "rk4":
        return disk.rk4_step(m, case["steps"], prm)
    if kind == "heun":
        return disk.heun_step(m, case["steps"], prm, seed=state["seed"], step0=None)
    if kind == "rk4_series":
        series = disk.rk4_series(m, case["steps"], prm, case["every"])
        return dict(series=state["record"].copy_(series), m=m)
    if kind == "heun_series":
        series = disk.heun_series(m, case["steps"], prm, case["every"], seed=state["seed"], step0=None)
        return dict(series=state["record"].copy_(series), m=m)
    if kind == "observe":
        return dict(core=disk.vortex_core_position(m, LAMBDA_NM), energy=disk.energy(m, prm), mean=disk.mean_m(m))
    if kind == "relax":
        m = m.clone()                # every pass relaxes the same start states
        record = disk.relax(m, state["X"], prm, tol=1e-12, max_sweeps=case["sweeps"], cutoff_nm=4.0 * LAMBDA_NM)
        return dict(m=m, record=record.float())      # multipliers and residual of a float32 state
    assert kind == "adjoint"
    theta = state["theta"]
    rc = core_trajectory(m, theta[0], theta[1], disk, prm, case["segments"], case["steps"], LAMBDA_NM,
                         noise_of(case, state["seed"])).float()
    loss = ((rc - state["target"]) ** 2).sum()
    gm, gt = torch.autograd.grad(loss, [m, theta])
    return dict(path=rc.detach(), m=gm, theta=theta.detach() - DESCENT * gt)


# ---------------------------------------------------------------- what a pass needs
def field_flops(d):
    """One field evaluation and stage update of a D x D box: three real transforms each
    way over the padded square (rows past the box are zero), the spectral product and
    about a hundred operations per cell."""
    p = 64
    while p < 2 * d:
        p *= 2
    lg, h = math.log2(p), p // 2 + 1
    return 2 * (3 * d * 2.5 * p * lg + 3 * h * 5.0 * p * lg) + 20.0 * h * p + 100.0 * d * d


def work(case):
    kind = case["kind"]
    if kind == "spectrum":
        n, length = case["n"], case["length"]
        return {"bytes": n * (8.0 * length + 8.0 * (length // 2 + 1)), "flops": n * 2.5 * length * math.log2(length)}
    geo = shapes(case)
    cells = sum(d * d for d, _ in geo)
    spec = sum(16.0 * (d + 1) ** 2 for d, _ in set(geo))      # kernel spectra of every geometry, read once
    evals = {"field": 1, "rhs": 1, "observe": 1, "rk4": 4 * case.get("steps", 0), "rk4_series": 4 * case.get("steps", 0),
             "heun": 2 * case.get("steps", 0), "heun_series": 2 * case.get("steps", 0),
             "relax": case.get("sweeps", 0)}.get(kind)
    if kind == "adjoint":                # forward, recomputation, reverse sweep
        evals = 3 * (2 if case["noise"] else 4) * case["segments"] * case["steps"]
    moved = (12.0 if kind == "observe" else 24.0) * cells + spec
    return {"bytes": moved, "flops": evals * sum(field_flops(d) for d, _ in geo)}


# ---------------------------------------------------------------- float64 values
class Reference:
    """Field, torque and observables of one geometry in float64, batched over disks."""

    def __init__(self, d, L, device):
        self.d, self.p, self.ell = d, 2 * d, L / A_NM
        g = torch.arange(-(d - 1), d, dtype=torch.float64, device=device)
        v, u = torch.meshgrid(g, g, indexing="ij")
        r2 = u * u + v * v
        r2[d - 1, d - 1] = 1.0
        ell = self.ell
        r, s = torch.sqrt(r2), torch.sqrt(r2 + ell * ell)
        pre = ell / (2.0 * math.pi * r2 * r2)
        kern = torch.stack([pre * (u * u / s - v * v / (s + r)), pre * (v * v / s - u * u / (s + r)),
                            pre * (2.0 * s + r) / (s + r) * u * v / s,
                            -ell / (2.0 * math.pi * r * s * (s + r))])
        ro = 1.0 / math.sqrt(math.pi)
        so = math.sqrt(ell * ell + ro * ro)
        nx, nz = (so - ro) / (2.0 * ell), (ell + ro - so) / ell
        kern[:, d - 1, d - 1] = torch.tensor([-nx, -nx, 0.0, -nz], dtype=torch.float64, device=device)
        wrap = torch.zeros(4, self.p, self.p, dtype=torch.float64, device=device)
        at = torch.arange(-(d - 1), d, device=device) % self.p
        wrap[:, at[:, None], at[None, :]] = kern
        self.k = torch.fft.rfft2(wrap)
        c = torch.arange(d, dtype=torch.float64, device=device) - (d - 1) / 2.0
        self.y, self.x = torch.meshgrid(c, c, indexing="ij")
        self.mask = (self.x ** 2 + self.y ** 2 <= (d / 2.0) ** 2).to(torch.float64)

    def demag(self, m):
        f = torch.fft.rfft2(m * self.mask, s=(self.p, self.p))
        kxx, kyy, kxy, kzz = self.k
        fx, fy, fz = f[:, 0], f[:, 1], f[:, 2]
        h = torch.fft.irfft2(torch.stack([kxx * fx + kxy * fy, kxy * fx + kyy * fy, kzz * fz], dim=1),
                             s=(self.p, self.p))
        return h[:, :, :self.d, :self.d] * self.mask

    def exchange(self, m):
        q = torch.nn.functional.pad(m * self.mask, (1, 1, 1, 1))
        return (q[:, :, 2:, 1:-1] + q[:, :, :-2, 1:-1] + q[:, :, 1:-1, 2:] + q[:, :, 1:-1, :-2]) * self.mask

    def torque(self, m, b, alpha):
        mxb = torch.linalg.cross(m, b, dim=1)
        return (mxb - alpha * torch.linalg.cross(m, mxb, dim=1)) * self.mask

    def normalise(self, m):
        n = torch.linalg.vector_norm(m, dim=1, keepdim=True)
        return m / torch.where(n > 0, n, torch.ones_like(n)) * self.mask

    def energy(self, m, h, c):
        """(E, exchange, demag, external) per disk; h: external field [n, 3, 1, 1]."""
        mm = m * self.mask
        ex = -0.5 * (mm * self.exchange(mm)).sum(dim=(1, 2, 3))
        dm = -0.5 * c * (mm * self.demag(mm)).sum(dim=(1, 2, 3))
        xt = -c * (mm * h).sum(dim=(1, 2, 3))
        return torch.stack([ex + dm + xt, ex, dm, xt], dim=1)

    def mean(self, m):
        return (m * self.mask).sum(dim=(2, 3)) / self.mask.sum()

    def core_set(self, m):
        """The +1 plaquette (corner, cells from the centre), their number and the weights' mask."""
        ph = torch.atan2(m[1], m[0])

        def wrap(t):
            return torch.remainder(t + math.pi, 2.0 * math.pi) - math.pi
        a, b, c, e = ph[:-1, :-1], ph[:-1, 1:], ph[1:, 1:], ph[1:, :-1]
        k = self.mask
        inside = k[:-1, :-1] * k[:-1, 1:] * k[1:, 1:] * k[1:, :-1] > 0
        wind = torch.round((wrap(b - a) + wrap(c - b) + wrap(e - c) + wrap(a - e)) / (2.0 * math.pi))
        hit = (wind == 1) & inside
        n = int(hit.sum())
        if n == 0:
            return math.nan, math.nan, 0, k
        z = m[2] ** 2
        score = torch.where(hit, z[:-1, :-1] + z[:-1, 1:] + z[1:, 1:] + z[1:, :-1], torch.full_like(a, -1.0))
        at = int(torch.argmax(score.reshape(-1)))
        j, i = divmod(at, self.d - 1)
        xv, yv = i - (self.d - 1) / 2.0 + 0.5, j - (self.d - 1) / 2.0 + 0.5
        near = ((self.x - xv) ** 2 + (self.y - yv) ** 2 < CUTOFF * CUTOFF).to(torch.float64) * k
        return xv, yv, n, near

    def centroid(self, m, near):
        w = m[2] ** 2 * near
        return torch.stack([(w * self.x).sum(), (w * self.y).sum()]) / w.sum() * A_NM


def normals(seed, step, replicas, d, device):
    """The noise [len(replicas), 3, D, D] of one Heun step (Philox4x32-10, Box-Muller)."""
    M32 = 0xFFFFFFFF
    pairs = (d + 1) // 2
    q = torch.arange(pairs * d, dtype=torch.int64, device=device)
    rep = torch.tensor(replicas, dtype=torch.int64, device=device)[:, None]

    def hi_lo(const, w):
        # 32 x 32 -> 64 bits by 16-bit halves (int64 is signed)
        low = const * (w & 0xFFFF)
        mid = const * (w >> 16) + (low >> 16)
        return (mid >> 16) & M32, ((mid & 0xFFFF) << 16) | (low & 0xFFFF)

    def block(h):
        shape = (len(replicas), pairs * d)
        c0, c1 = torch.full(shape, step & M32, device=device), torch.full(shape, step >> 32, device=device)
        c2, c3 = (2 * q + h).expand(shape) & M32, rep.expand(shape) & M32
        k0, k1 = seed & M32, (seed >> 32) & M32
        for _ in range(10):
            h0, l0 = hi_lo(0xD2511F53, c0)
            h1, l1 = hi_lo(0xCD9E8D57, c2)
            c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
            k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
        return [((c >> 8).to(torch.float64) + 0.5) * 2.0 ** -24 for c in (c0, c1, c2, c3)]
    u = block(0) + block(1)[:2]
    n = []
    for k in range(3):
        rad, ang = torch.sqrt(-2.0 * torch.log(u[2 * k])), 2.0 * math.pi * u[2 * k + 1]
        n += [rad * torch.cos(ang), rad * torch.sin(ang)]
    both = torch.stack([torch.stack(n[:3], dim=1), torch.stack(n[3:], dim=1)], dim=1)    # [r, row of the pair, 3, pairs*D]
    w = both.reshape(len(replicas), 2, 3, pairs, d).permute(0, 2, 3, 1, 4).reshape(len(replicas), 3, 2 * pairs, d)
    return w[:, :, :d]


class Group:
    """The disks of one geometry of a case: states [n, 3, D, D] and per-disk columns of the parameters."""

    def __init__(self, case, geo, at, states, device):
        self.case, self.at = case, at
        self.ref = Reference(*geo, device)
        self.m = torch.stack([states[k] for k in at]).to(device=device, dtype=torch.float64)
        self.dt, self.alpha = case.get("dtau", 0.04), case.get("alpha", 0.0)
        temp = temperature(case, geo[1])
        self.sigma = math.sqrt(2.0 * self.alpha * temp * self.dt)
        self.freq = torch.tensor([drive_frequency(k) for k in at], dtype=torch.float64, device=device)

    def h(self, tau):
        f = torch.zeros(len(self.at), 3, 1, 1, dtype=torch.float64, device=self.m.device)
        if self.case.get("drive"):
            f[:, 0, 0, 0] = self.case["drive"] * torch.sin(2.0 * math.pi * self.freq * tau)
        return f

    def b(self, m, tau, c=C_PY):
        return self.ref.exchange(m) + c * (self.h(tau) + self.ref.demag(m))

    def rhs(self, m, tau, alpha=None, c=C_PY):
        return self.ref.torque(m, self.b(m, tau, c), self.alpha if alpha is None else alpha)

    def rk4(self, m, n, alpha=None, c=C_PY):
        dt, t = self.dt, n * self.dt
        k1 = self.rhs(m, t, alpha, c)
        k2 = self.rhs(m + 0.5 * dt * k1, t + 0.5 * dt, alpha, c)
        k3 = self.rhs(m + 0.5 * dt * k2, t + 0.5 * dt, alpha, c)
        k4 = self.rhs(m + dt * k3, t + dt, alpha, c)
        return m + dt / 6.0 * (k1 + 2.0 * k2 + 2.0 * k3 + k4)

    def heun(self, m, w, sigma, alpha, c, renorm):
        def delta(x):
            return self.ref.torque(x, self.b(x, 0.0, c) * self.dt + sigma * w, alpha)
        d1 = delta(m)
        out = m + 0.5 * (d1 + delta(m + d1))
        return self.ref.normalise(out) if renorm else out

    def advance(self, n, seed):
        if self.case["kind"].startswith("heun"):
            w = normals(seed, n, self.at, self.ref.d, self.m.device)
            self.m = self.heun(self.m, w, self.sigma, self.alpha, C_PY, self.case["renorm"])
        else:
            self.m = self.rk4(self.m, n)

    def sample(self, n):
        return torch.cat([self.ref.mean(self.m), self.ref.energy(self.m, self.h(n * self.dt), C_PY)[:, :1]], dim=1)


def relaxed(group, X, sweeps):
    """Constrained alignment sweeps: states and the record (lambda, sweeps, residual, C) of each disk."""
    ref, m = group.ref, group.m * group.ref.mask
    X = torch.tensor(X, dtype=torch.float64, device=m.device) / A_NM
    dx, dy = ref.x - X[:, 0, None, None], ref.y - X[:, 1, None, None]
    near = (dx * dx + dy * dy < CUTOFF * CUTOFF).to(torch.float64) * ref.mask
    dx, dy = dx * near, dy * near
    lam = torch.zeros(len(X), 2, dtype=torch.float64, device=m.device)

    def total(w):
        return w.sum(dim=(1, 2))
    for _ in range(sweeps):
        bl = 2.0 * m[:, 2] * (lam[:, 0, None, None] * dx + lam[:, 1, None, None] * dy)
        b = group.b(m, 0.0)
        b = torch.stack([b[:, 0], b[:, 1], b[:, 2] + bl], dim=1)
        res = torch.linalg.vector_norm(torch.linalg.cross(m, b, dim=1), dim=1).mul(ref.mask).amax(dim=(1, 2))
        w0 = m[:, 2] ** 2
        C = torch.stack([total(w0 * dx), total(w0 * dy)], dim=1)
        t = b + 2.0 * m
        tn = torch.linalg.vector_norm(t, dim=1)
        tn = torch.where(tn > 0, tn, torch.ones_like(tn))
        m = t / tn[:, None] * ref.mask
        w1 = m[:, 2] ** 2
        gj = 4.0 * w1 * (1.0 - w1) / tn
        jxx, jxy, jyy = total(gj * dx * dx), total(gj * dx * dy), total(gj * dy * dy)
        cx, cy, det = total(w1 * dx), total(w1 * dy), jxx * jyy - jxy * jxy
        ok = det != 0
        det = torch.where(ok, det, torch.ones_like(det))
        lam = lam - torch.stack([(jyy * cx - jxy * cy) / det, (jxx * cy - jxy * cx) / det], dim=1) * ok[:, None]
    zero = torch.zeros_like(res)
    return m, torch.stack([lam[:, 0], lam[:, 1], zero + sweeps, res, C[:, 0], C[:, 1], zero, zero], dim=1)


def exact_adjoint(case, seed, group, states, device):
    m = states[0].to(device=device, dtype=torch.float64).requires_grad_(True)
    theta = torch.tensor([case["alpha"], C_PY]).to(device=device, dtype=torch.float64).requires_grad_(True)
    al, c = theta[0], theta[1]
    prm = adjoint_params(case)
    x, path, step = m[None], [], 0
    near = group.ref.core_set(m.detach() * group.ref.mask)[3]
    path.append(group.ref.centroid(m, near))
    x = x * group.ref.mask
    for _ in range(case["segments"]):
        for _ in range(case["steps"]):
            if case["noise"]:
                w = normals(1000 + seed, step, [0], group.ref.d, device)
                x = group.heun(x, w, torch.sqrt(2.0 * al * prm.temp * prm.dtau), al, c, True)
            else:
                x = group.rk4(x, step, al, c)
            step += 1
        near = group.ref.core_set(x[0].detach())[3]
        path.append(group.ref.centroid(x[0], near))
    rc = torch.stack(path)
    loss = ((rc - target_path(case, seed, rc).double()) ** 2).sum()
    gm, gt = torch.autograd.grad(loss, [m, theta])
    return dict(path=rc.detach(), m=gm.reshape(-1), theta=theta.detach() - DESCENT * gt)


def exact(case, seed):
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    if case["kind"] == "spectrum":
        x = signals(case, seed)
        n = case["length"]
        if case["mean"]:
            x = x - x.mean(dim=1, keepdim=True)
        if case["window"] == "hann":
            x = x * torch.sin(math.pi * torch.arange(n, dtype=torch.float64) / n) ** 2
        return torch.fft.rfft(x, dim=1).abs() ** 2 / n
    geo, states, kind = shapes(case), start_states(case, seed), case["kind"]
    groups = [Group(case, g, [k for k in range(len(geo)) if geo[k] == g], states, device)
              for g in dict.fromkeys(geo)]
    if kind == "adjoint":
        return exact_adjoint(case, seed, groups[0], states, device)

    def pack(values):                # [(group, [n, ...])] back to the order of the disks
        out = [None] * len(geo)
        for g, v in zip(groups, values):
            for k, row in zip(g.at, v):
                out[k] = row
        return out

    def flat(values):
        return torch.cat([v.reshape(-1) for v in pack(values)])
    if kind == "field":
        return flat([g.ref.demag(g.m) for g in groups])
    for g in groups:
        g.m = g.m * g.ref.mask
    if kind == "rhs":
        return flat([g.rhs(g.m, 0.0) for g in groups])
    if kind == "observe":
        cores = []
        for g in groups:
            rows = []
            for v in g.m:
                xv, yv, n, near = g.ref.core_set(v)
                x, y = g.ref.centroid(v, near).tolist()
                rows.append(torch.tensor([x, y, xv * A_NM, yv * A_NM, float(n)], dtype=torch.float64))
            cores.append(torch.stack(rows))
        return dict(core=torch.stack(pack(cores)),
                    energy=torch.stack(pack([g.ref.energy(g.m, g.h(0.0), C_PY) for g in groups])),
                    mean=torch.stack(pack([g.ref.mean(g.m) for g in groups])))
    if kind == "relax":
        X = targets(case)
        got = [relaxed(g, [X[k] for k in g.at], case["sweeps"]) for g in groups]
        return dict(m=flat([v[0] for v in got]), record=torch.stack(pack([v[1] for v in got])))
    series = []
    for n in range(case["steps"]):
        if kind.endswith("series") and n % case["every"] == 0:
            series.append(torch.stack(pack([g.sample(n) for g in groups])))
        for g in groups:
            g.advance(n, seed)
    m = flat([g.m for g in groups])
    return dict(series=torch.stack(series), m=m) if series else m
