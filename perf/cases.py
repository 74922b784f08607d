"""The work a program has this library do, as cases that can be timed.

A case is a dict of plain numbers and texts; `prepare` builds what a program holds before the call (a
resident simulation, a scan server, a bunch loaded into the window), `run` makes one pass through the
public entry points, and `exact` computes what the pass leaves behind in 64-bit floating point with plain
torch, from the equations and not from this library's code.

kinds
  step   `steps` whole steps of one resident simulation: the loop every run spends its time in
  scan   a burst of scan jobs through the serving front end
  beam   the diagnostics of a run that is going on: beam parameters, charge spectrum, conserved sums
  dump   one output of a run: grids and particles on the host
  bunch  the self-consistent fields of an injected bunch, solved before a run starts
"""
import math
import random

import numpy as np
import torch

import paper_1912_04674_amd as E
from paper_1912_04674_amd.serve import GpuBackend, ScanServer

# ---------------------------------------------------------------- cases --
_DEFAULTS = dict(kind="step", nx=512, nr=64, modes=1, ppc_x=2, ppc_r=2, ppc_t=2, order=1, filter=0,
                 precision="fp32", sort_every=0, profile="uniform", window=True, dx=0.8, dr=1.5, dt=0.6,
                 n0=0.002, a0=2.0, w0=50.0, tau=30.0, warm=24, steps=24, jobs=0, bunch=0)


def _case(**kw):
    c = dict(_DEFAULTS)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest run (the parity set-up's grid, 33 thousand particles), advanced one step per call as an
        # interactive or coupled program does: a handful of launches each
        _case(name="step1_256x32", nx=256, nr=32, ppc_t=1, a0=1.0, w0=20.0, steps=1),
        # a burst of eight scan jobs (the smallest serving grid), served together to the end
        _case(name="scan_8x_512x64", kind="scan", a0=1.5, n0=0.0025, w0=60.0, warm=0, steps=50, jobs=8),
        # a lone scan job of the middle serving grid
        _case(name="step_1024x128", nx=1024, nr=128, a0=1.5, n0=0.0025, w0=80.0),
        # the laser-wakefield benchmark: modes 0 and 1, 8.4 M particles, moving window with a density ramp
        _case(name="lwfa_2048x256", nx=2048, nr=256, modes=2, ppc_t=4, profile="ramp", n0=0.0017, w0=100.0,
              tau=60.0),
        # the same in double precision (the reference path of a precision study)
        _case(name="lwfa_2048x256_fp64", nx=2048, nr=256, modes=2, ppc_t=4, profile="ramp", n0=0.0017, w0=100.0,
              tau=60.0, precision="fp64"),
        # the nonlinear benchmark's window and resolution: quadratic shapes, seven filter passes, six particles
        # per cell, coarse in r
        _case(name="nonlinear_1088x224", nx=1088, nr=224, modes=2, ppc_x=1, ppc_r=2, ppc_t=3, order=2, filter=7,
              dr=3.5, dt=0.72, n0=0.0015, a0=2.96, w0=300.0, tau=60.0, warm=16, steps=16),
        # a static box of odd size, 15 particles per cell in three unequal directions, density noise
        _case(name="ragged_1003x149", nx=1003, nr=149, modes=2, ppc_x=1, ppc_r=3, ppc_t=5, profile="perturb",
              window=False, w0=60.0, tau=40.0),
        # the bandwidth workload: 33.5 M particles, sorted every step
        _case(name="bandwidth_4096x512", nx=4096, nr=512, modes=2, ppc_t=4, profile="perturb", window=False,
              sort_every=1, n0=0.001, a0=2.5, w0=150.0, tau=80.0, warm=8, steps=8),
        # the largest run: 151 M particles in a moving window, a density bump entering
        _case(name="scale_8192x768", nx=8192, nr=768, modes=2, ppc_t=6, profile="bump", n0=0.0015, a0=3.0,
              w0=200.0, tau=90.0, warm=4),
        # diagnostics of the wakefield run between steps
        _case(name="beam_2048x256", kind="beam", nx=2048, nr=256, modes=2, ppc_t=4, profile="ramp", n0=0.0017,
              w0=100.0, tau=60.0),
        # one output of a scan job: its mode-0 grids and its million particles
        _case(name="dump_1024x128", kind="dump", nx=1024, nr=128, a0=1.5, n0=0.0025, w0=80.0),
        # an externally injected bunch of 200 thousand particles on the wakefield grid
        _case(name="bunch_2048x256", kind="bunch", nx=2048, nr=256, ppc_x=1, ppc_r=1, ppc_t=1, profile="none",
              a0=0.0, warm=0, steps=0, bunch=200000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: grids from 96 x 24 to 4096 x 640 cells, up to 40 M particles, both shape
    orders, both precisions, one or two modes, every sort period, filter and density profile."""
    while True:
        kind = rng.choices(["step", "scan", "beam", "dump", "bunch"], [14, 2, 1, 1, 1])[0]
        hi_x, hi_r = {"step": (4096, 640), "scan": (1024, 128), "beam": (2048, 300), "dump": (1100, 160),
                      "bunch": (2048, 300)}[kind]
        nx, nr = _log_int(rng, 96, hi_x), _log_int(rng, 24, hi_r)
        c = _case(kind=kind, nx=nx, nr=nr, ppc_x=rng.choice([1, 2]), ppc_r=rng.choice([1, 2, 3]),
                  ppc_t=rng.choice([1, 2, 3, 4, 6]), modes=rng.choice([1, 2]))
        c["tau"] = round(rng.uniform(0.03, 0.06) * nx * c["dx"], 2)
        c["w0"] = round(rng.uniform(0.2, 0.35) * nr * c["dr"], 2)
        c["a0"] = round(rng.uniform(0.5, 3.0), 3)
        c["n0"] = round(rng.uniform(0.001, 0.004), 5)
        c["window"] = rng.random() < 0.7
        c["profile"] = rng.choice(["uniform", "ramp", "perturb", "bump"])
        if kind == "scan":
            c.update(modes=1, ppc_x=2, ppc_r=2, ppc_t=2, profile="uniform", window=True, warm=0,
                     steps=rng.choice([25, 50, 60]), jobs=rng.randint(1, 8))
        elif kind == "bunch":
            c.update(modes=1, ppc_x=1, ppc_r=1, ppc_t=1, profile="none", a0=0.0, window=True, warm=0, steps=0,
                     bunch=_log_int(rng, 5000, 200000), order=rng.choice([1, 2]))
        else:
            c["precision"] = "fp64" if rng.random() < 0.2 else "fp32"
            if rng.random() < 0.3:
                c.update(order=2, warm=16, steps=16)
            if kind == "step":
                most = 2 if c["order"] == 2 else 3
                c["sort_every"] = rng.choice([0, 0, 0, rng.randint(1, most)])
                if rng.random() < 0.25 and nx > 40 and nr > 18:
                    c["filter"] = rng.randint(1, 7)
                if _particles(c) < 200000 and rng.random() < 0.3:
                    c["steps"] = 1
        if _particles(c) <= 40e6 and (kind != "dump" or _particles(c) <= 1.5e6):
            return c


def _particles(c):
    return c["nx"] * c["nr"] * c["ppc_x"] * c["ppc_r"] * c["ppc_t"] if c["profile"] != "none" else c["bunch"]


def _config(c, seed, job=0):
    """The parameter dictionary of a case: the laser and plasma vary with the seed within ten percent."""
    rng = random.Random(seed * 1009 + job)
    lx = c["nx"] * c["dx"]
    return dict(nx=c["nx"], nr=c["nr"], n_modes=c["modes"], ppc=(c["ppc_x"], c["ppc_r"], c["ppc_t"]),
                profile=c["profile"], moving_window=int(c["window"]), seed=191204674 + rng.randrange(1 << 30),
                dx=c["dx"], dr=c["dr"], dt=c["dt"], a0=c["a0"] * rng.uniform(0.9, 1.1), w0=c["w0"],
                tau=c["tau"], x_c=lx - 3 * c["tau"] if c["window"] else lx / 2,
                x_f=lx - 3 * c["tau"] if c["window"] else lx / 2, n0=c["n0"] * rng.uniform(0.9, 1.1),
                ramp_len=min(200.0, lx / 4), perturb=0.01, bump_x=lx + 40.0, bump_w=min(100.0, lx / 8),
                filter_passes=c["filter"], shape_order=c["order"], sort_every=c["sort_every"])


def _dipole(cfg, seed):
    """A weak transverse field E_y of mode 1 around the pulse (which is never quite axisymmetric): the E_r and
    E_theta amplitudes."""
    e0 = 5e-4 * random.Random(seed + 17).uniform(0.5, 1.5)
    i, j = np.arange(cfg["nx"] + 1)[:, None], np.arange(cfg["nr"] + 1)[None, :]
    xi = (i * cfg["dx"] - cfg["x_c"]) / cfg["tau"]
    f = e0 * np.exp(-xi * xi) * np.sin(math.pi * i / cfg["nx"])
    return (f * (1 - np.minimum(1, (j + 0.5) / cfg["nr"]) ** 2) ** 2 + 0j,
            -1j * f * (1 - (j / cfg["nr"]) ** 2) ** 2)


BETA = 0.99  # velocity of the injected bunch


def _bunch(c, seed):
    """A Gaussian bunch in the middle of the window (lab-frame Cartesian arrays, ids 0 .. n-1)."""
    rng = np.random.default_rng(seed)
    n, lx, rmax = c["bunch"], c["nx"] * c["dx"], c["nr"] * c["dr"]
    sx, sr = min(8.0, lx / 20), min(3.0, rmax / 10)
    x = lx * rng.uniform(0.4, 0.6) + sx * np.clip(rng.normal(size=n), -4, 4)
    y, z = (sr * np.clip(rng.normal(size=n), -4, 4) for _ in range(2))
    zero = np.zeros(n)
    return dict(x=x, y=y, z=z, px=np.full(n, BETA / math.sqrt(1 - BETA * BETA)), py=zero, pz=zero,
                w=np.full(n, 20.0 / n), id=np.arange(n, dtype=np.uint32))


# -------------------------------------------------------- what is timed --
_EM0 = ("ex", "er", "bt", "bt_bar")
_EM1 = ("ex1", "er1", "et1", "bx1", "br1", "bt1", "bx1_bar", "br1_bar", "bt1_bar")
_J0, _J1 = ("jx", "jr"), ("jx1", "jr1", "jt1")
_PHASE = ("x", "y", "z"), ("px", "py", "pz")
# reading 10^8 particles back takes minutes; larger runs are compared by their grids (chi and J hold every particle)
READ_PARTICLES = 10_000_000


class Readout(dict):
    """What a pass left in the resident simulation, read through the library's IO when it is looked at (a
    program dumps now and then, not after every pass).  E and B of all modes are one array and so are the
    components of J and of the momentum: each is one quantity in one unit."""

    def __init__(self, sim, names, modes):
        super().__init__((n, None) for n in names)
        self._sim, self._modes = sim, modes

    def _grids(self, names0, names1):
        g = [self._sim.get_field(n) for n in names0]
        for n in names1 if self._modes == 2 else ():
            v = self._sim.get_field(n)
            g += [v.real, v.imag]
        return np.stack(g)

    def __getitem__(self, name):
        if name == "em":
            return self._grids(_EM0, _EM1)
        if name == "em0":
            return self._grids(_EM0, ())
        if name == "j":
            return self._grids(_J0, _J1)
        if name == "particles":
            p = self._sim.get_particles()
            return {"id": p["id"], "w": p["w"], "r": np.stack([p[k] for k in _PHASE[0]]),
                    "p": np.stack([p[k] for k in _PHASE[1]])}
        return self._sim.get_field(name)

    def get(self, name, default=None):
        return self[name] if name in self else default

    def values(self):
        return [self[n] for n in self]

    def items(self):
        return [(n, self[n]) for n in self]


def _names(c):
    return ("env", "env_prev", "chi", "em", "j") + (("particles",) if _particles(c) <= READ_PARTICLES else ())


def prepare(case, seed):
    c = case
    prec = E.FP64 if c["precision"] == "fp64" else E.FP32_BULK
    if c["kind"] == "scan":
        cfgs = [_config(c, seed, k) for k in range(c["jobs"])]
        backend = GpuBackend(sum(E.footprint(q) for q in cfgs) + (1 << 20))
        return {"case": c, "server": ScanServer(backend), "cfgs": cfgs}
    cfg = _config(c, seed)
    sim = E.Sim(cfg, prec)
    if c["kind"] == "bunch":
        sim.set_particles(_bunch(c, seed))
        return {"case": c, "sim": sim}
    if c["modes"] == 2:
        er1, et1 = _dipole(cfg, seed)
        sim.set_field("er1", er1)
        sim.set_field("et1", et1)
    sim.step(c["warm"])
    return {"case": c, "sim": sim}


def run(state):
    c = state["case"]
    if c["kind"] == "scan":
        jobs = state["server"].run_trace(state["cfgs"], [0.0] * c["jobs"], steps=c["steps"])
        for j in jobs:
            if j.result is None:
                raise RuntimeError(j.error)
        # (L_x is zero but for rounding; the beam parameters other than the charge hinge on which bin of the
        # spectrum is the fullest)
        sums = [_sums(j.result["diag"]) for j in jobs]
        return {"ex_axis": [j.result["ex_axis"] for j in jobs],
                "sums": {k: np.array([d[k] for d in sums]) for k in sums[0]},
                "charge_spectrum": np.array([j.result["beam"]["charge_spectrum"] for j in jobs])}
    sim = state["sim"]
    if c["kind"] == "step":
        sim.step(c["steps"])
        return Readout(sim, _names(c), c["modes"])
    if c["kind"] == "beam":
        params, hist = sim.beam(1e-3, 20.0, 512, with_hist=True)
        return {"hist": hist, "charge_spectrum": params["charge_spectrum"], "sums": _sums(sim.diagnostics())}
    if c["kind"] == "dump":
        out = {n: sim.get_field(n) for n in ("env", "chi")}
        out["em"] = np.stack([sim.get_field(n) for n in _EM0])
        out["j"] = np.stack([sim.get_field(n) for n in _J0])
        p = sim.get_particles()
        out["particles"] = {"id": p["id"], "w": p["w"], "r": np.stack([p[k] for k in _PHASE[0]]),
                            "p": np.stack([p[k] for k in _PHASE[1]])}
        return out
    sim.bunch_fields(0, c["bunch"], BETA)
    return Readout(sim, ("em0",), 1)


def _sums(d):
    return {k: float(d[k]) for k in ("count", "charge", "chi_v", "kin", "uem", "env2_v", "px")}


def work(case):
    """Bytes of one pass with every array read and written once per kernel stage that needs it, and its
    floating-point operations (counted from the equations, divisions and roots as one)."""
    c = case
    b = 8 if c["precision"] == "fp64" else 4
    n, cells, m2 = _particles(c), c["nx"] * c["nr"], c["modes"] == 2
    # a step reads the particle record twice (the envelope update lies between the momentum and the position
    # pass) and writes the momentum once and the position once; grids: gathers, deposits, Maxwell, envelope
    per_particle = 2 * (7 * b + 4) + 3 * b + 3 * b + 4
    per_cell = (6 + 6 + 9 + 7 + ((12 + 6 + 36) if m2 else 0)) * b
    # shape functions, gathers, push, deposits
    k = c["order"] + 1
    flops_p = 230 + k * k * (2 * (6 + (12 if m2 else 0)) + 2 * (1 + 4 + (6 if m2 else 0)))
    flops_c = 60 + (90 if m2 else 0)
    if c["kind"] == "scan":
        return {"bytes": c["jobs"] * c["steps"] * (n * per_particle + cells * per_cell),
                "flops": c["jobs"] * c["steps"] * (n * flops_p + cells * flops_c)}
    if c["kind"] == "step":
        return {"bytes": c["steps"] * (n * per_particle + cells * per_cell),
                "flops": c["steps"] * (n * flops_p + cells * flops_c)}
    if c["kind"] == "beam":  # the records once; energy, bin and moments
        return {"bytes": n * (6 * b + 4) + cells * (7 + (12 if m2 else 0)) * b, "flops": n * 60 + cells * 30}
    if c["kind"] == "dump":  # the records and grids read, written in FP64
        return {"bytes": n * (7 * b + 8 + 60) + cells * 9 * (b + 8), "flops": n * 10 + cells * 9}
    # charge of the bunch, a direct solve's reads and writes of one potential, the fields added
    return {"bytes": c["bunch"] * 20 + cells * (3 * 8 + 8 * 4), "flops": c["bunch"] * 30 + cells * (10 * math.log2(c["nx"]) + 20)}


def tolerance(case):
    """About four times the largest difference from `exact` of any output (2-norm): J, which follows the
    FP32 positions, is the least exact output of a step (FP32: 7e-5 on the bandwidth workload, 2e-5 elsewhere; FP64: 9e-12)."""
    if case["precision"] == "fp64":
        return {"rel": 4e-11}
    return {"rel": {"step": 3e-4, "scan": 3e-5, "beam": 3e-5, "dump": 3e-5, "bunch": 2e-7}[case["kind"]]}


# ------------------------------------------------ the same in 64 bits --
def exact(case, seed):
    c = case
    if c["kind"] == "bunch":
        return {"em0": _bunch_reference(c, seed)}
    if c["kind"] == "scan":
        if c["jobs"] * c["steps"] * (1e6 + _particles(c)) > 2e9:
            return None
        axis, sums, charge = [], [], []
        for k in range(c["jobs"]):
            s = _Reference(_config(c, seed, k))
            s.step(c["steps"])
            axis.append(s.np("ex")[:, 0])
            sums.append(s.sums())
            charge.append(s.spectrum(1e-3, 20.0, 256)[1])
        return {"ex_axis": axis, "sums": {k: np.array([d[k] for d in sums]) for k in sums[0]},
                "charge_spectrum": np.array(charge)}
    n = c["warm"] + (c["steps"] if c["kind"] == "step" else 0)
    if n * _particles(c) * (3 if c["order"] == 2 else 1) > 6e8:
        return None
    cfg = _config(c, seed)
    s = _Reference(cfg)
    if c["modes"] == 2:
        s.er1[:], s.et1[:] = (torch.from_numpy(v).to(s.dev) for v in _dipole(cfg, seed))
        s.er1[:, -1] = 0
    s.step(n)
    if c["kind"] == "beam":
        hist, charge = s.spectrum(1e-3, 20.0, 512)
        return {"hist": hist, "charge_spectrum": charge, "sums": s.sums()}
    names = _names(c) if c["kind"] == "step" else ("env", "chi", "em", "j", "particles")
    out = {}
    for name in names:
        if name in ("em", "j"):
            n0, n1 = (_EM0, _EM1) if name == "em" else (_J0, _J1)
            g = [s.np(k) for k in n0]
            for k in n1 if c["modes"] == 2 else ():
                g += [s.np(k).real, s.np(k).imag]
            out[name] = np.stack(g)
        elif name == "particles":
            o = torch.argsort(s.id)
            out[name] = {"id": None, "w": s.w[o].cpu().numpy(), "r": s.r[:, o].cpu().numpy(),
                         "p": s.p[:, o].cpu().numpy()}
        else:
            out[name] = s.np(name)
    return out


def _uniform(seed, stream, col, j):
    """SplitMix64 of a counter (Steele, Lea, Flood 2014): a deviate in [0, 1) for each cell (col, j)."""
    key = (np.uint64(stream) << np.uint64(56)) ^ (col.astype(np.uint64) << np.uint64(20)) ^ j.astype(np.uint64)
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (key + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return (z >> np.uint64(11)).astype(np.float64) * 2.0 ** -53


_PAD = 4  # rows and columns around a grid in gathers and deposits


class _Reference:
    """The envelope PIC loop in FP64 on window-relative (nx + 1) x (nr + 1) grids, written for clarity."""
    CHUNK = 1 << 22

    def __init__(self, cfg):
        self.cfg, self.dev = cfg, "cuda" if torch.cuda.is_available() else "cpu"
        self.nx, self.nr, self.m1 = cfg["nx"], cfg["nr"], cfg["n_modes"] == 2
        self.dx, self.dr, self.dt = cfg["dx"], cfg["dr"], cfg["dt"]
        self.order = cfg["shape_order"]
        self.n = self.shift = 0
        shape = (self.nx + 1, self.nr + 1)
        for k in _EM0 + _J0 + ("chi",):
            setattr(self, k, torch.zeros(shape, dtype=torch.float64, device=self.dev))
        for k in _EM1 + _J1:
            setattr(self, k, torch.zeros(shape, dtype=torch.complex128, device=self.dev))
        self.j = torch.arange(self.nr + 1, dtype=torch.float64, device=self.dev)
        self.vn = 2 * math.pi * self.j * self.dr ** 2 * self.dx
        self.vn[0] = math.pi * self.dr ** 2 * self.dx / 4
        self.vh = 2 * math.pi * (self.j + 0.5) * self.dr ** 2 * self.dx
        self.env, self.env_prev = self._pulse(0.0), self._pulse(-self.dt)
        self.r = torch.zeros((3, 0), dtype=torch.float64, device=self.dev)
        self.p, self.w = self.r.clone(), self.r[0].clone()
        self.id = torch.zeros(0, dtype=torch.int64, device=self.dev)
        self._load(0, self.nx)

    def np(self, name):
        return getattr(self, name).cpu().numpy()

    # ---- initial state
    def _pulse(self, t):
        g = self.cfg
        x = torch.arange(self.nx + 1, dtype=torch.float64, device=self.dev)[:, None] * self.dx
        r = self.j[None, :] * self.dr
        q = 1 + 1j * (x - g["x_f"]) / (0.5 * g["w0"] ** 2)
        sig = g["tau"] / (2 * math.sqrt(math.log(2)))
        a = g["a0"] * torch.exp(-r * r / (g["w0"] ** 2 * q)) / q * torch.exp(-((x - g["x_c"] - t) / sig) ** 2)
        a[0], a[-1], a[:, -1] = 0, 0, 0
        return a

    def _load(self, c0, c1):
        """Plasma of the lab columns c0 .. c1 - 1: regular in x and r, one random angle per cell."""
        g = self.cfg
        if g["profile"] == "none":
            return
        px, pr, pt = g["ppc"]
        ppc = px * pr * pt
        col, j = (v.reshape(-1) for v in np.meshgrid(np.arange(c0, c1), np.arange(self.nr), indexing="ij"))
        th0 = 2 * math.pi * _uniform(g["seed"], 1, col, j)
        k = np.arange(ppc)
        x = (col[:, None] + (k // (pr * pt) + 0.5) / px) * self.dx
        r = (j[:, None] + ((k // pt) % pr + 0.5) / pr) * self.dr
        th = th0[:, None] + 2 * math.pi * (k % pt) / pt
        dens = {"uniform": lambda: g["n0"] + 0 * x,
                "ramp": lambda: g["n0"] * np.clip(x / g["ramp_len"], 0, 1),
                "perturb": lambda: g["n0"] * (1 + g["perturb"] * (2 * _uniform(g["seed"], 2, col, j) - 1))[:, None] + 0 * x,
                "bump": lambda: g["n0"] * (1 + np.exp(-((x - g["bump_x"]) / g["bump_w"]) ** 2))}[g["profile"]]()
        w = dens * 2 * math.pi * r * (self.dr / pr) * (self.dx / px) / pt
        ids = col[:, None].astype(np.int64) * self.nr * ppc + j[:, None] * ppc + k
        new = [np.broadcast_to(v, w.shape).reshape(-1) for v in (x, r * np.cos(th), r * np.sin(th), w, ids)]
        live = new[3] > 0
        new = [torch.from_numpy(np.ascontiguousarray(v[live])).to(self.dev) for v in new]
        self.r = torch.cat([self.r, torch.stack(new[:3])], 1)
        self.p = torch.cat([self.p, torch.zeros((3, len(new[3])), dtype=torch.float64, device=self.dev)], 1)
        self.w, self.id = torch.cat([self.w, new[3]]), torch.cat([self.id, new[4]])

    # ---- shapes, gathers, deposits
    def _shape(self, u):
        """First node and the weights of the nodes from it (linear or quadratic B-spline)."""
        if self.order == 2:
            m = torch.floor(u + 0.5)
            d = u - m
            return m.long() - 1, [0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2]
        m = torch.floor(u)
        return m.long(), [1 - (u - m), u - m]

    def _pad(self, f, par, half_x, half_r):
        """f with _PAD nodes around it: zero outside, mirrored with its parity below the axis."""
        f = f[: self.nx + (0 if half_x else 1), : self.nr + (0 if half_r else 1)]
        low = f[:, :_PAD].flip(1) if half_r else f[:, 1:_PAD + 1].flip(1)
        out = torch.zeros((self.nx + 1 + 2 * _PAD, self.nr + 1 + 2 * _PAD), dtype=f.dtype, device=self.dev)
        out[_PAD:_PAD + f.shape[0], _PAD:_PAD + f.shape[1]] = f
        out[_PAD:_PAD + f.shape[0], :_PAD] = par * low
        return out

    def _pack(self, fields, half_x, half_r):
        cols = []
        for f, par in fields:
            q = self._pad(f, par, half_x, half_r).reshape(-1)
            cols += [q.real, q.imag] if q.is_complex() else [q]
        return torch.stack(cols, 1)

    def _index(self, i, j):
        return (i + _PAD).clamp(0, self.nx + 2 * _PAD) * (self.nr + 1 + 2 * _PAD) + (j + _PAD).clamp(0, self.nr + 2 * _PAD)

    def _gather(self, pack, sx, sr):
        out = None
        for a, wa in enumerate(sx[1]):
            for b, wb in enumerate(sr[1]):
                v = pack[self._index(sx[0] + a, sr[0] + b)] * (wa * wb)[:, None]
                out = v if out is None else out + v
        return out

    def _acc(self, k=1):
        return torch.zeros(((self.nx + 1 + 2 * _PAD) * (self.nr + 1 + 2 * _PAD), k), dtype=torch.float64, device=self.dev)

    def _fold(self, acc, sign, half_x, half_r, vol):
        """The deposit on the grid: rows below the axis onto their mirrors, nodes outside dropped, per volume."""
        a = acc.reshape(self.nx + 1 + 2 * _PAD, self.nr + 1 + 2 * _PAD, -1)
        a = a[..., 0] if a.shape[2] == 1 else torch.complex(a[..., 0].contiguous(), a[..., 1].contiguous())
        a = a[_PAD:-_PAD].clone()
        if half_r:
            a[:, _PAD:2 * _PAD] += sign * a[:, :_PAD].flip(1)
        else:
            a[:, _PAD + 1:2 * _PAD + 1] += sign * a[:, :_PAD].flip(1)
        a = a[:, _PAD:-_PAD] / vol
        if half_x:
            a[-1] = 0
        if half_r:
            a[:, -1] = 0
        return a

    # ---- one step
    def step(self, n):
        for _ in range(n):
            self._momentum()
            self._envelope()
            self._position()
            self._filter()
            self._maxwell()
            self._window()
            self.n += 1

    def _chunks(self):
        for lo in range(0, self.w.numel(), self.CHUNK):
            yield slice(lo, min(lo + self.CHUNK, self.w.numel()))

    def _momentum(self):
        phi = 0.5 * self.env.abs() ** 2
        gx, gr = torch.zeros_like(phi), torch.zeros_like(phi)
        gx[1:-1] = (phi[2:] - phi[:-2]) / (2 * self.dx)
        gx[0], gx[-1] = phi[1] / (2 * self.dx), -phi[-2] / (2 * self.dx)
        gr[:, 1:-1] = (phi[:, 2:] - phi[:, :-2]) / (2 * self.dr)
        gr[:, -1] = -phi[:, -2] / (2 * self.dr)
        m1 = self.m1
        dp = self._pack([(self.ex, 1)] + ([(self.ex1, -1), (self.br1_bar, 1)] if m1 else []), True, False)
        pd = self._pack([(self.er, -1)] + ([(self.er1, 1), (self.bx1_bar, -1)] if m1 else []), False, True)
        dd = self._pack([(self.bt_bar, -1)] + ([(self.bt1_bar, 1)] if m1 else []), True, True)
        pp = self._pack([(phi, 1), (gx, 1), (gr, -1)] + ([(self.et1, 1)] if m1 else []), False, False)
        acc = self._acc()
        for k in self._chunks():
            x, y, z = self.r[:, k]
            rad = torch.hypot(y, z)
            c = torch.where(rad > 0, y / rad, torch.ones_like(rad))
            s = torch.where(rad > 0, z / rad, torch.zeros_like(rad))
            ux, ur = x / self.dx - self.shift, rad / self.dr
            P, D, Pr, Dr = self._shape(ux), self._shape(ux - 0.5), self._shape(ur), self._shape(ur - 0.5)
            a, b, d, e = (self._gather(*v) for v in ((dp, D, Pr), (pd, P, Dr), (dd, D, Dr), (pp, P, Pr)))
            ex, er, bt, ph = a[:, 0], b[:, 0], d[:, 0], e[:, 0]
            et = bx = br = torch.zeros_like(ex)
            if m1:
                ex, br = ex + a[:, 1] * c + a[:, 2] * s, a[:, 3] * c + a[:, 4] * s
                er, bx = er + b[:, 1] * c + b[:, 2] * s, b[:, 3] * c + b[:, 4] * s
                bt, et = bt + d[:, 1] * c + d[:, 2] * s, e[:, 3] * c + e[:, 4] * s
            Ev = torch.stack([ex, er * c - et * s, er * s + et * c])
            Bv = torch.stack([bx, br * c - bt * s, br * s + bt * c])
            G = torch.stack([e[:, 1], e[:, 2] * c, e[:, 2] * s])
            p = self.p[:, k]
            F = -Ev - G / (2 * torch.sqrt(1 + (p * p).sum(0) + ph))
            pm = p + 0.5 * self.dt * F
            gb = torch.sqrt(1 + (pm * pm).sum(0) + ph)
            t = -0.5 * self.dt * Bv / gb
            pl = pm + torch.linalg.cross(pm + torch.linalg.cross(pm, t, dim=0), 2 * t / (1 + (t * t).sum(0)), dim=0)
            self.p[:, k] = pl + 0.5 * self.dt * F
            wg = self.w[k] / gb
            for i, wa in enumerate(P[1]):
                for j, wb in enumerate(Pr[1]):
                    acc.index_add_(0, self._index(P[0] + i, Pr[0] + j), (wg * wa * wb)[:, None])
        self.chi = self._fold(acc, 1, False, False, self.vn)

    def _envelope(self):
        A, dt = self.env, self.dt
        a = A[1:-1, :-1]
        lap = (A[2:, :-1] - 2 * a + A[:-2, :-1]) / self.dx ** 2
        up = A[1:-1, 1:]
        dn = torch.cat([A[1:-1, :1], A[1:-1, :-2]], 1)
        rad = (up - 2 * a + dn) / self.dr ** 2 + (up - dn) / (2 * self.j[:-1].clamp(min=1) * self.dr ** 2)
        rad[:, 0] = 4 * (A[1:-1, 1] - A[1:-1, 0]) / self.dr ** 2
        rhs = lap + rad - self.chi[1:-1, :-1] * a + 1j * (A[2:, :-1] - A[:-2, :-1]) / self.dx
        new = torch.zeros_like(A)
        new[1:-1, :-1] = (1 + 1j * dt) / (1 + dt * dt) * (2 * a - (1 + 1j * dt) * self.env_prev[1:-1, :-1] + dt * dt * rhs)
        self.env_prev, self.env = A, new

    def _position(self):
        phh = self._pack([(0.25 * (self.env.abs() ** 2 + self.env_prev.abs() ** 2), 1)], False, False)
        jx, jr = self._acc(), self._acc()
        j1 = [self._acc(2) for _ in range(3)] if self.m1 else None
        rmax, keep = self.nr * self.dr, torch.ones_like(self.w, dtype=torch.bool)
        for k in self._chunks():
            x, y, z = self.r[:, k].clone()
            rad = torch.hypot(y, z)
            ux, ur = x / self.dx - self.shift, rad / self.dr
            ph = self._gather(phh, self._shape(ux), self._shape(ur))[:, 0]
            p = self.p[:, k]
            v = p / torch.sqrt(1 + (p * p).sum(0) + ph)
            xn, yn, zn = x + self.dt * v[0], y + self.dt * v[1], z + self.dt * v[2]
            rn = torch.hypot(yn, zn)
            out = rn >= rmax
            if bool(out.any()):  # specular reflection at r_max
                safe = torch.where(out, rn, torch.ones_like(rn))
                cr, sr = yn / safe, zn / safe
                f = torch.where(out, (2 * rmax - rn) / safe, torch.ones_like(rn))
                yn, zn, rn = yn * f, zn * f, torch.where(out, 2 * rmax - rn, rn)
                prad = torch.where(out, p[1] * cr + p[2] * sr, torch.zeros_like(rn))
                self.p[1, k] = p[1] - 2 * prad * cr
                self.p[2, k] = p[2] - 2 * prad * sr
            uxn = xn / self.dx - self.shift
            ok = (uxn >= 0) & (uxn < self.nx)
            keep[k] = ok
            w = torch.where(ok, self.w[k], torch.zeros_like(x))
            uxn = torch.where(ok, uxn, ux)
            i0, S0x, S1x = self._union(ux, uxn)
            j0, S0r, S1r = self._union(ur, rn / self.dr)
            n = len(S0x)
            for b in range(n):
                c = torch.zeros_like(x)
                for a in range(n - 1):
                    c = c + (S1x[a] - S0x[a])
                    jx.index_add_(0, self._index(i0 + a, j0 + b), (w * c * (S0r[b] + S1r[b]) * 0.5)[:, None])
            for a in range(n):
                c = torch.zeros_like(x)
                for b in range(n - 1):
                    c = c + (S1r[b] - S0r[b])
                    jr.index_add_(0, self._index(i0 + a, j0 + b), (w * c * (S0x[a] + S1x[a]) * 0.5)[:, None])
            if self.m1:
                xm, ym, zm = 0.5 * (x + xn), 0.5 * (y + yn), 0.5 * (z + zn)
                rm = torch.hypot(ym, zm)
                c = torch.where(rm > 0, ym / rm, torch.ones_like(rm))
                s = torch.where(rm > 0, zm / rm, torch.zeros_like(rm))
                um, vm = torch.where(ok, xm / self.dx - self.shift, ux), rm / self.dr
                P, D, Pr, Dr = self._shape(um), self._shape(um - 0.5), self._shape(vm), self._shape(vm - 0.5)
                q = -2 * w
                for acc, X, Rr, vel in ((j1[0], D, Pr, v[0]), (j1[1], P, Dr, v[1] * c + v[2] * s), (j1[2], P, Pr, v[2] * c - v[1] * s)):
                    cs = torch.stack([q * vel * c, q * vel * s], 1)
                    for a, wa in enumerate(X[1]):
                        for b, wb in enumerate(Rr[1]):
                            acc.index_add_(0, self._index(X[0] + a, Rr[0] + b), cs * (wa * wb)[:, None])
            self.r[:, k] = torch.stack([xn, yn, zn])
        # (an electron: the current is minus the flux of its charge, hence the sign of the flux itself)
        ax = self.vn / self.dx
        ar = 2 * math.pi * (self.j + 0.5) * self.dr * self.dx
        self.jx = self._fold(jx, 1, True, False, ax * self.dt)
        self.jr = self._fold(jr, -1, False, True, ar * self.dt)
        if self.m1:
            self.jx1 = self._fold(j1[0], -1, True, False, self.vn)
            self.jr1 = self._fold(j1[1], 1, False, True, self.vh)
            self.jt1 = self._fold(j1[2], 1, False, False, self.vn)
        self._drop(keep)

    def _union(self, u0, u1):
        """The stencils of two positions less than a cell apart, on the union of their nodes."""
        (m0, w0), (m1, w1) = self._shape(u0), self._shape(u1)
        m = torch.minimum(m0, m1)
        zero = torch.zeros_like(u0)

        def place(first, w):
            late = first > m
            return [torch.where(late, w[k - 1] if k else zero, w[k] if k < len(w) else zero) for k in range(len(w) + 1)]
        return m, place(m0, w0), place(m1, w1)

    def _drop(self, keep):
        if not bool(keep.all()):
            self.r, self.p, self.w, self.id = self.r[:, keep], self.p[:, keep], self.w[keep], self.id[keep]

    def _filter(self):
        if self.cfg["filter_passes"] and self.m1:
            self.jx1[:, 0] = 0
        for _ in range(self.cfg["filter_passes"]):
            for name, hx, hr, par in [("jx", 1, 0, 1), ("jr", 0, 1, -1)] + (
                    [("jx1", 1, 0, -1), ("jr1", 0, 1, 1), ("jt1", 0, 0, 1)] if self.m1 else []):
                full = getattr(self, name)
                f = full[: self.nx + 1 - hx, : self.nr + 1 - hr]
                z = torch.zeros_like(f[:1])
                f = 0.25 * torch.cat([z, f[:-1]]) + 0.5 * f + 0.25 * torch.cat([f[1:], z])
                z = torch.zeros_like(f[:, :1])
                f = 0.25 * torch.cat([par * (f[:, :1] if hr else f[:, 1:2]), f[:, :-1]], 1) + 0.5 * f + 0.25 * torch.cat([f[:, 1:], z], 1)
                new = torch.zeros_like(full)
                new[: f.shape[0], : f.shape[1]] = f
                setattr(self, name, new)

    def _maxwell(self):
        dt, dx, dr, j = self.dt, self.dx, self.dr, self.j
        ji, jh = j[1:-1], j[:-1] + 0.5
        ex, er, bt = self.ex.clone(), self.er.clone(), self.bt
        er[1:-1, :-1] -= dt * ((bt[1:-1, :-1] - bt[:-2, :-1]) / dx + self.jr[1:-1, :-1])
        er[0], er[-1] = 0, 0
        ex[:-1, 0] += dt * (4 * bt[:-1, 0] / dr - self.jx[:-1, 0])
        ex[:-1, 1:-1] += dt * (((ji + 0.5) * bt[:-1, 1:-1] - (ji - 0.5) * bt[:-1, :-2]) / (ji * dr) - self.jx[:-1, 1:-1])
        ex[:, -1] = 0
        new = torch.zeros_like(bt)
        new[:-1, :-1] = bt[:-1, :-1] + dt * ((ex[:-1, 1:] - ex[:-1, :-1]) / dr - (er[1:, :-1] - er[:-1, :-1]) / dx)
        self.ex, self.er, self.bt, self.bt_bar = ex, er, new, 0.5 * (bt + new)
        if not self.m1:
            return
        ex, er, et, bx, br, bt = (getattr(self, k).clone() for k in ("ex1", "er1", "et1", "bx1", "br1", "bt1"))
        ex[:-1, 1:-1] += dt * (((ji + 0.5) * bt[:-1, 1:-1] - (ji - 0.5) * bt[:-1, :-2]) / (ji * dr)
                               + 1j * br[:-1, 1:-1] / (ji * dr) - self.jx1[:-1, 1:-1])
        ex[:, 0], ex[:, -1] = 0, 0
        er[1:-1, :-1] += dt * (-1j * bx[1:-1, :-1] / (jh * dr) - (bt[1:-1, :-1] - bt[:-2, :-1]) / dx - self.jr1[1:-1, :-1])
        et[1:-1, 0] += dt * ((br[1:-1, 0] - br[:-2, 0]) / dx - 2 * bx[1:-1, 0] / dr - self.jt1[1:-1, 0])
        et[1:-1, 1:-1] += dt * ((br[1:-1, 1:-1] - br[:-2, 1:-1]) / dx - (bx[1:-1, 1:-1] - bx[1:-1, :-2]) / dr - self.jt1[1:-1, 1:-1])
        er[0], er[-1], et[0], et[-1], et[:, -1] = 0, 0, 0, 0, 0
        nbx, nbr, nbt = bx.clone(), br.clone(), bt.clone()
        nbx[:, :-1] -= dt * (((j[:-1] + 1) * et[:, 1:] - j[:-1] * et[:, :-1]) / (jh * dr) + 1j * er[:, :-1] / (jh * dr))
        exr = torch.cat([ex[:, 1:2] / dr, ex[:, 1:] / (j[1:] * dr)], 1)
        nbr[:-1] += dt * (1j * exr[:-1] + (et[1:] - et[:-1]) / dx)
        nbt[:-1, :-1] += dt * ((ex[:-1, 1:] - ex[:-1, :-1]) / dr - (er[1:, :-1] - er[:-1, :-1]) / dx)
        self.ex1, self.er1, self.et1, self.bx1, self.br1, self.bt1 = ex, er, et, nbx, nbr, nbt
        self.bx1_bar, self.br1_bar, self.bt1_bar = 0.5 * (bx + nbx), 0.5 * (br + nbr), 0.5 * (bt + nbt)

    def _window(self):
        if not self.cfg["moving_window"] or (self.n + 1) * self.dt < (self.shift + 1) * self.dx:
            return
        self._drop(self.r[0] >= (self.shift + 1) * self.dx)
        half = ("ex", "bt", "bt_bar", "jx", "ex1", "br1", "bt1", "br1_bar", "bt1_bar", "jx1")
        for name in ("env", "env_prev", "chi") + _EM0 + _J0 + (_EM1 + _J1 if self.m1 else ()):
            f = getattr(self, name)
            f = torch.cat([f[1:], torch.zeros_like(f[:1])])
            if name in half:
                f[-2:] = 0
            setattr(self, name, f)
        self.shift += 1
        self.env[0], self.env_prev[0], self.er[0] = 0, 0, 0
        if self.m1:
            self.er1[0], self.et1[0] = 0, 0
        self._load(self.shift + self.nx - 1, self.shift + self.nx)

    # ---- what a program reads
    def sums(self):
        p2 = (self.p ** 2).sum(0)
        sq = lambda f, v: float(((f.abs() ** 2) * v).sum())  # noqa: E731
        u = 0.5 * (sq(self.ex[:-1], self.vn) + sq(self.er[:, :-1], self.vh[:-1]) + sq(self.bt[:-1, :-1], self.vh[:-1]))
        if self.m1:
            u += 0.25 * (sq(self.ex1[:-1], self.vn) + sq(self.er1[:, :-1], self.vh[:-1]) + sq(self.et1, self.vn)
                         + sq(self.bx1[:, :-1], self.vh[:-1]) + sq(self.br1[:-1], self.vn) + sq(self.bt1[:-1, :-1], self.vh[:-1]))
        return {"count": float(self.w.numel()), "charge": -float(self.w.sum()), "chi_v": float((self.chi * self.vn).sum()),
                "kin": float((self.w * p2 / (1 + torch.sqrt(1 + p2))).sum()), "uem": u, "env2_v": sq(self.env, self.vn),
                "px": float((self.w * self.p[0]).sum())}

    def spectrum(self, lo, hi, bins):
        p2 = (self.p ** 2).sum(0)
        e = p2 / (1 + torch.sqrt(1 + p2))
        ok = (e >= lo) & (e < hi)
        k = torch.clamp(torch.floor((e[ok] - lo) / ((hi - lo) / bins)).long(), max=bins - 1)
        h = torch.zeros(bins, dtype=torch.float64, device=self.dev).index_add_(0, k, self.w[ok])
        return h.cpu().numpy(), -float(self.w[ok].sum())


def _bunch_reference(c, seed):
    """E_x, E_r, B_theta and Bbar_theta of the bunch: the discrete relativistic Poisson equation solved by sine
    modes along x and a tridiagonal elimination along r."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    cfg = dict(_config(c, seed), profile="none")
    s = _Reference(cfg)
    b = _bunch(c, seed)
    x, y, z, w = (torch.from_numpy(b[k]).to(dev) for k in ("x", "y", "z", "w"))
    X, R = s._shape(x / s.dx), s._shape(torch.hypot(y, z) / s.dr)
    acc = s._acc()
    for a, wa in enumerate(X[1]):
        for k, wb in enumerate(R[1]):
            acc.index_add_(0, s._index(X[0] + a, R[0] + k), (-w * wa * wb)[:, None])
    rhs = s._fold(acc, 1, False, False, torch.ones_like(s.vn))[1:-1, :-1]
    n, g2 = s.nx - 1, 1 - BETA * BETA
    m = torch.arange(1, n + 1, dtype=torch.float64, device=dev)
    S = torch.sin(math.pi * m[:, None] * m[None, :] / s.nx)
    f = S @ rhs * (2.0 / s.nx)
    lam = (2 - 2 * torch.cos(math.pi * m / s.nx)) * g2 / s.dx ** 2
    face = 2 * math.pi * (s.j[:-1] + 0.5) * s.dx
    low = torch.cat([torch.zeros(1, dtype=torch.float64, device=dev), face[:-1]])
    diag = lam[:, None] * s.vn[:-1] + face + low
    cp, dp = torch.zeros_like(diag), torch.zeros_like(diag)
    for k in range(s.nr):
        den = diag[:, k] + (low[k] * cp[:, k - 1] if k else 0)
        cp[:, k] = -face[k] / den
        dp[:, k] = (f[:, k] + (low[k] * dp[:, k - 1] if k else 0)) / den
    for k in range(s.nr - 2, -1, -1):
        dp[:, k] -= cp[:, k] * dp[:, k + 1]
    phi = torch.zeros((s.nx + 1, s.nr + 1), dtype=torch.float64, device=dev)
    phi[1:-1, :-1] = S @ dp
    ex, er, bt = (torch.zeros_like(phi) for _ in range(3))
    ex[:-1] = -(phi[1:] - phi[:-1]) * g2 / s.dx
    er[:, :-1] = -(phi[:, 1:] - phi[:, :-1]) / s.dr
    bt[:-1, :-1] = BETA * 0.5 * (er[:-1, :-1] + er[1:, :-1])
    return torch.stack([ex, er, bt, bt]).cpu().numpy()
