"""Performance cases of the Lees-Edwards shear-flow library: what its users run.

A pass is one chunk of a program's main loop (some steps with the stress
sampled every ten, then the state or the analysis the program reads), or one
force evaluation of a given configuration, through the public entry points
(Sim, StepGraph, BatchGraph, the C ABI's binding).  Sizes are those of the
repository's tests, benchmark and sweeps: LJ fluids of 1000 to 256,000
particles at density 0.8442, Kremer-Grest melts of up to 800,000 beads at
0.85, and batches of such systems.  Starts are the lattice starts of
paper_2109_11083_amd.inputs (overlap-free, made on the host from the seed
alone), or random walks where the capped warm-up is the subject.

exact() integrates the same motion in plain float64 torch (pair lists from a
direct search, the crossing applied to every particle every step).
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2109_11083_amd import binding as B
from paper_2109_11083_amd import inputs
from paper_2109_11083_amd.serve import request_params, sweep_trace
from paper_2109_11083_amd.sim import BatchGraph, Params, Sim, StepGraph
from paper_2109_11083_amd.tune import filling_skin

WCA_RC = 2.0 ** (1.0 / 6.0)
SAMPLE_EVERY = 10
MSD_BINS = 50   # bins of the profiles along the gradient axis


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # forces of one configuration for a caller that holds no simulation (le_forces_static):
        # the smallest call of the library, bounded by its chain of launches
        dict(name="forces_lj_1000", kind="forces", model="lj", n=1000, shear=0.1, precision="fp64"),
        # the same at the size limit of the library's own scratch, in mixed precision
        dict(name="forces_lj_27000_mixed", kind="forces", model="lj", n=27000, shear=0.1, precision="mixed"),
        # the smallest run of the tests: 1000 LJ particles, launches and latency only
        dict(name="step_lj_1000", kind="step", model="lj", n=1000, shear=0.1, steps=100, thermostat="langevin",
             velocity="lab"),
        # one serving request run alone: chunks of 100 steps replayed as a HIP graph; odd size
        dict(name="graph_lj_17389", kind="graph", model="lj", n=17389, shear=0.03, steps=100,
             thermostat="langevin", velocity="lab"),
        # the LJ fluid of the benchmark
        dict(name="step_lj_256000", kind="step", model="lj", n=256000, shear=0.1, steps=50, thermostat="langevin",
             velocity="lab"),
        # the paper's own velocity storage at a high shear rate, in between
        dict(name="step_lj_64000_peculiar", kind="step", model="lj", n=64000, shear=1.0, steps=50,
             thermostat="langevin", velocity="peculiar"),
        # the benchmark's headline melt
        dict(name="step_kg_400000", kind="step", model="kg", chains=2000, length=200, shear=0.01, steps=50, dt=0.01,
             angle=0.0),
        # a mid-size melt with the paper's bending term
        dict(name="step_kg_50000_angle", kind="step", model="kg", chains=250, length=200, shear=0.1, steps=50,
             dt=0.005, angle=1.5),
        # the momentum-conserving thermostat
        dict(name="step_dpd_256000", kind="step", model="lj", n=256000, shear=0.1, steps=20, thermostat="dpd",
             velocity="lab"),
        # a full server: 64 requests of 2000 to 64,000 particles advanced as one batch, mixed precision
        dict(name="batch_lj_64_mixed", kind="batch", model="lj", count=64, trace=41, steps=40, precision="mixed"),
        # the sweep of 16 melts over shear rates, with the unwrapped coordinates of its MSD
        dict(name="batch_kg_16", kind="batch", model="kg", count=16, trace=51, steps=100, precision="fp64"),
        # profiles, MSD and stress read every 20 steps (Figs. profile and msd)
        dict(name="analysis_lj_256000", kind="analysis", model="lj", n=256000, shear=0.5, steps=20,
             thermostat="langevin", velocity="lab"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forces", "step", "step", "graph", "kg", "kg", "dpd", "batch", "batch_kg", "analysis",
                       "warmup"])
    shear = float("%.4g" % math.exp(rng.uniform(math.log(1e-3), 0.0)))
    if kind == "forces":
        if rng.random() < 0.5:
            return dict(kind="forces", model="lj", n=_log_int(rng, 1000, 27000), shear=shear,
                        precision=rng.choice(["fp64", "mixed"]))
        return dict(kind="forces", model="kg", chains=_log_int(rng, 10, 100), length=rng.randint(50, 300), shear=shear,
                    precision=rng.choice(["fp64", "mixed"]))
    if kind in ("step", "graph"):
        return dict(kind=kind, model="lj", n=_log_int(rng, 1000, 256000), shear=shear,
                    steps=rng.choice([20, 50, 100]),
                    thermostat=rng.choice(["langevin", "langevin_abs"]) if kind == "step" else "langevin",
                    velocity="lab")
    if kind == "kg":
        return dict(kind="step", model="kg", chains=_log_int(rng, 50, 2000), length=rng.randint(100, 400),
                    shear=float("%.4g" % min(shear, 0.1)), steps=rng.choice([20, 50]), dt=0.005,
                    angle=rng.choice([0.0, 1.5]))
    if kind == "dpd":
        return dict(kind="step", model="lj", n=_log_int(rng, 2000, 256000), shear=shear, steps=20, thermostat="dpd",
                    velocity="lab")
    if kind == "batch":
        precision = rng.choice(["fp64", "mixed"])
        return dict(kind="batch", model="lj", count=rng.randint(3, 40), trace=rng.randint(100, 999),
                    steps=40 if precision == "mixed" else 100, precision=precision)
    if kind == "batch_kg":
        return dict(kind="batch", model="kg", count=rng.randint(3, 16), trace=rng.randint(100, 999), steps=100,
                    precision="fp64")
    if kind == "analysis":
        return dict(kind="analysis", model="lj", n=_log_int(rng, 2000, 256000), shear=shear, steps=20,
                    thermostat="langevin", velocity="lab")
    # the first capped stage of the warm-up of a random-walk melt
    return dict(kind="warmup", model="kg", chains=_log_int(rng, 50, 400), length=rng.randint(100, 300), shear=0.0,
                steps=50, dt=0.002, angle=0.0)


# ------------------------------------------------------------- their inputs
def _filled(p, skin):
    f = filling_skin(p, skin)
    return dataclasses.replace(p, skin=f if f is not None else skin)


def _system(case, seed):
    """(x, u, Params) of a single system (host arrays)."""
    kind, precision = case["kind"], case.get("precision", "fp64")
    if case["model"] == "lj":
        therm = case.get("thermostat", "langevin")
        velocity = case.get("velocity", "lab")
        w = inputs.lj_workload(n=case["n"], shear_rate=case["shear"] if velocity == "lab" else 0.0, seed=seed)
        p = Params(n=case["n"], box=w.box, shear_rate=case["shear"], seed=seed, precision=precision, rc=2.5,
                   dt=0.005, kT=1.0, gamma=5.0 if therm == "dpd" else 1.0, thermostat=therm, velocity=velocity)
        if kind == "forces":
            return w.x, w.u, p  # the default skin: a single evaluation keeps no lists
        # the cell-filling skins the autotuner takes: 0.3 under DPD, 0.4 for requests, 0.5 for a large fluid
        return w.x, w.u, _filled(p, 0.3 if therm == "dpd" else 0.5 if case["n"] >= 100000 else 0.4)
    w = inputs.kg_workload(case["chains"], case["length"], shear_rate=case["shear"], seed=seed,
                           layout="walk" if kind == "warmup" else "snake")
    p = Params(n=w.x.shape[1], box=w.box, shear_rate=case["shear"], seed=seed, precision=precision, rc=WCA_RC,
               pair="wca", n_chains=case["chains"], chain_len=case["length"], dt=case.get("dt", 0.005), kT=1.0,
               gamma=0.5, angle_k=case.get("angle", 0.0))
    if kind == "warmup":
        return w.x, w.u, dataclasses.replace(p, gamma=1.0, force_cap=10.0)
    return w.x, w.u, _filled(p, 0.6) if kind == "step" else p


def _members(case, seed):
    """[(x, u, Params)] of a batch: sizes and shear rates from case["trace"], states from seed."""
    out = []
    if case["model"] == "lj":
        for r in sweep_trace(count=case["count"], seed=case["trace"], precision=case["precision"], burst=True):
            w, p = request_params(dataclasses.replace(r, seed=1000 * seed + r.rid))
            out.append((w.x, w.u, p))
        return out
    rng = np.random.default_rng(case["trace"])
    for k in range(case["count"]):
        chains, length = int(round(0.1 * rng.integers(500, 2001))), int(rng.integers(100, 401))
        shear = 10.0 ** (-4.0 + 3.0 * k / case["count"])
        w = inputs.kg_workload(chains, length, shear_rate=shear, seed=1000 * seed + k)
        p = Params(n=w.x.shape[1], box=w.box, shear_rate=shear, seed=1000 * seed + k, rc=WCA_RC, pair="wca",
                   precision=case["precision"], n_chains=chains, chain_len=length, dt=0.005, kT=1.0, gamma=0.5)
        out.append((w.x, w.u, _filled(p, 0.5)))
    return out


def _step0(seed):
    return 250 + seed % 1000  # forces of a configuration part way through a sheared run


class _Program:
    """What a program keeps between its passes."""

    def __init__(self):
        self.graph = None

    def __del__(self):
        if self.graph is not None:
            self.graph.close()


def prepare(case, seed):
    s = _Program()
    s.kind, s.steps = case["kind"], case.get("steps", 0)
    f64 = dict(dtype=torch.float64, device="cuda")
    if s.kind == "batch":
        stream = torch.cuda.Stream()
        s.sims = [Sim(p, x, u, stream=stream) for x, u, p in _members(case, seed)]
        s.rings = [torch.zeros((s.steps // SAMPLE_EVERY, 6), **f64) for _ in s.sims]
        torch.cuda.synchronize()
        s.graph = BatchGraph(s.sims, s.steps, SAMPLE_EVERY, s.rings)
        s.msd = case["model"] == "kg"
        return s
    x, u, p = _system(case, seed)
    s.f = torch.zeros((3, p.n), **f64)
    if s.kind == "forces":
        s.c, s.step0 = p.to_c(), _step0(seed)
        s.x = torch.as_tensor(x, device="cuda")
        s.w = torch.zeros(6, **f64)
        s.status = torch.zeros(1, dtype=torch.int32, device="cuda")
        return s
    stream = torch.cuda.Stream() if s.kind == "graph" else None
    s.sim = Sim(p, x, u, stream=stream)
    s.ring = torch.zeros((s.steps // SAMPLE_EVERY, 6), **f64)
    if s.kind == "analysis":
        s.ref = s.sim.unwrapped(host=False)
        return s
    s.x, s.u = torch.zeros_like(s.f), torch.zeros_like(s.f)
    if s.kind == "graph":
        torch.cuda.synchronize()
        s.graph = StepGraph(s.sim, s.steps, SAMPLE_EVERY, s.ring)
    return s


# ------------------------------------------------------------------- a pass
def run(s):
    if s.kind == "forces":
        B.le_forces_static(s.c, s.x.data_ptr(), s.f.data_ptr(), s.w.data_ptr(), s.status.data_ptr(), s.step0,
                           torch.cuda.current_stream().cuda_stream)
        return dict(f=s.f, virial=s.w, status=s.status)
    if s.kind == "batch":
        s.graph.launch()
        if s.msd:
            return dict(stress=s.rings, yz=[m.unwrapped(host=False) for m in s.sims])
        return dict(stress=s.rings)
    if s.kind == "analysis":
        s.sim.step(s.steps, SAMPLE_EVERY, s.ring)
        return dict(ring=s.ring, profiles=s.sim.observables(MSD_BINS), msd=s.sim.msd(s.ref), stress=s.sim.stress())
    if s.kind == "graph":
        s.graph.launch()
    else:
        s.sim.step(s.steps, SAMPLE_EVERY, s.ring)
    step = B.le_get_state(s.sim.handle, s.x.data_ptr(), s.u.data_ptr(), s.f.data_ptr())
    return dict(ring=s.ring, x=s.x, u=s.u, f=s.f, step=step)


def _pairs_per_particle(rc, density):
    return 4.0 / 3.0 * math.pi * rc ** 3 * density / 2.0


def _particles(case):
    """[(number, pairs per particle, bonds per particle)] of the systems of a case."""
    lj = _pairs_per_particle(2.5, inputs.LJ_DENSITY)
    kg = _pairs_per_particle(WCA_RC, inputs.KG_DENSITY)
    if case["kind"] == "batch":
        if case["model"] == "lj":
            return [(r.n, lj, 0.0) for r in sweep_trace(count=case["count"], seed=case["trace"], burst=True)]
        rng = np.random.default_rng(case["trace"])
        return [(int(round(0.1 * rng.integers(500, 2001))) * int(rng.integers(100, 401)), kg, 1.0)
                for _ in range(case["count"])]
    return [(case["n"], lj, 0.0)] if case["model"] == "lj" else [(case["chains"] * case["length"], kg, 1.0)]


def work(case):
    """Per step and particle: read x, u and the tag, write x and u (100 bytes); 26 operations
    a pair (56 with the pair thermostat), 26 a bond, 40 for the integrator and thermostat.
    A force evaluation reads positions and writes forces."""
    nbytes = flops = 0.0
    pair_flops = 56.0 if case.get("thermostat") == "dpd" else 26.0
    for n, pairs, bonds in _particles(case):
        per = pairs * pair_flops + bonds * 26.0
        if case["kind"] == "forces":
            nbytes += 48.0 * n
            flops += n * per
        else:
            nbytes += case["steps"] * 100.0 * n
            flops += case["steps"] * n * (per + 40.0)
            nbytes += {"step": 72.0, "warmup": 72.0, "graph": 72.0, "analysis": 100.0,
                       "batch": 16.0 if case["model"] == "kg" else 0.0}[case["kind"]] * n
    return dict(bytes=nbytes, flops=flops)


# ---------------------------------------------- the same motion in 64 bits
def _offset(p, step):
    d = math.fmod(p.shear_rate * p.box[1] * (step * p.dt), p.box[0])
    return d + p.box[0] if d < 0.0 else d


def _philox0(c, key):
    """Philox4x32-10 (Salmon et al. 2011) on int64 tensors holding 32-bit words."""
    m32 = 0xFFFFFFFF
    k0, k1 = key
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57   # low 64 bits, wrapping
        c = [((p1 >> 32) & m32) ^ c[1] ^ k0, p1 & m32, ((p0 >> 32) & m32) ^ c[3] ^ k1, p0 & m32]
    return c


def _theta(word):
    return (word.double() + 0.5) / 4294967296.0 - 0.5


class _Exact:
    """Velocity Verlet under the Lees-Edwards boundary, every particle crossed and wrapped every step."""

    def __init__(self, x, u, p, step0):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.p, self.step, self.dev = p, step0, dev
        self.x = torch.as_tensor(np.ascontiguousarray(x), device=dev).clone()
        self.u = torch.as_tensor(np.ascontiguousarray(u), device=dev).clone()
        self.yz = self.x[1:].clone()                     # unwrapped
        self.sv = p.shear_rate * p.box[1]
        self.pec = p.velocity == "peculiar"
        self.half = 0.5 * p.box[1]
        self.Delta = _offset(p, step0)
        self.built = None
        self._cross()

    def _cross(self):
        Lx, Ly, Lz = self.p.box
        ky = torch.floor(self.x[1] / Ly)
        self.x[1] -= ky * Ly
        self.x[0] -= ky * self.Delta
        if not self.pec:
            self.u[0] -= ky * self.sv
        self.x[0] -= torch.floor(self.x[0] / Lx) * Lx
        self.x[2] -= torch.floor(self.x[2] / Lz) * Lz

    def _disp(self, i, j):
        Lx, Ly, Lz = self.p.box
        d = self.x[:, i] - self.x[:, j]
        sy = torch.round(d[1] / Ly)
        d[1] -= sy * Ly
        d[0] -= sy * self.Delta
        d[0] -= torch.round(d[0] / Lx) * Lx
        d[2] -= torch.round(d[2] / Lz) * Lz
        return d, sy

    def _peculiar(self):
        c = self.u.clone()
        if not self.pec:
            c[0] -= self.p.shear_rate * (self.x[1] - self.half)
        return c

    def _search(self, r):
        """Every pair i < j within r: particles in chunks along z against their window of z."""
        p, n = self.p, self.p.n
        Lx, Ly, Lz = p.box
        order = torch.argsort(self.x[2])
        z = self.x[2][order]
        zz, oo = torch.cat([z - Lz, z, z + Lz]), torch.cat([order, order, order])
        chunk = max(64, min(n, int(4e7 / (n * min(1.0, (2 * r + 1.0) / Lz)))))
        xs = self.x
        got = []
        for a in range(0, n, chunk):
            i = order[a:a + chunk]
            ends = torch.stack([z[a] - r, z[min(a + chunk, n) - 1] + r])
            lo, hi = torch.searchsorted(zz, ends).tolist()
            j = oo[lo:min(hi, lo + n)]
            d1 = xs[1, i][:, None] - xs[1, j][None, :]
            sy = torch.round(d1 / Ly)
            r2 = (d1 - sy * Ly) ** 2
            d0 = xs[0, i][:, None] - xs[0, j][None, :] - sy * self.Delta
            r2 += (d0 - torch.round(d0 / Lx) * Lx) ** 2
            d2 = xs[2, i][:, None] - xs[2, j][None, :]
            r2 += (d2 - torch.round(d2 / Lz) * Lz) ** 2
            k, m = torch.nonzero((r2 < r * r) & (i[:, None] < j[None, :]), as_tuple=True)
            got.append((i[k], j[m]))
        self.i, self.j = torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got])

    def _pairs(self):
        """The pair list, searched again before any pair outside it can have come within r_c."""
        extra = 0.6
        if self.built is not None:
            t0, path = self.built
            s = abs(self.p.shear_rate) * (self.step - t0) * self.p.dt
            g = 0.5 * s + math.sqrt(1.0 + 0.25 * s * s)
            if g * (self.p.rc + 2.0 * g * path) < self.p.rc + extra:
                return
        self._search(min(self.p.rc + extra, 0.5 * min(self.p.box)))
        self.built = (self.step, 0.0)

    def _forces(self):
        """Conservative forces and virial, and the pair thermostat's forces (or None)."""
        p = self.p
        self._pairs()
        i, j = self.i, self.j
        d, sy = self._disp(i, j)
        r2 = (d * d).sum(dim=0)
        keep = r2 < p.rc * p.rc
        i, j, d, sy, r2 = i[keep], j[keep], d[:, keep], sy[keep], r2[keep]
        s6 = (p.sigma * p.sigma / r2) ** 3
        f = 24.0 * p.eps * s6 * (2.0 * s6 - 1.0) / r2
        if p.force_cap > 0.0:
            lim = p.force_cap / torch.sqrt(r2)
            f = torch.minimum(torch.maximum(f, -lim), lim)
        F = torch.zeros_like(self.x)
        W = torch.zeros(6, dtype=torch.float64, device=self.dev)

        def add(i, j, d, f):
            g = f * d
            F.index_add_(1, i, g)
            F.index_add_(1, j, -g)
            for k, (a, b) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
                W[k] += (d[a] * g[b]).sum()

        add(i, j, d, f)
        G = None
        if p.thermostat == "dpd":
            rc = p.dpd_rc or p.rc
            r = torch.sqrt(r2)
            e = d / r
            v = self.u[:, i] - self.u[:, j]
            v[0] -= sy * self.sv
            w = torch.clamp(1.0 - r / rc, min=0.0)
            words = _philox0([torch.full_like(i, self.step & 0xFFFFFFFF), torch.full_like(i, self.step >> 32),
                              torch.minimum(i, j), torch.maximum(i, j)],
                             (p.seed & 0xFFFFFFFF, ((p.seed >> 32) & 0xFFFFFFFF) ^ 0x44504421))
            g = (-p.gamma * w * w * (e * v).sum(dim=0)
                 + math.sqrt(24.0 * p.gamma * p.kT / p.dt) * w * _theta(words[0])) * e
            G = torch.zeros_like(F)
            G.index_add_(1, i, g)
            G.index_add_(1, j, -g)
        if p.n_chains > 0:
            t = torch.arange(p.n_chains * p.chain_len, device=self.dev).view(p.n_chains, p.chain_len)
            a, b = t[:, :-1].reshape(-1), t[:, 1:].reshape(-1)
            d, _ = self._disp(a, b)
            add(a, b, d, -p.fene_k / (1.0 - (d * d).sum(dim=0) / p.fene_r0 ** 2))
            if p.angle_k != 0.0 and p.chain_len >= 3:
                a, m, b = t[:, :-2].reshape(-1), t[:, 1:-1].reshape(-1), t[:, 2:].reshape(-1)
                b1, b2 = self._disp(a, m)[0], self._disp(b, m)[0]
                l11, l22 = (b1 * b1).sum(dim=0), (b2 * b2).sum(dim=0)
                l12 = torch.sqrt(l11) * torch.sqrt(l22)
                c = (b1 * b2).sum(dim=0) / l12
                Fa, Fb = -p.angle_k * (b2 / l12 - c * b1 / l11), -p.angle_k * (b1 / l12 - c * b2 / l22)
                F.index_add_(1, a, Fa)
                F.index_add_(1, b, Fb)
                F.index_add_(1, m, -(Fa + Fb))
                for k, (q, s) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
                    W[k] += (b1[q] * Fa[s] + b2[q] * Fb[s]).sum()
        self.W = W
        return F, G

    def total_force(self):
        p = self.p
        F, G = self._forces()
        if G is not None:
            return F + G
        tag = torch.arange(p.n, device=self.dev)
        words = _philox0([torch.full_like(tag, self.step & 0xFFFFFFFF), torch.full_like(tag, self.step >> 32), tag,
                          torch.zeros_like(tag)], (p.seed & 0xFFFFFFFF, (p.seed >> 32) & 0xFFFFFFFF))
        c = self.u if p.thermostat == "langevin_abs" else self._peculiar()
        noise = torch.stack([_theta(words[a]) for a in range(3)])
        return F - p.gamma * p.mass * c + math.sqrt(24.0 * p.gamma * p.mass * p.kT / p.dt) * noise

    def stress(self):
        c = self._peculiar()
        K = torch.stack([self.p.mass * (c[a] * c[b]).sum()
                         for a, b in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))])
        return -(K + self.W) / (self.p.box[0] * self.p.box[1] * self.p.box[2])

    def advance(self, steps):
        """The stress samples of `steps` steps."""
        p = self.p
        self.F = self.total_force()
        ring = []
        for k in range(1, steps + 1):
            self.u += 0.5 * p.dt / p.mass * self.F
            self.built = (self.built[0], self.built[1] + p.dt * math.sqrt(float(
                (self._peculiar() ** 2).sum(dim=0).max())))
            y = self.x[1].clone()
            self.x += p.dt * self.u
            if self.pec:
                self.x[0] += p.dt * p.shear_rate * (y - self.half)
            self.yz += p.dt * self.u[1:]
            self.step += 1
            self.Delta = _offset(p, self.step)
            self._cross()
            self.F = self.total_force()
            self.u += 0.5 * p.dt / p.mass * self.F
            if k % SAMPLE_EVERY == 0:
                ring.append(self.stress())
        return torch.stack(ring)


def _exact_profiles(e):
    p = e.p
    lab = e.u[0] + (p.shear_rate * (e.x[1] - e.half) if e.pec else 0.0)
    mc2 = p.mass * (e._peculiar() ** 2).sum(dim=0)
    b = (e.x[1] / p.box[1] * MSD_BINS).long().clamp(0, MSD_BINS - 1)

    def hist(v):
        return torch.zeros(MSD_BINS, dtype=torch.float64, device=e.dev).index_add_(0, b, v).cpu().numpy()

    return dict(count=hist(torch.ones_like(lab)), sum_ux=hist(lab), sum_mc2=hist(mc2),
                kT=float(mc2.sum() / (3.0 * p.n - 3.0)),
                com=torch.stack([lab.mean(), e.u[1].mean(), e.u[2].mean()]).cpu().numpy())


def exact(case, seed):
    if case["kind"] == "batch":
        stress, yz = [], []
        for x, u, p in _members(case, seed):
            e = _Exact(x, u, p, 0)
            stress.append(e.advance(case["steps"]))
            yz.append(e.yz)
        return dict(stress=stress, yz=yz) if case["model"] == "kg" else dict(stress=stress)
    x, u, p = _system(case, seed)
    if case["kind"] == "forces":
        e = _Exact(x, u, p, _step0(seed))
        f, _ = e._forces()
        return dict(f=f, virial=e.W, status=None)
    e = _Exact(x, u, p, 0)
    ref = e.yz.clone()
    ring = e.advance(case["steps"])
    if case["kind"] == "analysis":
        return dict(ring=ring, profiles=_exact_profiles(e), msd=((e.yz - ref) ** 2).mean(dim=1).cpu().numpy(),
                    stress=e.stress().cpu().numpy())
    return dict(ring=ring, x=e.x, u=e.u, f=e.F, step=None)
