"""Kernels at the sizes where their work split changes (edges of tiles and
rounds, remainders, the smallest and largest of a range), against the FP64
oracle.  Tolerances: counts and pair sets exact; sums of n terms of one sign
or of scale s within n eps s, with the margin of the bars of
test_gpu_parity (1e-12 relative)."""
import time

import numpy as np
import pytest
import torch

import oracle as O
from paper_2109_11083_amd import binding as B
from paper_2109_11083_amd import inputs
from paper_2109_11083_amd.sim import Params, Sim, step_batch, workspace_bytes

pytestmark = pytest.mark.gpu


def _oracle_params(p: Params):
    return O.make_params(p.n, p.box, shear_rate=p.shear_rate, dt=p.dt, kT=p.kT, gamma=p.gamma, mass=p.mass,
                         eps=p.eps, sigma=p.sigma, rc=p.rc, fene_k=p.fene_k, fene_r0=p.fene_r0, seed=p.seed,
                         chain_len=p.chain_len, n_chains=p.n_chains, thermostat=p.thermostat, dpd_rc=p.dpd_rc,
                         velocity=p.velocity, angle_k=p.angle_k)


def _lj(n, shear_rate, seed, **kw):
    w = inputs.lj_workload(n=n, shear_rate=shear_rate, seed=seed)
    return w, Params(n=n, box=w.box, shear_rate=shear_rate, seed=seed, **kw)


# one partly filled block; the last size of one round; two rounds with empty blocks at the end
@pytest.mark.parametrize("n,nbins", [(1001, 7), (131072, 256), (131400, 50)])
def test_observables_rounds(n, nbins):
    w, p = _lj(n, 0.3, 5)
    sim = Sim(p, w.x, w.u)
    got = sim.observables(nbins)
    x, u, _, _ = sim.state()
    sim.close()
    ref = O.observables(x, u, 0.0, _oracle_params(p), nbins=nbins)
    assert np.array_equal(got["count"], ref["count"])
    assert np.abs(got["sum_ux"] - ref["sum_ux"]).max() <= 1e-12 * np.abs(u[0]).sum()
    assert np.abs(got["sum_mc2"] - ref["sum_mc2"]).max() <= 1e-12 * ref["sum_mc2"].max()
    assert abs(got["kT"] - ref["kT"]) <= 1e-12 * ref["kT"]
    assert np.abs(got["com"] - ref["com"]).max() <= 1e-12 * np.abs(u).mean()


def _slab(seed):
    """A lattice filling the lowest third of the box: about 80 particles per cell, so
    that a tile's halo holds more positions than the search looks at."""
    rng = np.random.default_rng(seed)
    L = 20.0
    g = [np.arange(26) * (L / 26), np.arange(26) * (L / 26), np.arange(12) * 0.5]
    x = np.stack([a.ravel() for a in np.meshgrid(*g, indexing="ij")]) + rng.uniform(0.0, 0.02, (3, 26 * 26 * 12))
    return x, dict(n=x.shape[1], box=(L, L, L), max_neighbors=900)


def _gas(seed):
    """A gas of 0.08 particles per cell: a tile covers many beams of cells, nothing is staged."""
    rng = np.random.default_rng(seed)
    return rng.uniform(0.0, 60.0, (3, 700)), dict(n=700, box=(60.0, 60.0, 60.0))


def _fluid(n):
    def make(seed):
        w = inputs.lj_workload(n=n, shear_rate=0.2, seed=seed)
        return w.x, dict(n=n, box=w.box)
    return make


def _melt(chains, length, skin):
    def make(seed):
        w = inputs.kg_workload(chains, length, shear_rate=0.2, seed=seed)
        return w.x, dict(n=chains * length, box=w.box, rc=2.0 ** (1.0 / 6.0), pair="wca", n_chains=chains,
                         chain_len=length, skin=skin)
    return make


# small tiles with a ragged end, the last size with small tiles and the first
# with large ones (dense, sparse), a tile in two beams of two widths, and the
# two ways out of the staged halo
SEARCH = {"lj_1009": _fluid(1009), "lj_10000": _fluid(10000), "lj_10001": _fluid(10001), "lj_16500": _fluid(16500),
          "kg_2000": _melt(20, 100, 0.6), "kg_2010": _melt(30, 67, 0.6), "kg_12000_wide": _melt(60, 200, 1.2),
          "slab": _slab, "gas": _gas}


@pytest.mark.parametrize("tune", [1, 2])
@pytest.mark.parametrize("name", list(SEARCH))
def test_list_search_and_forces_at_tile_edges(name, tune):
    """The pair set is the oracle's, exactly; cells and order too; forces and virial within 1e-12."""
    x, kw = SEARCH[name](3)
    p = Params(shear_rate=0.2, seed=3, tune=tune, **{"rc": 2.5, "skin": 0.3, **kw})
    step0 = 1237
    sim = Sim(p, x, np.zeros_like(x), step0=step0)
    out = sim.build_cells()
    F, W = sim.forces()
    sim.close()
    op = _oracle_params(p)
    Delta = O.offset(step0, p.dt, p.shear_rate, p.box[0], p.box[1])
    xw, _ = O.le_wrap(x, np.zeros_like(x), Delta, op)
    nc = tuple(int(np.floor(L / (p.rlist * (1 + 1e-9)))) for L in p.box)
    cells, order = O.cells(xw, nc, p.box)
    assert np.array_equal(out["cell_of"], cells) and np.array_equal(out["order"], order)
    ref = O.pairs_cells(xw, Delta, p.box, p.rlist)
    got = np.sort(out["pairs"][:, 0] * p.n + out["pairs"][:, 1])
    lo, hi = ref.min(axis=1).astype(np.int64), ref.max(axis=1).astype(np.int64)
    assert np.array_equal(got, np.sort(lo * p.n + hi))
    Fr, Wr, _ = O.forces(xw, Delta, op)
    assert np.sqrt(((F - Fr) ** 2).sum(axis=0)).max() <= 1e-12 * np.sqrt((Fr ** 2).sum(axis=0).mean())
    assert np.abs(W - Wr).max() <= 1e-12 * np.abs(Wr[:3]).max()


# the sort in one launch within a step (up to 65,536 particles) and the two
# launches of a batch and of larger systems: whole binning blocks of 512, one
# more, the last size of the one launch and the first of the two.  The same
# arithmetic, so the states are equal bit for bit, also when calls alternate.
@pytest.mark.parametrize("n", [512, 1025, 65536, 65537])
def test_sort_in_one_launch_and_in_two(n):
    w, p = _lj(n, 0.3, 7, skin=0.3)
    a, b = Sim(p, w.x, w.u), Sim(p, w.x, w.u)
    for k in range(4):
        a.step(6)
        if k % 2 == 0:
            step_batch([b], 6)
        else:
            b.step(6)
    (xa, ua, fa, _), (xb, ub, fb, _) = a.state(), b.state()
    assert a.stats() == b.stats() and a.stats()["rebuilds"] > 1
    assert np.array_equal(xa, xb) and np.array_equal(ua, ub) and np.array_equal(fa, fb)
    a.close()
    b.close()


# DPD partners from the LDS halo against partners from global memory: a ragged
# small tile, the first size of large tiles, beads with bonds, and rows of a
# stencil beyond what the halo holds.  The two differ by the rounding of the
# coordinates' images: a few 1e-16 of the box (20 to 25) against distances of
# 0.5 and more in forces up to r^-13, 1e-12 of the largest force; mixed
# precision evaluates the pair force in FP32, 1e-5.
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("name", ["lj_1009", "lj_10001", "kg_12000_wide", "slab"])
def test_dpd_forces_from_the_halo_and_from_memory(name, precision, tol):
    x, kw = SEARCH[name](3)
    u = np.random.default_rng(8).normal(size=x.shape)
    out = []
    for tune in (0, 2):
        p = Params(shear_rate=0.2, seed=3, tune=tune, thermostat="dpd", gamma=5.0, precision=precision,
                   **{"rc": 2.5, "skin": 0.3, **kw})
        sim = Sim(p, x, u, step0=1237)
        out.append(sim.state())
        sim.close()
    (xa, ua, fa, _), (xb, ub, fb, _) = out
    assert np.array_equal(xa, xb) and np.array_equal(ua, ub)
    assert np.abs(fa - fb).max() <= tol * np.abs(fb).max()


# random-walk melts of uneven density: beams narrower than a tile at the box's
# upper faces, and tiles with more halo cells than the search's block has threads
@pytest.mark.parametrize("chains,length", [(15, 200), (30, 200), (100, 300)])
def test_list_search_of_uneven_melts(chains, length):
    """The pair set is the oracle's, exactly."""
    x, kw = _melt(chains, length, 0.3)(3)
    p = Params(shear_rate=0.2, seed=3, **kw)
    sim = Sim(p, x, np.zeros_like(x), step0=1237)
    out = sim.build_cells()
    sim.close()
    op = _oracle_params(p)
    Delta = O.offset(1237, p.dt, p.shear_rate, p.box[0], p.box[1])
    xw, _ = O.le_wrap(x, np.zeros_like(x), Delta, op)
    ref = O.pairs_cells(xw, Delta, p.box, p.rlist)
    got = np.sort(out["pairs"][:, 0] * p.n + out["pairs"][:, 1])
    lo, hi = ref.min(axis=1).astype(np.int64), ref.max(axis=1).astype(np.int64)
    assert np.array_equal(got, np.sort(lo * p.n + hi))


# the launches whose blocks wait for one another (the whole rebuild up to 20,000
# particles, the sort up to 65,536), many at a time on streams of their own: more
# waiting blocks than the GPU holds, in dense small and large tiles, sparse tiles
# and the global layout.  Each steps as it does alone, bit for bit.
def test_rebuilds_of_many_streams_at_once():
    kinds = [("lj_10000", {}), ("lj_10001", {}), ("lj_10000", dict(tune=2)), ("kg_12000_wide", {}),
             ("lj_16500", dict(thermostat="dpd", gamma=5.0)), ("lj_20001", {})]
    make = {**SEARCH, "lj_20001": _fluid(20001)}

    def start(k, stream):
        name, over = kinds[k % len(kinds)]
        x, kw = make[name](k)
        u = np.random.default_rng(k).normal(size=x.shape)
        p = Params(shear_rate=0.2, seed=3 + k, dt=0.002, **{"rc": 2.5, "skin": 0.1, **kw, **over})
        return Sim(p, x, u, stream=stream)

    alone = []
    for k in range(12):
        s = start(k, torch.cuda.Stream())
        s.step(60)
        alone.append((s.state(), s.stats()))
        s.close()
    sims = [start(k, torch.cuda.Stream()) for k in range(12)]
    for _ in range(6):
        for s in sims:
            s.step(10)
    for s, (ref, stats) in zip(sims, alone):
        got = s.state()
        assert all(np.array_equal(a, b) for a, b in zip(got[:3], ref[:3])) and got[3] == ref[3] == 60
        assert s.stats() == stats
        s.close()


# DPD members of a batch restarted from a state with forces (no evaluation before the
# first step), in workspaces that held other data: whole blocks of 256 particles and one
# more, partners from the halo and from memory.  As alone, bit for bit.
@pytest.mark.parametrize("tune", [0, 2])
@pytest.mark.parametrize("n", [2048, 2049])
def test_dpd_restart_in_a_batch(n, tune):
    w, p = _lj(n, 0.3, 7, skin=0.3, thermostat="dpd", gamma=5.0, tune=tune)
    f0 = 0.1 * np.random.default_rng(5).normal(size=w.x.shape)
    sims = []
    for _ in range(2):
        ws = torch.full((workspace_bytes(p),), 255, dtype=torch.uint8, device="cuda")
        sims.append(Sim(p, w.x, w.u, f0=f0, workspace=ws))
    step_batch(sims[:1], 20)
    sims[1].step(20)
    (xa, ua, fa, _), (xb, ub, fb, _) = (s.state() for s in sims)
    assert np.isfinite(fa).all()
    assert np.array_equal(xa, xb) and np.array_equal(ua, ub) and np.array_equal(fa, fb)
    for s in sims:
        s.close()


# non-finite positions are reported as such, one or all of them (all meet in one
# cell, more than its bucket holds)
@pytest.mark.parametrize("bad", [1, 1000])
def test_nonfinite_positions_are_reported(bad):
    w, p = _lj(1000, 0.3, 7)
    x = w.x.copy()
    x[1, :bad] = np.nan
    sim = Sim(p, x, w.u)
    assert sim.stats()["status"] == B.LE_E_NONFINITE
    sim.close()
    xt = torch.as_tensor(x, device="cuda")
    f = torch.empty((3, p.n), dtype=torch.float64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.le_forces_static(p.to_c(), xt.data_ptr(), f.data_ptr(), None, status.data_ptr(), 0,
                       torch.cuda.current_stream().cuda_stream)
    assert int(status.cpu()[0]) == B.LE_E_NONFINITE


# an error that the sort's first blocks latch while later ones have not started
# (3000 blocks): those leave, and no block waits for what they would have published
def test_sort_ends_after_an_error_in_its_first_blocks():
    w, p = _lj(1_500_000, 0.0, 7)
    u = w.u.copy()
    u[2] = np.nan
    Sim(p, w.x, w.u).close()
    t0 = time.perf_counter()
    sim = Sim(p, w.x, u)
    status = sim.stats()["status"]
    elapsed = time.perf_counter() - t0
    assert status == B.LE_E_NONFINITE
    assert elapsed < 2.0  # (the bound of the wait is reached after some seconds)
    sim.close()


# 14 partners each (a body-centred lattice in few, full cells, of which a tile's halo
# holds a part), where the lists have room for 16: whatever the mix of staged
# and walked partners
@pytest.mark.parametrize("tune", [0, 1, 2])
def test_list_capacity_in_any_mix(tune):
    m, L = 12, 30.0
    g = np.arange(m) * (L / m)
    a = np.stack([v.ravel() for v in np.meshgrid(g, g, g, indexing="ij")])
    x = np.concatenate([a, a + 0.5 * L / m], axis=1) + np.random.default_rng(1).uniform(0.0, 0.01, (3, 2 * m ** 3))
    p = Params(n=x.shape[1], box=(L, L, L), rc=2.6, skin=0.2, cells=(3, 3, 3), max_neighbors=16, tune=tune)
    sim = Sim(p, x, np.zeros_like(x))
    out = sim.build_cells()
    F, W = sim.forces()
    assert sim.stats()["max_neighbors"] == 14
    sim.close()
    assert len(out["pairs"]) == 7 * p.n
    Fr, Wr, _ = O.forces(x, 0.0, _oracle_params(p))
    # (in a perfect lattice the forces cancel: against the force of one pair)
    assert np.abs(F - Fr).max() <= 1e-12 * 24.0 / 2.165 ** 7 * 14
    assert np.abs(W - Wr).max() <= 1e-12 * np.abs(Wr[:3]).max()


# lengths in a unit of 2^90 (an exact scaling): sigma^12 is no double, but the forces are
# those of sigma = 1 in that unit
@pytest.mark.parametrize("tune,force_cap", [(1, 0.0), (2, 0.0), (0, 1e6)])
@pytest.mark.parametrize("name", ["lj_1009", "kg_2000"])
def test_forces_in_small_units_of_length(name, tune, force_cap):
    x, kw = SEARCH[name](3)
    kw = {"rc": 2.5, "skin": 0.3, **kw}
    out = []
    for e in (0, -90):
        c = 2.0 ** e
        k = dict(kw, rc=kw["rc"] * c, skin=kw["skin"] * c, box=tuple(L * c for L in kw["box"]), sigma=c,
                 fene_r0=1.5 * c, fene_k=30.0 / c ** 2, force_cap=force_cap / c)
        sim = Sim(Params(shear_rate=0.2, seed=3, tune=tune, **k), x * c, np.zeros_like(x), step0=1237)
        F, W = sim.forces()
        sim.close()
        out.append((F * c, W))
    (Fa, Wa), (Fb, Wb) = out
    assert np.abs(Fa - Fb).max() <= 1e-12 * np.sqrt((Fa ** 2).sum(axis=0).mean())
    assert np.abs(Wa - Wb).max() <= 1e-12 * np.abs(Wa[:3]).max()


def _lattice(density, L):
    a = density ** (-1.0 / 3.0)
    g = np.arange(int(L / a)) * a
    x = np.stack([v.ravel() for v in np.meshgrid(g, g, g, indexing="ij")])
    return x + np.random.default_rng(3).uniform(0.0, 0.1, x.shape)


def _thin(n, L):
    return np.random.default_rng(3).uniform(0.0, L, (3, n)), dict(n=n, box=(L, L, L))


def _part(L, keep):
    x = _lattice(0.8, L)
    x = x[:, keep(x / L)]
    return x, dict(n=x.shape[1], box=(L, L, L), max_neighbors=400)


# cells that are nearly empty (tiles in one, two and more beams, with more halo cells than
# the search's table), and dense parts of mostly empty boxes, at a gradient face and away
UNEVEN = {"gas_1000_50": lambda: _thin(1000, 50.0), "gas_1000_100": lambda: _thin(1000, 100.0),
          "gas_5000_90": lambda: _thin(5000, 90.0), "gas_20000_90": lambda: _thin(20000, 90.0),
          "drop": lambda: _part(50.0, lambda s: ((s - 0.5) ** 2).sum(axis=0) < 0.09),
          "film": lambda: _part(40.0, lambda s: s[1] < 0.2),
          "slab": lambda: _part(40.0, lambda s: s[2] < 0.2)}


@pytest.mark.parametrize("tune", [1, 2])
@pytest.mark.parametrize("name", list(UNEVEN))
def test_list_search_of_gases_and_dense_parts(name, tune):
    """The pair set is the oracle's, exactly; forces and virial within 1e-12 of the largest."""
    x, kw = UNEVEN[name]()
    p = Params(shear_rate=0.2, seed=3, tune=tune, skin=0.3, **kw)
    sim = Sim(p, x, np.zeros_like(x), step0=1237)
    out = sim.build_cells()
    F, W = sim.forces()
    sim.close()
    op = _oracle_params(p)
    Delta = O.offset(1237, p.dt, p.shear_rate, p.box[0], p.box[1])
    xw, _ = O.le_wrap(x, np.zeros_like(x), Delta, op)
    ref = O.pairs_cells(xw, Delta, p.box, p.rlist)
    got = np.sort(out["pairs"][:, 0] * p.n + out["pairs"][:, 1])
    lo, hi = ref.min(axis=1).astype(np.int64), ref.max(axis=1).astype(np.int64)
    assert np.array_equal(got, np.sort(lo * p.n + hi))
    Fr, Wr, _ = O.forces(xw, Delta, op)
    assert np.abs(F - Fr).max() <= 1e-12 * np.abs(Fr).max()
    assert np.abs(W - Wr).max() <= 1e-12 * np.abs(Wr).max()


# Steps alone (the rebuild in one launch up to 20,000 particles, the sort in one up to
# 65,536, separate launches above and where nearly empty cells make more than 512
# blocks) against a batch's separate launches, bit for bit: both lines, a ragged size
# between, a gas on either side of the limit of blocks, and every kind of tile.
STEPS = {"lj_20000": (_fluid(20000), {}), "lj_20001": (_fluid(20001), {}), "lj_33333": (_fluid(33333), {}),
         "gas_1000_130": (lambda seed: _thin(1000, 130.0), {}), "gas_1000_150": (lambda seed: _thin(1000, 150.0), {}),
         "gas_30000_130": (lambda seed: _thin(30000, 130.0), {}), "gas_30000_170": (lambda seed: _thin(30000, 170.0), {}),
         "lj_1009_global": (_fluid(1009), dict(tune=2)), "lj_16500_global": (_fluid(16500), dict(tune=2)),
         "lj_1009_dpd": (_fluid(1009), dict(thermostat="dpd", gamma=5.0)),
         "kg_2010": (_melt(30, 67, 0.6), {}), "kg_12000_wide": (_melt(60, 200, 1.2), dict(skin=0.4)),
         "kg_12000_global": (_melt(60, 200, 0.6), dict(tune=2))}


@pytest.mark.parametrize("name", list(STEPS))
def test_steps_alone_and_in_a_batch(name):
    make, over = STEPS[name]
    x, kw = make(3)
    if name.startswith("gas"):  # no overlaps: a jittered lattice
        m = int(np.ceil(kw["n"] ** (1.0 / 3.0)))
        g = np.arange(m) * (kw["box"][0] / m)
        x = np.stack([v.ravel() for v in np.meshgrid(g, g, g, indexing="ij")])[:, :kw["n"]]
        x = x + np.random.default_rng(4).uniform(0.0, 0.4 * kw["box"][0] / m, x.shape)
    u = np.random.default_rng(8).normal(size=x.shape)
    p = Params(shear_rate=0.3, seed=7, dt=0.004, **{"rc": 2.5, "skin": 0.3, **kw, **over})
    a, b = Sim(p, x, u), Sim(p, x, u)
    for k in range(3):
        a.step(8)
        if k < 2:
            step_batch([b], 8)
        else:
            b.step(8)
    (xa, ua, fa, _), (xb, ub, fb, _) = a.state(), b.state()
    assert a.stats() == b.stats() and a.stats()["rebuilds"] > 2
    assert np.array_equal(xa, xb) and np.array_equal(ua, ub) and np.array_equal(fa, fb)
    a.close()
    b.close()


# the reported order over several blocks of cells (one block of 1024 cells, one cell
# more than that, and 215,940), cells of unequal edges
@pytest.mark.parametrize("cells", [(16, 8, 8), (41, 5, 5), (59, 61, 60)])
def test_cell_order_over_many_cells(cells):
    box = tuple(3.0 * c for c in cells)
    x = np.random.default_rng(6).uniform(0.0, 1.0, (3, 5000)) * np.array(box)[:, None]
    p = Params(n=5000, box=box, shear_rate=0.2, rc=2.5, skin=0.3, cells=cells)
    sim = Sim(p, x, np.zeros_like(x), step0=1237)
    out = sim.build_cells(want_pairs=False)
    again = sim.build_cells(want_pairs=False)
    sim.close()
    xw, _ = O.le_wrap(x, np.zeros_like(x), O.offset(1237, p.dt, p.shear_rate, box[0], box[1]), _oracle_params(p))
    ref_cells, ref_order = O.cells(xw, cells, box)
    for o in (out, again):
        assert np.array_equal(o["cell_of"], ref_cells) and np.array_equal(o["order"], ref_order)


# as many bins in a wave as it has lanes, one bin, and just what it takes one by one
@pytest.mark.parametrize("nbins", [1, 9, 256])
def test_observables_with_few_particles_per_bin(nbins):
    test_observables_rounds(1000, nbins)
