"""Kernels at the sizes where their work split changes (edges of tiles and
rounds, remainders, the smallest and largest of a range), against the FP64
oracle.  Tolerances: counts and pair sets exact; sums of n terms of one sign
or of scale s within n eps s, with the margin of the bars of
test_gpu_parity (1e-12 relative)."""
import numpy as np
import pytest

import oracle as O
from paper_2109_11083_amd import inputs
from paper_2109_11083_amd.sim import Params, Sim

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
