"""CPU checks of the pair layout the host chooses, seen in the workspace it asks for."""
import math

import pytest

from paper_2109_11083_amd.sim import Params, workspace_bytes


def _box(n, density):
    return ((n / density) ** (1.0 / 3.0),) * 3


# the systems of the GPU test that compares DPD partners from the LDS halo (tune 0) with
# partners from memory (tune 2): with one layout for both it would compare a kernel with itself
@pytest.mark.parametrize("kw", [
    dict(n=1009, box=_box(1009, 0.8442), rc=2.5, skin=0.3),
    dict(n=10001, box=_box(10001, 0.8442), rc=2.5, skin=0.3),
    dict(n=12000, box=_box(12000, 0.85), rc=2.0 ** (1.0 / 6.0), pair="wca", n_chains=60, chain_len=200, skin=1.2),
    dict(n=8112, box=(20.0, 20.0, 20.0), rc=2.5, skin=0.3, max_neighbors=900)])
def test_dense_dpd_systems_take_the_halo(kw):
    p0, p2 = (Params(thermostat="dpd", gamma=5.0, tune=t, **kw) for t in (0, 2))
    langevin = {t: workspace_bytes(Params(tune=t, **kw)) for t in (0, 1, 2)}
    assert langevin[0] == langevin[1] != langevin[2]
    # (as much larger as the Langevin layouts are apart, less the rounding of the arrays)
    assert math.isclose(workspace_bytes(p0) - workspace_bytes(p2), langevin[1] - langevin[2], abs_tol=1024)


# the largest systems that the no-allocation entry point took when both kinds of a list
# had units of their own and small tiles did not exist: it still takes them
@pytest.mark.parametrize("n,density,kw", [
    (37119, 0.8442, dict(rc=2.5)), (29119, 0.01, dict(rc=2.5)), (59136, 0.85, dict(rc=2.0 ** (1.0 / 6.0), pair="wca")),
    (36607, 0.8442, dict(rc=2.5, thermostat="dpd")), (2000, 0.8442, dict(rc=2.5, max_neighbors=5392)),
    (5000, 0.8442, dict(rc=2.5, max_neighbors=2112)), (10000, 0.8442, dict(rc=2.5, max_neighbors=1024))])
def test_sizes_that_fit_the_library_s_own_scratch(n, density, kw):
    assert workspace_bytes(Params(n=n, box=_box(n, density), skin=0.3, **kw)) <= 64 << 20
