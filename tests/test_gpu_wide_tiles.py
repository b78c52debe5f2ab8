"""Tiles of a wide horizon: single slices, some of whose records do not fit a CU's LDS twice and
take two passes, against the direct sum in 64-bit arithmetic."""
import numpy as np
import pytest

from parity import say
from test_gpu_tiles import C, DX, VOL, _direct, _lattice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,m,weights", [
    ((37, 33, 29), 5.015, False),
    ((37, 33, 29), 5.015, True),    # with 8 bytes more a record: other cuts
    ((41, 30, 28), 6.015, False),
])
def test_force_of_wide_tiles(dims, m, weights):
    import paper_2105_04150_amd as pd
    rng = np.random.default_rng(3)
    x = _lattice(dims)
    u = 1e-3 * (x * [1.0, -0.3, 0.2] + 0.3 * DX * rng.uniform(-1, 1, x.shape))
    vol = VOL * (rng.uniform(0.5, 1.5, len(x)) if weights else np.ones(len(x)))
    with pd.Simulation(0, pd.PD_FP64) as sim:
        sim.set_mapping("staged")
        sim.build_family(x, m * DX)
        sim.set_integrator("euler_cromer", 1.0e-9)
        sim.set_material(2400.0, C, 10.0, 0.0, VOL, vol if weights else None)
        sim.set_state(u=u)
        got = sim.force()
    want = _direct(dims, m, u, vol)
    # the rounding of |y|^2 - |xi|^2 (4 units of 2^-52 over the strain) and the slots' 6.5e-14
    tol = 4 * 2.0 ** -52 / 1e-3 + 6.5e-14
    err = np.abs(got - want).max() / np.abs(want).max()
    say(f"[wide] {dims} m {m}: {err:.2e} (tolerance {tol:.1e})")
    assert err <= tol
