"""Calls after which the staged layout is made anew: everything the problem holds is carried over."""
import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

DX = 1.0e-3


def _lattice(dims):
    k, j, i = np.meshgrid(*[np.arange(d) for d in dims[::-1]], indexing="ij")
    return DX * np.stack([i.ravel(), j.ravel(), k.ravel()], axis=1).astype(np.float64)


def _problem(sim, dims, m=3.015, c=1.0e19, s0=1.0e-3, scheme="euler_cromer"):
    x = _lattice(dims)
    sim.set_mapping("staged")
    sim.build_family(x, m * DX)
    sim.set_integrator(scheme, 1.0e-8)
    sim.set_material(2400.0, c, s0, 0.0, DX ** 3)
    return x


@pytest.mark.parametrize("how", ["model", "mapping"])
def test_a_non_finite_step_is_still_reported(how):
    """A step that overflowed is not waited for; a call that rebuilds the device problem comes
    before the next check, which must still report it."""
    import paper_2105_04150_amd as pd
    dims = (61, 60, 57)  # four slices a tile: the state-based pairs cut the tiles anew
    with pd.Simulation() as sim:
        x = _problem(sim, dims, s0=1.0e9)
        u = np.zeros_like(x)
        v = np.zeros_like(x)
        v[0] = 1.0e307
        sim.set_state(u=u, v=v)
        sim.set_integrator("euler_cromer", 1.0e3)
        sim.step(1)
        if how == "model":
            sim.set_model("state_based", 1.0e10, 6.0e9)
        else:
            sim.set_mapping("sliced")
        with pytest.raises(pd.PdmiError, match="non-finite"):
            sim.sync()
