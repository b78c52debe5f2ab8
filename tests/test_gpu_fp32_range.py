"""Range of the FP32 build: stiffness fields, volumes and family volumes whose single factors
leave the range of single precision while the force densities do not."""
import numpy as np
import pytest

from parity import say
from test_gpu_tiles import _direct, _lattice
import test_gpu_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dx", [1.0e-3, 1.0e-8, 1.0e-13])
@pytest.mark.parametrize("what", ["slot", "slot_volumes", "node", "volumes", "corrections"])
def test_small_lengths(what, dx):
    """A lattice in ever smaller length units: c as 1/dx^4, V as dx^3.  The bar is the FP32
    build's: the rounding of the bond vectors, 1e-5."""
    import paper_2105_04150_amd as pd
    dims, m = (9, 8, 7), 3.015
    x = _lattice(dims) * (dx / tiles.DX)
    n = len(x)
    rng = np.random.default_rng(2)
    u = 1.0e-3 * (x * [1.0, -0.3, 0.2])
    c, vol = 1.0e11 / dx ** 4, dx ** 3
    uneven = rng.uniform(0.5, 1.5, n) if what in ("volumes", "slot_volumes") else np.ones(n)
    with pd.Simulation(0, pd.PD_FP32) as sim:
        sim.set_mapping("staged")
        sim.build_family(x, m * dx)
        sim.set_integrator("euler_cromer", 1.0e-9)
        sim.set_material(2400.0, c, 10.0, 0.0, vol, vol * uneven if not (uneven == 1.0).all() else None)
        if what.startswith("slot"):
            sim.set_bond_stiffness(c * np.ones(sim.family()[0][-1]))
        elif what == "node":
            sim.set_node_stiffness(c * np.ones(n))
        elif what == "corrections":
            sim.set_corrections({"micro": "constant", "surface": True, "delta": m * dx})
        sim.set_state(u=u)
        got = sim.force()
        if what == "corrections":
            rp, col = sim.family()
    assert np.isfinite(got).all()
    scale = tiles.DX / dx
    want = _direct(dims, m, u * scale, uneven) * (c * vol / tiles.C)  # C V of one in that unit
    if what == "corrections":  # the same sum over the bonds, with the surface factor
        row = np.repeat(np.arange(n), np.diff(rp))
        fam = np.bincount(row, minlength=n) * 1.0
        xi = (x[col] - x[row]) / dx
        eta = (u[col] - u[row]) / dx
        y = xi + eta
        r, L = np.sqrt((y * y).sum(1)), np.sqrt((xi * xi).sum(1))
        s = (eta * (xi + y)).sum(1) / (L * (r + L))
        f = (c * vol * 2.0 * fam.max() / (fam[row] + fam[col]) * s / r)[:, None] * y
        want = np.stack([np.bincount(row, f[:, d], minlength=n) for d in range(3)], axis=1)
    err = np.abs(got - want).max() / np.abs(want).max()
    say(f"[fp32 range] {what} dx {dx:g}: {err:.2e}")
    assert err <= 1e-5
