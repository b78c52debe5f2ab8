"""The staged kernels' tiles: one force evaluation against a direct sum over lattice offsets in
64-bit arithmetic, at the sizes where the tiles change (one node, a slice and one node more,
two slices a tile from 512 slices on, four from 3072), where a tile's records take several
passes through LDS (horizon 8 spacings), and at strains on every side of the ranges of the
kernels' series (short, long, closed form; FP32 the same).

Tolerance, norm-wise: the short series' 1e-12, and the rounding of |y|^2 - |xi|^2 (both
builds' reference forms it as the kernels do not: 4 units of 2^-52 over the strain); FP32 its
rounding of the bond vectors, 1e-5.
"""
import numpy as np
import pytest

from lattice_math import family_offsets
from parity import say

pytestmark = pytest.mark.gpu

DX, C, VOL = 1.0e-3, 1.0e20, 1.0e-9


@pytest.fixture(scope="module", autouse=True)
def _lib():
    from paper_2105_04150_amd import _binding as B
    B.load()


def _lattice(dims):
    k, j, i = np.meshgrid(*[np.arange(d) for d in dims[::-1]], indexing="ij")
    return DX * np.stack([i.ravel(), j.ravel(), k.ravel()], axis=1).astype(np.float64)


def _direct(dims, m, u, volume):
    """Sum of c s V y / |y| over the offsets, on (z, y, x) grids."""
    shape = tuple(dims[::-1])
    U, V = u.reshape(shape + (3,)), volume.reshape(shape)
    F = np.zeros_like(U)
    for o in family_offsets(m):
        if any(abs(int(o[d])) >= dims[d] for d in range(3)):
            continue
        own = tuple(slice(max(0, -int(d)), s - max(0, int(d))) for d, s in zip(o[::-1], shape))
        oth = tuple(slice(max(0, int(d)), s - max(0, -int(d))) for d, s in zip(o[::-1], shape))
        xi = DX * o.astype(np.float64)
        eta = U[oth] - U[own]
        y = xi + eta
        r, L = np.sqrt((y * y).sum(-1)), np.sqrt((xi * xi).sum())
        # (r - L) / L without cancellation
        s = (eta * (xi + y)).sum(-1) / (L * (r + L))
        F[own] += (C * s * V[oth] / r)[..., None] * y
    return F.reshape(-1, 3)


@pytest.mark.parametrize("dims,m,strain,build,weights", [
    ((1, 1, 1), 3.015, 1e-3, "f64", False),
    ((2, 1, 1), 3.015, 1e-3, "f64", False),
    ((63, 1, 1), 3.015, 1e-3, "f64", False),
    ((4, 4, 4), 3.015, 1e-3, "f64", True),
    ((13, 5, 1), 3.015, 1e-3, "f64", True),
    ((43, 3, 1), 3.015, 1e-3, "f32", False),
    ((19, 9, 3), 3.015, 1e-3, "f64", True),
    ((33, 33, 30), 3.015, 1e-4, "f64", False),   # 511 slices: one a tile
    ((33, 32, 31), 3.015, 1e-4, "f64", True),    # 512: two
    ((61, 57, 57), 3.015, 1e-4, "f64", False),   # 3097: four
    ((59, 59, 57), 3.14, 2e-2, "f64", True),     # four, cut where they do not fit twice
    ((20, 17, 14), 8.015, 1e-3, "f64", True),    # several passes of records
    ((20, 17, 14), 8.015, 1e-3, "f32", False),
    ((12, 11, 10), 3.015, 1.9e-3, "f64", False),  # either side of the series' ranges
    ((12, 11, 10), 3.015, 2.2e-3, "f64", False),
    ((12, 11, 10), 3.015, 3.3e-2, "f64", True),
    ((12, 11, 10), 3.015, 6e-2, "f64", True),
    ((12, 11, 10), 3.015, -0.3, "f64", False),
    ((12, 11, 10), 3.015, 2e-2, "f32", True),
    ((12, 11, 10), 3.015, 0.3, "f32", False),
])
def test_force_of_tiles(dims, m, strain, build, weights):
    import paper_2105_04150_amd as pd
    rng = np.random.default_rng(7)
    x = _lattice(dims)
    n = len(x)
    # a stretch along x, a shear and a random part of the same size
    u = strain * (x * [1.0, -0.3, 0.2] + 0.3 * x[:, [1, 2, 0]] + 0.3 * DX * rng.uniform(-1, 1, x.shape))
    if build == "f32":
        u = u.astype(np.float32).astype(np.float64)
    vol = VOL * (rng.uniform(0.5, 1.5, n) if weights else np.ones(n))
    sim = pd.Simulation(0, pd.PD_FP32 if build == "f32" else pd.PD_FP64)
    sim.set_mapping("staged", 2)
    sim.build_family(x, m * DX)
    sim.set_integrator("euler_cromer", 1.0e-9)
    sim.set_material(2400.0, C, 10.0, 0.0, VOL, vol if weights else None)
    sim.set_state(u=u)
    got = sim.force()
    sim.close()
    want = _direct(dims, m, u, vol)
    top = np.abs(want).max()
    if n == 1:
        assert not got.any()
        return
    tol = 1e-5 if build == "f32" else 1e-12 + 4 * 2.0 ** -52 / abs(strain)
    err = np.abs(got - want).max() / top
    say(f"[tiles] {dims} m {m} strain {strain} {build}: {err:.2e} (tolerance {tol:.1e})")
    assert err <= tol


@pytest.mark.parametrize("build", ["f64", "f32"])
def test_overflowing_squares_stay_apart(build):
    """One node so far away that its bonds' squares overflow: the rest of its tile is untouched
    by the non-finite sums, the general form is taken for its wavefront."""
    import paper_2105_04150_amd as pd
    dims = (9, 8, 7)
    x = _lattice(dims)
    u = 1e-3 * x
    far = 250
    u[far] = 1e160 if build == "f64" else 1e22
    sim = pd.Simulation(0, pd.PD_FP32 if build == "f32" else pd.PD_FP64)
    sim.set_mapping("staged")
    sim.build_family(x, 3.015 * DX)
    sim.set_integrator("euler_cromer", 1.0e-9)
    sim.set_material(2400.0, C, 10.0, 0.0, VOL)
    sim.set_state(u=u)
    got = sim.force()
    sim.close()
    with np.errstate(all="ignore"):
        want = _direct(dims, 3.015, u.astype(np.float32).astype(np.float64) if build == "f32" else u,
                       VOL * np.ones(len(x)))
    near = np.zeros(len(x), bool)
    near[far] = True
    near |= (np.abs(x - x[far]) <= 3.015 * DX).all(1)
    tol = 1e-5 if build == "f32" else 1e-12 + 4 * 2.0 ** -52 / 1e-3
    assert np.abs(got[~near] - want[~near]).max() <= tol * np.abs(want[~near]).max()
