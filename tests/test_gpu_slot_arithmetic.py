"""Arithmetic of one slot of the staged FP64 kernels, seen through single bonds.

Bonds of length L = 1 + k/1024 stretched by e = j/4096 have exact squares, so the force
density c V e has no rounding in its stretch and what is left is the error of the kernel's
series and reciprocal root.  Its bound: 9/8 e^2 of the refined estimate, e <= 2^-22 by the
instruction's specification, 6.4e-14, and a dozen roundings of 2^-53.
"""
import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

TOL = 1.125 * 2.0 ** -44 + 12 * 2.0 ** -53


@pytest.fixture(scope="module", autouse=True)
def _lib():
    from paper_2105_04150_amd import _binding as B
    B.load()


def _force(x, pairs, u, model="pmb", s0=10.0, build="f64", zones=None, broken=None):
    """Force densities of a problem with the given bonds; c V = 1."""
    import paper_2105_04150_amd as pd
    n = len(x)
    both = np.concatenate([pairs, pairs[:, ::-1]])
    both = both[np.lexsort((both[:, 1], both[:, 0]))]
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(np.bincount(both[:, 0], minlength=n))
    with pd.Simulation(0, pd.PD_FP32 if build == "f32" else pd.PD_FP64) as sim:
        sim.set_mapping("staged")
        sim.set_family(x, rp, both[:, 1].astype(np.int32))
        sim.set_integrator("euler_cromer", 1.0e-9)
        sim.set_material(1.0, 1.0, s0, 0.0, 1.0)
        if model == "state_based":
            sim.set_model("state_based", 1.0, 0.5)
        if zones is not None:
            sim.set_no_fail(zones)
        if broken is not None:
            sim.set_state(u=u, broken=broken(both).astype(np.uint8))
        else:
            sim.set_state(u=u)
        return sim.force()


@pytest.mark.parametrize("j", [1, 4, 7, -7, 14, -14, 60, 130, 400, -400])
def test_single_bonds(j):
    k = np.arange(1024)
    length = 1.0 + k / 1024.0
    x = np.zeros((2048, 3))
    x[0::2, 0] = 16.0 * (k % 32)
    x[0::2, 1] = 16.0 * (k // 32)
    x[1::2] = x[0::2]
    x[1::2, 2] += length
    u = np.zeros_like(x)
    u[1::2, 2] = length * (j / 4096.0)
    f = _force(x, np.stack([2 * k, 2 * k + 1], axis=1), u)
    assert not f[:, :2].any()
    err = np.abs(f[0::2, 2] / (j / 4096.0) - 1.0).max()
    say(f"[slot] stretch {j}/4096: {err:.2e} (tolerance {TOL:.1e})")
    assert err <= TOL
    assert np.array_equal(f[0::2, 2], -f[1::2, 2])


@pytest.mark.parametrize("model,build", [("pmb", "f64"), ("pmb", "f32"), ("state_based", "f64")])
@pytest.mark.parametrize("big", [2.0e-2, 0.3])
def test_both_slots_of_a_bond_agree(model, build, big):
    """Bonds from one slice to the next carry opposite forces bit for bit, also where one of the
    two slices holds a bond that its block's short (or long) series does not cover."""
    rng = np.random.default_rng(5)
    n = 64
    x = np.zeros((2 * n, 3))
    x[:, 1] = np.tile(np.arange(n) % 8, 2) + 0.01 * rng.uniform(-1, 1, 2 * n)
    x[:, 2] = np.tile(np.arange(n) // 8, 2) + 0.01 * rng.uniform(-1, 1, 2 * n)
    x[n:, 0] = 30.0 + 0.01 * rng.uniform(-1, 1, n)
    u = 1.0e-3 * rng.uniform(-1, 1, x.shape) * [30.0, 1.0, 1.0]
    u = u.astype(np.float32).astype(np.float64)
    u[n + 1, 1] = u[n, 1] + big
    cross = np.stack([np.arange(2, n), n + np.arange(2, n)], axis=1)
    pairs = np.concatenate([[[0, 1]], cross, [[n, n + 1]]])
    f = _force(x, pairs, u, model, build=build)
    assert np.abs(f[2:n]).min() > 0.0
    assert np.array_equal(f[2:n], -f[n + 2:])
