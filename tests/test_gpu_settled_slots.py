"""Slots that the staged kernels settle one by one (softened, over the threshold, beyond the
series), against the sliced kernel on the same state: shares of more than 32 row pairs, blocks that
change level within a share, zones, and nodes whose bonds are all broken."""
import numpy as np
import pytest

from parity import say

pytestmark = pytest.mark.gpu

DX = 1.0e-3
LAW = ((2.3e-4, 2.42e-4, 1.45e-3), (1.0, 0.25, 0.0))


@pytest.fixture(scope="module", autouse=True)
def _lib():
    from paper_2105_04150_amd import _binding as B
    B.load()


def _lattice(dims):
    k, j, i = np.meshgrid(*[np.arange(d) for d in dims[::-1]], indexing="ij")
    return DX * np.stack([i.ravel(), j.ravel(), k.ravel()], axis=1).astype(np.float64)


def _state(dims, peak):
    """Stretch growing from zero at one end of x to `peak` at the other, and a random part."""
    rng = np.random.default_rng(11)
    x = _lattice(dims)
    u = np.zeros_like(x)
    u[:, 0] = peak * x[:, 0] ** 2 / (2.0 * x[:, 0].max())
    u += 0.1 * peak * DX * rng.uniform(-1, 1, x.shape)
    return x, u


def _run(mapping, x, u, m, law, zones, s0, steps, field):
    import paper_2105_04150_amd as pd
    with pd.Simulation(0, pd.PD_FP64) as sim:
        sim.set_mapping(mapping)
        sim.build_family(x, m * DX)
        sim.set_integrator("euler_cromer", 1.0e-8)
        sim.set_material(2400.0, 1.0e19, s0, 0.0, DX ** 3)
        if field:
            row_ptr, _ = sim.family()
            sim.set_bond_stiffness(1.0e19 * np.ones(row_ptr[-1]))
        if law:
            sim.set_damage_law(0, *LAW)
        if zones:
            sim.set_no_fail(np.nonzero(x[:, 1] < 1.5 * DX)[0])
        sim.set_state(u=u)
        f = [sim.force()]
        sim.step(steps)
        f.append(sim.force())
        return f, sim.u(), sim.broken().astype(bool), sim.max_stretch() if law else None


@pytest.mark.parametrize("dims,m", [((24, 7, 6), 3.015), ((14, 13, 12), 8.015)])
@pytest.mark.parametrize("law,zones,s0,peak,field", [
    (True, False, 1.0, 4.0e-4, False),
    (True, True, 1.0, 3.0e-3, False),
    (True, True, 1.0, 3.0e-3, True),
    (False, True, 5.0e-3, 2.0e-2, False),   # zone bonds far beyond the threshold
    (False, False, 0.2, 0.6, False),        # both series and the closed form, some break
    (False, False, 1.0e-3, 1.05e-3, True),
])
def test_settled_slots_match_the_sliced_kernel(dims, m, law, zones, s0, peak, field):
    x, u = _state(dims, peak)
    steps = 6
    a, b = (_run(k, x, u, m, law, zones, s0, steps, field) for k in ("staged", "sliced"))
    say(f"[settled] {dims} m {m} law {law} zones {zones}: broken {a[2].mean():.3f}"
        + (f" softened {(a[3] > 0).mean():.3f}" if law else ""))
    assert np.array_equal(a[2], b[2])
    # both kernels: the rounding of |y|^2 - |xi|^2, 4 units of 2^-52 over the smallest stretch that counts
    tol = 1e-13 + 8 * 2.0 ** -52 / min(peak, 2.3e-4)
    for fa, fb in zip(a[0], b[0]):
        assert np.abs(fa - fb).max() <= tol * np.abs(fb).max()
    assert np.abs(a[1] - b[1]).max() <= 1e-13 * np.abs(b[1]).max()
    if law:
        assert np.array_equal(a[3] > 0, b[3] > 0)
        assert np.abs(a[3] - b[3]).max() <= 1e-12


@pytest.mark.parametrize("build,far", [("f64", 1.0e99), ("f64", 1.0e120), ("f32", 1.0e18)])
def test_a_free_node_feels_nothing_wherever_it_is(build, far):
    """A node whose bonds are all broken has no force, however far it has gone."""
    import paper_2105_04150_amd as pd
    x = _lattice((9, 8, 7))
    n, free = len(x), 250
    with pd.Simulation(0, pd.PD_FP32 if build == "f32" else pd.PD_FP64) as sim:
        sim.set_mapping("staged")
        sim.build_family(x, 3.015 * DX)
        sim.set_integrator("euler_cromer", 1.0e-9)
        sim.set_material(2400.0, 1.0e20, 10.0, 0.0, DX ** 3)
        rp, col = sim.family()
        row = np.repeat(np.arange(n), np.diff(rp))
        u = 1e-3 * x
        u[free] = far
        sim.set_state(u=u, broken=((row == free) | (col == free)).astype(np.uint8))
        f = sim.force()
    assert not f[free].any()
    assert np.isfinite(f).all() and np.abs(f).max() > 0.0


@pytest.mark.parametrize("build,far", [("f64", 1.0e99), ("f64", 1.0e120), ("f32", 1.0e18)])
def test_a_free_node_has_no_dilation_wherever_it_is(build, far):
    """The same with the state-based model: neither force nor dilation, and none is passed on."""
    import paper_2105_04150_amd as pd
    x = _lattice((9, 8, 7))
    n, free = len(x), 250
    out = []
    for where in (far, 0.0):
        with pd.Simulation(0, pd.PD_FP32 if build == "f32" else pd.PD_FP64) as sim:
            sim.set_mapping("staged")
            sim.build_family(x, 3.015 * DX)
            sim.set_integrator("euler_cromer", 1.0e-9)
            sim.set_material(2400.0, 1.0, 10.0, 0.0, DX ** 3)
            sim.set_model("state_based", 1.4e10, 1.0e10)
            rp, col = sim.family()
            row = np.repeat(np.arange(n), np.diff(rp))
            u = 1e-3 * x
            u[free] = where
            sim.set_state(u=u, broken=((row == free) | (col == free)).astype(np.uint8))
            out.append((sim.dilation(), sim.force()))
    for t, f in out:
        assert t[free] == 0.0 and not f[free].any()
        assert np.abs(t).max() > 0.0 and np.abs(f).max() > 0.0
    # the rest is untouched by where the free node is (its wavefront may take another series)
    eps = 1e-5 if build == "f32" else 1e-12
    assert np.abs(out[0][0] - out[1][0]).max() <= eps * np.abs(out[1][0]).max()
    assert np.abs(out[0][1] - out[1][1]).max() <= eps * np.abs(out[1][1]).max()


@pytest.mark.parametrize("part", [0.002, 0.02, 0.1, 0.5, 1.0])
@pytest.mark.parametrize("build", ["f64", "f32"])
def test_any_number_of_softened_slots(part, build):
    """From a few softened slots a wavefront, shared out among its lanes, to all of them: the
    force of the state, against a direct sum over the bonds."""
    import paper_2105_04150_amd as pd
    dims = (17, 11, 9)
    x, u = _state(dims, 2.0e-4)
    u = u.astype(np.float32).astype(np.float64)
    n = len(x)
    (s1, s2, s3), (_, r2, _) = LAW
    with pd.Simulation(0, pd.PD_FP32 if build == "f32" else pd.PD_FP64) as sim:
        sim.set_mapping("staged")
        sim.build_family(x, 3.015 * DX)
        sim.set_integrator("euler_cromer", 1.0e-8)
        sim.set_material(2400.0, 1.0e19, 1.0, 0.0, DX ** 3)
        sim.set_damage_law(0, *LAW)
        rp, col = sim.family()
        row = np.repeat(np.arange(n), np.diff(rp))
        rng = np.random.default_rng(6)
        key = np.minimum(row, col) * n + np.maximum(row, col)
        draw = rng.random(n * n)[key]
        level = rng.uniform(s1 * 1.001, s3 * 0.99, n * n)[key]
        sm = np.where(draw < part, level, 0.0)
        sim.set_state(u=u)
        sim.set_max_stretch(sm)
        got = sim.force()
        assert np.array_equal(sim.max_stretch(), sm)
    xi, eta = x[col] - x[row], u[col] - u[row]
    y = xi + eta
    r, L = np.sqrt((y * y).sum(1)), np.sqrt((xi * xi).sum(1))
    s = (eta * (xi + y)).sum(1) / (L * (r + L))
    rho = np.where(sm < s2, 1.0 + (r2 - 1.0) * (sm - s1) / (s2 - s1), r2 * (s3 - sm) / (s3 - s2))
    w = np.where(sm > 0, s1 * rho / np.where(sm > 0, sm, 1.0), 1.0)
    f = (1.0e19 * DX ** 3 * w * s / r)[:, None] * y
    want = np.stack([np.bincount(row, f[:, d], minlength=n) for d in range(3)], axis=1)
    # the rounding of |y|^2 - |xi|^2 over the stretch, and of rho on its steep first branch (below 60 times)
    tol = 1e-5 if build == "f32" else 4 * 2.0 ** -52 / 2.0e-4 + 60 * 8 * 2.0 ** -52
    assert np.abs(got - want).max() <= tol * np.abs(want).max()
