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


def _pull(x, peak):
    rng = np.random.default_rng(4)
    u = np.zeros_like(x)
    u[:, 0] = peak * x[:, 0] ** 2 / (2.0 * x[:, 0].max())
    return u + 0.05 * peak * DX * rng.uniform(-1, 1, x.shape)


@pytest.mark.parametrize("dims,m,scheme", [
    ((61, 60, 57), 3.015, "velocity_verlet"),   # four slices a tile, cut in two
    ((37, 33, 29), 4.015, "euler_cromer"),      # two, cut in one
    ((14, 13, 12), 8.015, "velocity_verlet"),   # several phases, in other places
])
def test_new_volumes_and_laws_keep_the_state(dims, m, scheme):
    """Steps with breaking bonds, then volumes and a damage law set in the middle of the run
    (and taken away again): the state stays, bit for bit, and the run goes on as on the sliced
    mapping, whose layout never changes."""
    import paper_2105_04150_amd as pd
    out = []
    for mapping in ("staged", "sliced"):
        with pd.Simulation() as sim:
            x = _problem(sim, dims, m, scheme=scheme, c=1.0e19 * (3.0 / m) ** 4)
            if mapping == "sliced":
                sim.set_mapping("sliced")
            vol = DX ** 3 * np.random.default_rng(1).uniform(0.8, 1.2, len(x))
            sim.set_state(u=_pull(x, 1.2e-3))
            sim.step(4)

            def state():
                return sim.u(), sim.v(), sim.a(), sim.broken(), sim.break_steps(), np.array(sim.step_count)
            before = state()
            assert before[3].any()
            sim.set_material(2400.0, 1.0e19 * (3.0 / m) ** 4, 1.0e-3, 0.0, 1.0, vol)
            sim.set_damage_law(0, (8.0e-4, 2.0e-3), (1.0, 0.0))
            sim.force()  # runs a kernel: the tiles are made anew here
            for a, b in zip(before, state()):
                assert np.array_equal(a, b)
            sim.step(4)
            soft = sim.max_stretch()
            middle = sim.u()
            sim.set_material(2400.0, 1.0e19 * (3.0 / m) ** 4, 1.0e-3, 0.0, DX ** 3)
            sim.force()
            assert np.array_equal(sim.max_stretch(), soft) and np.array_equal(sim.u(), middle)
            sim.clear_damage_laws()
            sim.step(4)
            out.append((sim.u(), sim.broken(), soft))
    (us, bs, ss), (ug, bg, sg) = out
    say(f"[relayout] {dims} m {m}: broken {bg.mean():.3f}, softened {(sg > 0).mean():.3f}")
    assert np.array_equal(bs, bg) and np.array_equal(ss > 0, sg > 0)
    assert np.abs(us - ug).max() <= 1e-12 * np.abs(ug).max()


def test_reverse_pass_over_several_phases():
    """Horizon of eight spacings: a forward run with breaking bonds and its reverse pass, against
    the sliced mapping."""
    import paper_2105_04150_amd as pd
    dims, m = (13, 12, 11), 8.015
    out = []
    for mapping in ("staged", "sliced"):
        with pd.Simulation() as sim:
            x = _problem(sim, dims, m, c=2.0e17)
            if mapping == "sliced":
                sim.set_mapping("sliced")
            sim.set_state(u=_pull(x, 1.2e-3))
            rec = sim.adj_forward(6, 3)
            assert sim.broken().any()
            dl = 1.0e-5 * np.random.default_rng(2).standard_normal((20, 3))
            out.append(sim.adj_backward(np.arange(20) * 37, dl, rec) + (sim.broken(),))
    (ks, as_, bs), (kg, ag, bg) = out
    assert np.array_equal(bs, bg)
    assert np.abs(ks - kg).max() <= 1e-9 * np.abs(kg).max()
    assert abs(as_ - ag) <= 1e-9 * max(abs(ag), 1e-300)


@pytest.mark.parametrize("mapping", ["staged", "sliced"])
def test_calls_before_the_layout_exists(mapping):
    """Readouts and setters right after the family, in any order."""
    import paper_2105_04150_amd as pd
    x = _lattice((9, 8, 7))
    n = len(x)

    def made():
        sim = pd.Simulation()
        sim.set_mapping(mapping)
        sim.build_family(x, 3.015 * DX)
        return sim

    with made() as sim:
        info = sim.info()
        assert info["n_nodes"] == n and info["n_nodes_dev"] >= n and info["n_slots_dev"] >= info["n_slots"]
    with made() as sim:
        sim.sync()
        assert not sim.u().any() and not sim.broken().any() and not sim.force().any()
    with made() as sim:
        sim.set_damage_law(0, (1.0e-3, 2.0e-3), (1.0, 0.0))
        sim.set_no_fail(np.arange(10))
        nnz = sim.family()[0][-1]
        assert not sim.max_stretch().any()
        sim.set_mapping("staged" if mapping == "sliced" else "sliced")
        assert sim.info()["n_slots"] == nnz
        sim.clear_damage_laws()
        sim.step(1)
        sim.sync()
    with made() as sim:
        with pytest.raises(pd.PdmiError):
            sim.resultant(np.array([n]))
        with pytest.raises(pd.PdmiError):
            sim.set_max_stretch(np.zeros(sim.family()[0][-1]))
        sim.set_step(5)
        assert sim.step_count == 5
        sim.step(2)
        sim.sync()
        assert sim.step_count == 7 and not sim.u().any()
