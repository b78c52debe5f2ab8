"""Calls that change the mapping of a problem that is on the staged one."""
import numpy as np
import pytest

import pd_inputs as pi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("build", ["f64", "f32"])
def test_autotune_keeps_what_the_staged_mapping_does_not_use(build):
    """Staged lanes and node order change nothing, so trying them out cannot choose them: what
    was given is reported back, and the state is as before."""
    import paper_2105_04150_amd as pd
    w = pi.workload("block10", dims=(12, 10, 9), steps=50)
    with pd.Simulation(0, pd.PD_FP32 if build == "f32" else pd.PD_FP64) as sim:
        sim.set_mapping("staged", 4)
        sim.build_family(w.coords, w.horizon, "auto")
        pd.apply_workload(sim, w)
        sim.set_integrator("euler_cromer", w.dt)
        if build == "f64":
            sim.set_model("state_based", 1.0e10, 6.0e9)  # staged mapping only
        sim.step(20)
        u = sim.u()
        for _ in range(2):
            sim.autotune(3)
            info = sim.info()
            assert info["mapping"] == pd.PD_MAP_STAGED and info["waves_per_slice"] == 4
            assert info["order"] == pd.PD_ORDER_NATURAL
        assert np.array_equal(sim.u(), u) and sim.step_count == 20


def test_staged_lanes_change_nothing():
    import paper_2105_04150_amd as pd
    w = pi.workload("block10", dims=(12, 10, 9), steps=50)
    out = []
    for lanes in (1, 2, 4):
        with pd.Simulation() as sim:
            sim.set_mapping("staged", 1)
            sim.build_family(w.coords, w.horizon)
            pd.apply_workload(sim, w)
            sim.set_integrator("velocity_verlet", w.dt)
            sim.step(21)
            steps = sim.break_steps()
            sim.set_mapping("staged", lanes)
            assert sim.info()["waves_per_slice"] == lanes
            assert np.array_equal(sim.break_steps(), steps)
            sim.step(21)
            out.append(sim.u())
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
