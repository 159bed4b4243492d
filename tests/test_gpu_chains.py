"""Steps launched in chains, one behind another: however a run is cut into
calls and chains, with broad-phase runs falling anywhere between, the state is
the same bit for bit; a failure inside a chain is reported and can be mended."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bed(verlet, n=600):
    from paper_2301_00611_amd import dem
    rng = np.random.default_rng(4)
    s = dem.Scene(gravity=(0, 0, -9.81), damping=0.2, verlet_dist=verlet)
    m = s.add_material(2600.0, 1e7, 0.3, 0.5)
    s.add_wall(2, 0.0, 0, m)
    k = int(np.ceil(n ** (1 / 3)))
    pos = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n] * 2.02e-3 + 1.1e-3
    s.add_spheres(pos, rng.uniform(0.9e-3, 1e-3, n), vel=0.3 * rng.uniform(-1, 1, pos.shape), default_mat=m)
    s.set_dt(4e-6)
    return s


@pytest.mark.parametrize("verlet", [-0.01, -0.05, -0.5])
def test_chains_and_calls_do_not_change_results(verlet):
    ref = None
    for chunk, calls in ((32, [400]), (32, [1] * 400), (2, [400]), (8, [399, 1]), (64, [150, 3, 247]), (4096, [400])):
        s = _bed(verlet)
        s.set_tuning(chunk=chunk)
        for c in calls:
            s.step(c)
        out = s.get_state(), s.get_contacts(), s.stats()
        s.close()
        assert out[2]["iter"] == 400
        ref = ref or out
        if verlet > -0.1:
            assert ref[2]["rebuilds"] > 5
        assert out[2]["rebuilds"] == ref[2]["rebuilds"]
        for k in ref[0]:
            assert np.array_equal(out[0][k], ref[0][k]), (chunk, k)
        assert np.array_equal(out[1], ref[1])


@pytest.mark.parametrize("verlet", [-0.5, 0.05])
@pytest.mark.parametrize("at", [5, 40, 100, 170, 300])
def test_failure_in_a_chain(at, verlet):
    """Two soft spheres that pass through one another from step `at` on: the
    run ends with an error, the count of steps is that of the steps done (a
    third sphere in free flight tells), and a mended state goes on."""
    from paper_2301_00611_amd import dem
    r, v, dt = 1e-3, 50.0, 1e-6
    s = dem.Scene(gravity=(0, 0, 0), damping=0.0, verlet_dist=verlet)
    m = s.add_material(2600.0, 1e4, 0.3, 0.5)
    x0 = np.array([[0, 0, 0], [2 * r + at * v * dt, 0, 0], [0, 0.2, 0]])
    v0 = np.array([[v, 0, 0], [0, 0, 0], [0, 0, 8.0]])
    s.add_spheres(x0, np.full(3, r), vel=v0, default_mat=m)
    s.set_dt(dt)
    with pytest.raises(dem.DemError):
        s.step(1000)
    it = s.stats()["iter"]
    assert at < it < at + 32 * 2 + 64
    assert abs(s.get_state()["pos"][2, 2] - 8.0 * dt * it) <= 1e-12
    s.set_state(pos=x0 + [[0, 0, 0], [0.1, 0, 0], [0, 0, 0]], vel=v0)
    s.step(100)
    assert s.stats()["iter"] == it + 100
    assert abs(s.get_state()["pos"][2, 2] - 8.0 * dt * 100) <= 1e-12
    s.close()
