"""A failed step ends the call no later than its own chain of steps: whatever
was launched behind that chain does not run."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _scene(at, verlet):
    """A sphere that goes through another from step `at` on."""
    from paper_2301_00611_amd import dem
    r, v, dt = 1e-3, 50.0, 1e-6
    s = dem.Scene(gravity=(0, 0, 0), damping=0.0, verlet_dist=verlet)
    m = s.add_material(2600.0, 1e4, 0.3, 0.5)
    s.add_spheres([[0, 0, 0], [2 * r + at * v * dt, 0, 0], [0, 0.2, 0]], np.full(3, r),
                  vel=[[v, 0, 0], [0, 0, 0], [0, 0, 8.0]], default_mat=m)
    s.set_dt(dt)
    return s


@pytest.mark.parametrize("verlet", [-0.5, 0.05])
@pytest.mark.parametrize("chunk", [8, 32, 64])
@pytest.mark.parametrize("at", [5, 170, 300])
def test_failure_ends_its_own_chain(at, chunk, verlet):
    from paper_2301_00611_amd import dem
    one = _scene(at, verlet)
    with pytest.raises(dem.DemError) as e:
        for _ in range(1000):
            one.step(1)
    failed = one.stats()["iter"]
    assert at < failed and e.value.code == dem.DEM_EUNSTABLE
    one.close()

    s = _scene(at, verlet)
    s.set_tuning(chunk=chunk)
    with pytest.raises(dem.DemError) as e:
        s.step(2000)
    st = s.stats()
    assert e.value.code == dem.DEM_EUNSTABLE
    assert failed <= st["iter"] <= failed + chunk - 1
    assert abs(s.get_state()["pos"][2, 2] - 8e-6 * st["iter"]) <= 1e-12
    # it goes on when told to, without a broad-phase run that no step asked for
    with pytest.raises(dem.DemError):
        s.step(1)
    assert s.stats()["iter"] == st["iter"] + 1
    if verlet > 0:
        assert s.stats()["rebuilds"] == st["rebuilds"]
    s.close()
