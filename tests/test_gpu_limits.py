"""A broad-phase run that cannot be finished is refused with an error; the
scene stays as it was and can be used again."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(n):
    i = np.arange(n)
    k = int(np.ceil(n ** (1 / 3)))
    return (np.stack([i % k, i // k % k, i // k ** 2], 1) + 0.5) * 1.99e-3


@pytest.mark.parametrize("n", [50_000, 70_000])
def test_too_many_candidates(n):
    """Every sphere beside every other: n^2 row entries, more than an index
    holds, and at 70,000 more than 32 bits count."""
    from paper_2301_00611_amd import dem
    x = _lattice(n)
    s, twin = dem.Scene(gravity=(0, 0, -9.81)), dem.Scene(gravity=(0, 0, -9.81))
    for g in (s, twin):
        m = g.add_material(2600.0, 1e7, 0.3, 0.5)
        g.add_wall(2, 0.0, 0, m)
        g.add_spheres(x, np.full(n, 1e-3), default_mat=m)
        g.set_dt(1e-6)
        g.step(20)
    a = s.get_state()
    assert len(s.get_contacts()) > n
    pos = a["pos"].copy()
    pos[1:] *= 1e-3
    s.set_state(pos=pos)
    for call in (lambda: s.step(0), lambda: s.step(3), lambda: s.get_stress(1e-3), lambda: s.unbalanced_force()):
        with pytest.raises(dem.DemError) as e:
            call()
        assert e.value.code == dem.DEM_ENOMEM
    with pytest.raises(dem.DemError):
        s.get_stress_noalloc(1e-3)
    now = s.get_state()
    assert np.array_equal(now["pos"], pos) and np.array_equal(now["vel"], a["vel"])
    assert not now["force"].any() and len(s.get_contacts()) == 0
    assert s.stats()["iter"] == 20 and s.stats()["max_overlap_ratio"] == 0.0
    for g in (s, twin):
        g.set_state(**{k: a[k] for k in ("pos", "vel", "angvel", "ori")})
        g.step(40)
    b, c = s.get_state(), twin.get_state()
    for k in b:
        assert np.array_equal(b[k][1:], c[k][1:]), k
    assert np.array_equal(s.get_contacts(), twin.get_contacts())
    s.close()
    twin.close()
