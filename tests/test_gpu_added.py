"""Reports between steps when bodies were added since the last one: what is
said about the last step's contacts stays what it was, whatever places the
bodies have in memory by then."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
SIDE = 0.03
VOLUME = SIDE ** 3


def _polydisperse(n=300, seed=6):
    """A lattice of spheres of which about a third overlap their neighbours."""
    rng = np.random.default_rng(seed)
    r = rng.uniform(0.7e-3, 1.2e-3, n)
    i = np.arange(n)
    x = (np.stack([i % 7, i // 7 % 7, i // 49], 1) + 0.5) * 2e-3
    return x, r, rng.uniform(-0.3, 0.3, (n, 3)), rng.uniform(-30, 30, (n, 3))


def _fill(view, n=300, seed=6):
    x, r, v, w = _polydisperse(n, seed)
    m = [view.add_material(2600.0, 1e7, 0.3, 0.5), view.add_material(2000.0, 4e7, 0.2, 0.3)]
    for axis in range(3):
        view.add_wall(axis, 0.0, 0, m[0])
    view.add_spheres(x, r, vel=v, angvel=w, mat=np.arange(n) % 2, default_mat=m[0])
    view.set_dt(1e-6)


def _far(n):
    """Spheres out of everyone's way, smaller than all the others."""
    i = np.arange(n)
    return np.stack([i % 10, i // 10 % 10, i // 100], 1) * 1.5e-3 + 0.05, np.full(n, 0.5e-3)


def _reports(s):
    return {"stress": s.get_stress(VOLUME), "dt": s.stiffness_dt(0.5), "largest": s.unbalanced_force(use_max=True)}


def _same(a, b, contacts):
    # sums of the same terms in another order
    scale = (np.linalg.norm(contacts["fn"] + contacts["fs"], axis=1) * 3e-3).sum() / VOLUME
    assert np.abs(a["stress"] - b["stress"]).max() <= 1e-12 * scale
    assert a["dt"] == b["dt"]
    assert abs(a["largest"] - b["largest"]) <= 1e-12 * a["largest"]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("more", [1, 400])
def test_reports_after_bodies_were_added(more, precision):
    from paper_2301_00611_amd import dem
    s = dem.Scene(gravity=(0, 0, -9.81), damping=0.2, precision=precision)
    _fill(s)
    s.step(60)
    before, state, contacts = _reports(s), s.get_state(), s.get_contacts()
    nb = len(state["pos"])
    assert (contacts["is_wall"] == 0).sum() > 5
    x, r = _far(more)
    s.add_spheres(x, r, default_mat=0)
    # of bodies not yet seen by a step nothing is known, and nothing is said
    assert len(s.get_contacts()) == 0 and not s.get_state()["force"].any()
    _same(before, _reports(s), contacts)
    for _ in range(2):
        now = s.get_state()
        for k in state:
            # (a boundary's reaction is added in the order of the pairs, which a run renews)
            assert np.array_equal(now[k][3 if k == "force" else 0:nb], state[k][3 if k == "force" else 0:]), k
        f = np.linalg.norm(contacts["fn"] + contacts["fs"], axis=1).sum()
        assert np.abs(now["force"][:3] - state["force"][:3]).max() <= 1e-12 * f
        assert not now["force"][nb:].any()
        assert np.array_equal(s.get_contacts(), contacts)
        assert np.array_equal(s.get_stress_noalloc(VOLUME), s.get_stress_noalloc(VOLUME))
        s.step(0)
    _same(before, _reports(s), contacts)
    s.close()


def test_timestepper_after_bodies_were_added():
    from paper_2301_00611_amd import dem
    s = dem.Scene(gravity=(0, 0, -9.81), damping=0.2)
    _fill(s)
    s.step(60)
    want = s.stiffness_dt(0.5)
    t = s.stats()["time"]
    s.add_spheres(*_far(400), default_mat=0)
    s.set_stiffness_timestepper(0.5, 1)
    s.step(1)
    assert abs(s.stats()["time"] - t - want) <= 1e-12 * want
    s.close()


def test_other_scenes_of_a_batch_keep_their_contacts():
    """Bodies added to one scene of a batch, then another's history replaced:
    the third goes on as if nothing had happened."""
    from paper_2301_00611_amd import dem
    out = []
    for touch in (False, True):
        b = dem.Batch([dem.make_params(dt=1e-6, gravity=(0, 0, -9.81)) for _ in range(3)])
        v = [b.scene(i) for i in range(3)]
        for i in range(3):
            _fill(v[i], n=150 + i, seed=3 + i)
        b.step(60)
        c = v[2].get_contacts()
        assert len(c) > 5
        if touch:
            stress, h = v[2].get_stress(VOLUME), v[1].get_history()
            v[0].add_spheres(*_far(300), default_mat=0)
            scale = (np.linalg.norm(c["fn"] + c["fs"], axis=1) * 3e-3).sum() / VOLUME
            assert np.abs(v[2].get_stress(VOLUME) - stress).max() <= 1e-12 * scale
            v[0].add_spheres(_far(300)[0] + 0.1, _far(300)[1], default_mat=0)
            v[1].set_history(h["id1"], h["id2"], h["fs"], h["nprev"], h["cell"])
        b.step(50)
        out.append((v[2].get_state(), v[2].get_contacts()))
        b.close()
    for k in out[0][0]:
        assert np.array_equal(out[0][0][k][3:], out[1][0][k][3:]), k
    assert np.array_equal(out[0][1], out[1][1])
