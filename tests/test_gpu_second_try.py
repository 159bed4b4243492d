"""A broad-phase run is sized by the one before with an eighth to spare.  When
its entries, or its pairs alone, are more, the run is done again by its own
counts: against a scene whose run is sized by its own counts at once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
R, N, CLUSTER = 1e-3, 2000, 343


def _at(what):
    """Places of the spheres that move: a loose lattice, a dense one, or a
    loose layer just above the planes."""
    i = np.arange(N)
    if what == "layer":
        return np.stack([i % 45 * 4e-3, i // 45 * 4e-3, np.full(N, 1.3 * R)], 1) + [0.1, 0, 0]
    s = 4e-3 if what == "loose" else 2.01e-3
    return (np.stack([i % 13, i // 13 % 13, i // 169], 1) + 0.5) * s + [0.1, 0.0, 0.02]


def _scene(precision, first):
    """A cluster of touching spheres, which keeps its contacts' history, and
    the others; twelve planes below."""
    from paper_2301_00611_amd import dem
    rng = np.random.default_rng(5)
    s = dem.Scene(gravity=(0, 0, -9.81), damping=0.2, precision=precision)
    m = s.add_material(2600.0, 1e6, 0.3, 0.5)
    for k in range(12):
        s.add_wall(2, -1e-6 * k, 1, m)
    j = np.arange(CLUSTER)
    c = (np.stack([j % 7, j // 7 % 7, j // 49], 1) + 0.5) * 1.98e-3 + [0, 0, 0.02]
    v = np.zeros((CLUSTER + N, 3))
    v[:CLUSTER] = rng.uniform(-0.2, 0.2, (CLUSTER, 3))
    s.add_spheres(np.concatenate([c, _at(first)]), np.full(CLUSTER + N, R), vel=v,
                  angvel=200 * v, default_mat=m)
    s.set_dt(1e-6)
    return s


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("first,then", [("loose", "dense"), ("dense", "layer"), ("dense", "loose")])
def test_run_done_again(first, then, precision):
    out = []
    for own_counts in (False, True):
        s = _scene(precision, first)
        s.step(40)
        before = s.stats()["n_candidates"]
        if own_counts:
            s.set_tuning(verlet_factor=0.5)  # (as it was: the counts of the run before are not used)
        pos = s.get_state()["pos"]
        pos[12 + CLUSTER:] = _at(then)
        s.set_state(pos=pos)
        s.step(0)
        st = s.stats()
        if then == "dense":   # entries: about two per pair
            assert st["n_candidates"] > 2 * before + 1024
        if then == "layer":   # one entry per pair now: fewer entries, more pairs
            walls = 12 * N
            assert before * 9 / 8 + 1024 < walls <= st["n_candidates"] < 2 * before
        state, contacts = [s.get_state()], [s.get_contacts()]
        for _ in range(2):
            s.step(30)
            state.append(s.get_state())
            contacts.append(s.get_contacts())
        out.append((st["n_candidates"], state, contacts))
        s.close()
    assert out[0][0] == out[1][0]
    assert (np.linalg.norm(out[0][2][0]["fs"], axis=1) > 0).sum() > CLUSTER
    for a, b in zip(out[0][1], out[1][1]):
        for k in a:
            first_id = 12 if k == "force" else 0
            assert np.array_equal(a[k][first_id:], b[k][first_id:]), k
    for a, b in zip(out[0][2], out[1][2]):
        assert np.array_equal(a, b)
