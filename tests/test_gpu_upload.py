"""Bodies as they reach the device: boundaries between them, records in more
than one chunk, bodies added after steps, several scenes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(n, z0, rng):
    k = int(np.ceil(np.sqrt(n / 16)))
    i = np.arange(n)
    pos = np.stack([i % k, (i // k) % k, i // (k * k)], 1) * 3e-3 + [0, 0, z0]
    return pos + 1e-5 * rng.uniform(-1, 1, pos.shape)


@pytest.mark.parametrize("counts", [(1,), (1, 1, 1), (262143,), (262144, 1), (5, 262150, 70)])
def test_added_bodies_come_back(counts):
    from paper_2301_00611_amd import dem
    rng = np.random.default_rng(sum(counts))
    s = dem.Scene(gravity=(0, 0, 0), damping=0.0)
    m = [s.add_material(2600.0, 1e7, 0.3, 0.5), s.add_material(1800.0, 1e7, 0.3, 0.5)]
    want = {k: [] for k in ("pos", "vel", "angvel")}
    ids, z = [], 0.1
    for c in counts:
        s.add_wall(2, -1.0, 1, m[0])
        pos, v, w = _lattice(c, z, rng), rng.uniform(-1, 1, (c, 3)), rng.uniform(-1, 1, (c, 3))
        z = pos[:, 2].max() + 5e-3
        first = s.add_spheres(pos, np.full(c, 1e-3), vel=v, angvel=w, mat=rng.integers(0, 2, c).astype(np.int32),
                              blocked=(63 * (np.arange(c) % 2)).astype(np.uint8))
        ids.append(np.arange(c) + first)
        for k, x in zip(want, (pos, v, w)):
            want[k].append(x)
    s.add_wall(0, -1.0, 1, m[0])
    s.set_dt(1e-7)
    ids, want = np.concatenate(ids), {k: np.concatenate(x) for k, x in want.items()}
    s.step(0)
    st = s.get_state()
    for k in want:
        assert np.array_equal(st[k][ids], want[k]), k
    assert np.array_equal(st["ori"][ids], np.tile([1.0, 0, 0, 0], (len(ids), 1)))
    s.step(1)
    # free flight, a blocked body at the velocity it was given
    assert np.abs(s.get_state()["pos"][ids] - want["pos"] - 1e-7 * want["vel"]).max() <= 1e-15
    s.close()


def test_bodies_added_to_a_running_batch():
    from paper_2301_00611_amd import dem
    rng = np.random.default_rng(2)
    b = dem.Batch([dem.make_params(dt=1e-6, gravity=(0, 0, 0), damping=0.0) for _ in range(3)])
    pos, vel, ids = [[] for _ in range(3)], [[] for _ in range(3)], [[] for _ in range(3)]
    z = 0.1
    for r in range(3):
        for i in range(3):
            s = b.scene(i)
            if r == 0:
                s.add_material(2600.0, 1e7, 0.3, 0.5)
            if r != 1:
                s.add_wall(2, -1.0 - i, 1, 0)
            c = 3 + 4 * i + r
            p, v = _lattice(c, z, rng), rng.uniform(-1, 1, (c, 3))
            first = s.add_spheres(p, np.full(c, 1e-3), vel=v, default_mat=0)
            pos[i].append(p - v * 1e-6 * 2 * r), vel[i].append(v), ids[i].append(np.arange(c) + first)
        z += 0.1
        b.step(2)
    for i in range(3):
        p, v, k = (np.concatenate(x[i]) for x in (pos, vel, ids))
        st = b.scene(i).get_state()
        assert np.array_equal(st["vel"][k], v)
        assert np.abs(st["pos"][k] - p - 6e-6 * v).max() <= 1e-15
    b.close()
