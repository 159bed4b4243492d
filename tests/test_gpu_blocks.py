"""A scene's own choice of threads per block moves no result, and the tuned
values are reported and kept as set."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(n, tuning, precision=0):
    from paper_2301_00611_amd import dem
    rng = np.random.default_rng(n)
    k = int(np.ceil(n ** (1 / 3)))
    pos = np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n] * 1.99e-3 + 1e-3
    pos += 5e-6 * rng.uniform(-1, 1, pos.shape)
    s = dem.Scene(gravity=(0, 0, -9.81), damping=0.2, precision=precision)
    m = s.add_material(2600.0, 1e7, 0.3, 0.5)
    s.add_wall(2, 0.0, 0, m)
    s.add_spheres(pos, np.full(n, 1e-3), vel=0.05 * rng.uniform(-1, 1, pos.shape), default_mat=m)
    s.set_dt(2e-6)
    if tuning:
        s.set_tuning(**tuning)
    kept = s.get_tuning()
    s.step(40)
    out = s.get_state(), s.get_contacts(), kept, s.get_tuning()
    s.close()
    return out


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [40, 16384, 33000, 65536])
def test_blocks_do_not_change_results(n, precision):
    st0, c0, t0, t1 = _run(n, None, precision)
    assert t0["block_contact"] == t0["block_integrate"] == t1["block_contact"] == t1["block_integrate"] == 256
    for b in ({"block_contact": 512, "block_integrate": 64}, {"block_contact": 128, "block_integrate": 1024},
              {"chunk": 16}):
        st, c, t, _ = _run(n, b, precision)
        assert all(t[k] == v for k, v in b.items())
        for k in st0:
            assert np.array_equal(st[k], st0[k]), k
        assert np.array_equal(c, c0)
