"""The choice between one and two grid levels follows how crowded it is around
the bodies, not how far the outermost ones are: a sphere that leaves an open
bed does not make the search in the bed an order of magnitude longer."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
RS, RL = 0.5e-3, 2e-3


def _bed(n, far):
    """n small spheres in a dense lattice, a few large ones on top; with
    `far` one more, which stretches the bounding box to `far` times the
    bed's."""
    k = int(round(n ** (1 / 3)))
    i = np.arange(n)
    side = k * 1.03e-3
    x = (np.stack([i % k, i // k % k, i // k ** 2], 1) + 0.5) * 1.03e-3
    j = np.arange(9)
    big = np.stack([(j % 3 + 0.5) * side / 3, (j // 3 + 0.5) * side / 3, np.full(9, side + RL)], 1)
    x = np.concatenate([x, big, [[0.5 * side, 0.5 * side, (far or 1) * side]]])
    return x, np.concatenate([np.full(n, RS), np.full(9, RL), [RS]])


def _run_ms(step, timed, again):
    """The time of a broad-phase run on unchanged bodies, the least of five."""
    timed.set_timing(True)
    best = np.inf
    for _ in range(5):
        again()
        step(0)
        best = min(best, timed.get_timing("rebuild")[0])
    return best


def _count(x, r):
    from scipy.spatial import cKDTree
    small = cKDTree(x[r == RS])
    d = 0.5 * RS * 2
    n = len(small.query_pairs(2 * RS + d))
    big = x[r == RL]
    n += sum(len(q) for q in small.query_ball_point(big, RS + RL + d))
    return n + len(cKDTree(big).query_pairs(2 * RL + d))


@pytest.mark.parametrize("far", [40, 70, 1000])
def test_a_far_sphere_leaves_the_search_short(far):
    from paper_2301_00611_amd import dem
    ms = []
    for f in (0, far):
        x, r = _bed(185_193, f)
        s = dem.Scene(gravity=(0, 0, 0))
        m = s.add_material(2600.0, 1e7, 0.3, 0.5)
        s.add_spheres(x, r, default_mat=m)
        s.set_dt(1e-6)
        s.step(0)
        assert s.stats()["n_candidates"] == _count(x, r)
        ms.append(_run_ms(s.step, s, lambda: s.set_state(pos=x)))
        assert s.stats()["n_candidates"] == _count(x, r)
        s.close()
    print("ms per run without and with it:", ms)
    # cells grow with the box (at most 4 per body): at 70 times the volume a
    # sphere tests 5.4 times as many others as without the far one (about twice
    # the time), on one level 27 times as many (about six times); at 1,000 times
    # the cells are larger than the plain ones either way
    if far <= 70:
        assert ms[1] < 4 * ms[0]


def test_scenes_of_a_batch_choose_for_themselves():
    from paper_2301_00611_amd import dem
    xs = [_bed(8000, 0), _bed(27_000, 40), _bed(8000, 0)]
    xs[2] = (xs[2][0] * 40.0, xs[2][1])  # loose
    b = dem.Batch([dem.make_params(dt=1e-6) for _ in range(3)])
    v = [b.scene(i) for i in range(3)]
    m = v[0].add_material(2600.0, 1e7, 0.3, 0.5)
    for i in range(3):
        v[i].add_spheres(*xs[i], default_mat=m)
    want = sum(_count(*x) for x in xs)
    for _ in range(3):
        b.step(0)
        assert b.stats()["n_candidates"] == want
        v[1].set_state(pos=xs[1][0])
    b.close()
