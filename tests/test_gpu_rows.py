"""Force sums of rows past the entries a lane walks alone, through both ways
of finishing them: every row of the wave a little longer (the lanes walk on)
and a few rows much longer (the wave shares them)."""
import numpy as np
import pytest

from gpu_helpers import body_force_errors, contact_errors, keyset, twin

pytestmark = pytest.mark.gpu


def _fcc(cells, r, seed, large):
    """Face-centred lattice of nearly touching spheres in a periodic cube;
    `large` of them (spread over the ids) grown to three times the radius,
    with the spheres inside them taken out."""
    rng = np.random.default_rng(seed)
    a = 2.0 * np.sqrt(2.0) * r * (1.0 + 5e-5)
    base = np.array([[0, 0, 0], [.5, .5, 0], [.5, 0, .5], [0, .5, .5]]) + 0.25
    nodes = np.stack(np.meshgrid(*[np.arange(cells)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    pos = ((nodes + base).reshape(-1, 3)) * a
    side = cells * a
    radius = np.full(len(pos), r)
    keep = np.ones(len(pos), bool)
    for i in np.linspace(0, len(pos) - 1, large, dtype=int) if large else ():
        if not keep[i]:
            continue
        d = pos - pos[i]
        d -= side * np.round(d / side)
        near = np.linalg.norm(d, axis=1) < 4.0 * r * (1 - 1e-9)
        if (radius[near & keep] > r).any():
            continue
        keep &= ~near
        keep[i] = True
        radius[i] = 3.0 * r
    pos, radius = pos[keep], radius[keep]
    n = len(radius)
    radius = radius * (1.0 + 4e-4 * rng.uniform(-1, 1, n))
    return pos + 4e-4 * r * rng.uniform(-1, 1, (n, 3)), radius, side


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("verlet,large", [(-0.2, 0), (-0.5, 0), (-0.5, 3), (-1.1, 5)])
def test_rows_past_the_solo_walk(verlet, large, precision, tol):
    from paper_2301_00611_amd.scenes import Material, Scene, random_velocities
    cells = 9 if large else 5  # three coarse cells across
    pos, radius, side = _fcc(cells, 1e-3, 3, large)
    n = len(radius)
    v, w = random_velocities(n, 0.02, 8)
    spec = Scene(pos=pos, radius=radius, material=Material(2600.0, 1e8, 0.3, 0.5), gravity=(0, 0, 0), damping=0.3)
    g, o, dt = twin(spec, precision=precision, periodic=True, hsize=np.eye(3) * side, velgrad=np.zeros((3, 3)),
                    vel=v, angvel=w * 0.05, verlet_dist=verlet)
    g.step(1)
    o.step(1)
    # every second neighbour is a candidate from 0.42 r on: rows of 18 and more
    assert 2 * g.stats()["n_candidates"] >= (12 if verlet > -0.4 else 16) * n
    cg, co = g.get_contacts(), o.get_contacts()
    assert len(co) > n and keyset(cg) == keyset(co)
    assert contact_errors(cg, co)["f"].max() <= tol
    ef, _ = body_force_errors(g.get_state(), o.get_state(), co)
    assert ef.max() <= tol
    g.step(6)
    o.step(6)
    assert keyset(g.get_contacts()) == keyset(o.get_contacts())
    ds = np.linalg.norm(g.get_state()["vel"] - o.get_state()["vel"], axis=1).max()
    assert ds <= tol * np.linalg.norm(o.get_state()["vel"], axis=1).max()
