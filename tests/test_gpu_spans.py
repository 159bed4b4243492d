"""Force sums over spans of row entries: rows that end at, just before and
just after a span and the rounds that share a long row, and the history
records read by quads in a scene of many bodies."""
import numpy as np
import pytest

from gpu_helpers import body_force_errors, keyset, twin
from test_gpu_rows import _fcc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("around", [1, 23, 24, 25, 28, 47, 48, 49, 64, 88, 89, 96])
def test_large_sphere_among_small(around, precision, tol):
    """Nine large spheres, each touched by `around` small ones that do not
    touch one another: rows of exactly `around` entries next to rows of one."""
    from paper_2301_00611_amd.scenes import Material, Scene
    rng = np.random.default_rng(around)
    r, R = 1e-3, 6.5e-3
    k = np.arange(around) + 0.5
    z, phi = 1.0 - 2.0 * k / around, np.pi * (1.0 + np.sqrt(5.0)) * k
    ring = np.stack([np.sqrt(1 - z * z) * np.cos(phi), np.sqrt(1 - z * z) * np.sin(phi), z], 1)
    pos, radius = [], []
    for i in range(9):
        c = np.array([i % 3, i // 3, 0.0]) * 20e-3
        dist = R + r * (1.0 - 4e-3 * rng.uniform(0.2, 1.0, (around, 1)))
        pos += [c[None], c + ring * dist]
        radius += [[R], np.full(around, r)]
    pos, radius = np.concatenate(pos), np.concatenate(radius)
    spec = Scene(pos=pos, radius=radius, material=Material(2600.0, 1e7, 0.3, 0.5), gravity=(0, 0, 0), damping=0.3)
    g, o, dt = twin(spec, precision=precision, vel=0.05 * rng.uniform(-1, 1, pos.shape),
                    angvel=2.0 * rng.uniform(-1, 1, pos.shape))
    g.step(1)
    o.step(1)
    co = o.get_contacts()
    assert len(co) == 9 * around and keyset(g.get_contacts()) == keyset(co)
    ef, _ = body_force_errors(g.get_state(), o.get_state(), co)
    assert ef.max() <= tol
    g.step(5)
    o.step(5)
    vg, vo = g.get_state()["vel"], o.get_state()["vel"]
    assert np.linalg.norm(vg - vo, axis=1).max() <= tol * np.linalg.norm(vo, axis=1).max()


@pytest.mark.parametrize("block", [256, 1024])
@pytest.mark.parametrize("verlet", [-0.5, -1.1])
def test_many_bodies_are_copies_of_few(verlet, block):
    """A periodic cube of 500 spheres and one made of 9 x 9 x 10 copies of it
    (405,000): every copy moves as the original does.  A position near 0.14 m
    is off by up to 1.4e-17 m, an overlap (some 4e-7 m) by 1e-10 of itself,
    more where it is small; 1e-8 of the largest velocity leaves room."""
    from paper_2301_00611_amd import dem
    from paper_2301_00611_amd.scenes import random_velocities
    pos, radius, side = _fcc(5, 1e-3, 3, 0)
    n = len(radius)
    v, w = random_velocities(n, 0.02, 8)
    out = []
    for m in ((1, 1, 1), (9, 9, 10)):
        shift = np.stack(np.meshgrid(*[np.arange(k) for k in m], indexing="ij"), -1).reshape(-1, 1, 3) * side
        c = len(shift)
        s = dem.Scene(periodic=True, hsize=np.diag(np.array(m) * side), velgrad=np.zeros((3, 3)), damping=0.3,
                      gravity=(0, 0, 0), verlet_dist=verlet)
        s.set_tuning(block_integrate=block)
        mat = s.add_material(2600.0, 1e8, 0.3, 0.5)
        s.add_spheres((pos[None] + shift).reshape(-1, 3), np.tile(radius, c), vel=np.tile(v, (c, 1)),
                      angvel=np.tile(w * 0.05, (c, 1)), default_mat=mat)
        s.set_dt(1e-6)
        s.step(6)
        st = s.get_state()
        out.append([st[k].reshape(c, n, 3) for k in ("vel", "angvel", "force", "torque")])
        s.close()
    for few, many in zip(*out):
        scale = np.linalg.norm(few, axis=2).max()
        assert scale > 0 and np.linalg.norm(many - few, axis=2).max() <= 1e-8 * scale
