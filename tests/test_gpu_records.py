"""Reports of the last step's forces whichever record they are read from: the
history (linear law) or the force records (visco-elastic law), when a material
of the other law is added between steps and when a broad-phase run renews the
pair list."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
SIDE = 0.015
VOLUME = SIDE ** 3


def _scene(law, precision, n=300, seed=6):
    from paper_2301_00611_amd import dem
    rng = np.random.default_rng(seed)
    r = rng.uniform(0.7e-3, 1.2e-3, n)
    i = np.arange(n)
    x = (np.stack([i % 7, i // 7 % 7, i // 49], 1) + 0.5) * 2e-3
    s = dem.Scene(gravity=(0, 0, -9.81), damping=0.2, precision=precision)
    m = s.add_viscel_material(2600.0, 2e-4, 0.6, 0.7, 0.5) if law else s.add_material(2600.0, 1e7, 0.3, 0.5)
    for axis in range(3):
        s.add_wall(axis, 0.0, 0, m)
    s.add_spheres(x, r, vel=rng.uniform(-0.3, 0.3, (n, 3)), angvel=rng.uniform(-30, 30, (n, 3)), default_mat=m)
    s.set_dt(1e-6)
    return s


def _reports(s):
    st = s.get_state()
    return {"force": st["force"][3:], "torque": st["torque"][3:], "contacts": s.get_contacts(),
            "walls": st["force"][:3], "stress": s.get_stress(VOLUME), "unbalanced": s.unbalanced_force()}


def _same(a, b):
    f = np.linalg.norm(a["contacts"]["fn"] + a["contacts"]["fs"], axis=1)
    assert (a["contacts"]["is_wall"] == 0).sum() > 50 and a["walls"].any()
    for k in ("force", "torque", "contacts"):
        assert np.array_equal(a[k], b[k]), k
    # summed over pairs or blocks in another order
    assert np.abs(a["walls"] - b["walls"]).max() <= 1e-12 * f.sum()
    assert np.abs(a["stress"] - b["stress"]).max() <= 1e-12 * f.sum() * 3e-3 / VOLUME
    assert abs(a["unbalanced"] - b["unbalanced"]) <= 1e-12 * a["unbalanced"]


def _consistent(s, precision):
    """The resultants are the sums of the contacts' forces."""
    st, c = s.get_state(), s.get_contacts()
    want = np.zeros_like(st["force"])
    np.add.at(want, c["id2"], c["fn"] + c["fs"])
    np.add.at(want, c["id1"], -(c["fn"] + c["fs"]))
    # FP64 (or FP32) sums of what the contact list holds apart
    scale = np.linalg.norm(c["fn"] + c["fs"], axis=1).max()
    assert np.abs(st["force"] - want).max() <= (1e-12 if precision == 0 else 1e-5) * scale


@pytest.mark.parametrize("precision", [0, 1])
def test_material_of_the_other_law_added_between_steps(precision):
    s = _scene(0, precision)
    s.step(60)
    _consistent(s, precision)
    before = _reports(s)
    s.add_viscel_material(2600.0, 2e-4, 0.6, 0.7, 0.5)  # no body's
    _same(before, _reports(s))
    runs = s.stats()["rebuilds"]
    s.set_tuning(chunk=32)  # asks for a run
    s.step(0)
    assert s.stats()["rebuilds"] == runs + 1
    _same(before, _reports(s))
    s.step(3)
    _consistent(s, precision)
    after = _reports(s)
    s.set_tuning(chunk=32)
    s.step(0)
    _same(after, _reports(s))
    s.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_viscoelastic_forces_through_a_run(precision):
    s = _scene(1, precision)
    s.step(60)
    _consistent(s, precision)
    before = _reports(s)
    runs = s.stats()["rebuilds"]
    s.set_tuning(chunk=32)
    s.step(0)
    assert s.stats()["rebuilds"] == runs + 1
    _same(before, _reports(s))
    s.add_spheres([[0.1, 0.1, 0.1]], [1e-3], default_mat=0)
    stress = s.get_stress(VOLUME)
    f = np.linalg.norm(before["contacts"]["fn"] + before["contacts"]["fs"], axis=1).sum()
    assert np.abs(stress - before["stress"]).max() <= 1e-12 * f * 3e-3 / VOLUME
    assert np.array_equal(s.get_state()["force"][3:-1], before["force"])
    s.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_only_the_viscoelastic_law_keeps_records(precision):
    """48 (FP32-mixed: 24) bytes per pair of each list."""
    import torch
    from paper_2301_00611_amd import dem
    n = 100_000
    i = np.arange(n)
    x = (np.stack([i % 47, i // 47 % 47, i // 47 ** 2], 1) + 0.5) * 2.001e-3
    used = []
    for law in (0, 1, 0):  # (the first warms the device up)
        s = dem.Scene(gravity=(0, 0, -9.81), precision=precision)
        m = s.add_viscel_material(2600.0, 2e-4, 0.6, 0.7, 0.5) if law else s.add_material(2600.0, 1e7, 0.3, 0.5)
        s.add_spheres(x, np.full(n, 1e-3), default_mat=m)
        s.set_dt(1e-6)
        free = torch.cuda.mem_get_info()[0]
        s.step(2)
        s.set_state(pos=x)
        s.step(2)
        pairs = s.stats()["n_candidates"]
        used.append(free - torch.cuda.mem_get_info()[0])
        s.close()
    assert pairs > 2 * n
    assert used[1] - used[2] >= 2 * pairs * (48 if precision == 0 else 24)
