"""The candidate list whichever way the broad phase searches: exactly the
pairs closer than r_i + r_j + 2 Delta L, counted here by brute force, for
loose and dense scenes of wide and narrow size ratios (one grid level or
two), and the same contacts after several runs as the oracle's."""
import numpy as np
import pytest

from gpu_helpers import keyset, twin

pytestmark = pytest.mark.gpu


def _count(pos, radius, dl, side=None):
    n = 0
    for i in range(len(radius) - 1):
        d = pos[i + 1:] - pos[i]
        if side is not None:
            d -= side * np.round(d / side)
        n += int((np.einsum("ij,ij->i", d, d) < (radius[i] + radius[i + 1:] + 2 * dl) ** 2).sum())
    return n


@pytest.mark.parametrize("n", [1, 2, 65, 1300])
@pytest.mark.parametrize("spacing", [1.0, 1.3, 4.0])
@pytest.mark.parametrize("sizes", ["equal", "uniform", "few large", "many large"])
def test_candidates_open(sizes, spacing, n):
    from paper_2301_00611_amd.scenes import Material, Scene
    rng = np.random.default_rng(7)
    r = {"equal": np.full(n, 1e-3), "uniform": rng.uniform(0.5e-3, 1.5e-3, n),
         "few large": np.where(np.arange(n) % 100 == 0, 4e-3, 1e-3),
         "many large": np.where(np.arange(n) % 4 == 0, 0.5e-3, 2e-3)}[sizes]
    k = int(np.ceil(n ** (1 / 3)))
    s = 2 * r.max() * spacing * (0.55 if sizes == "few large" else 1.0)
    i = np.arange(n)
    pos = (np.stack([i % k, i // k % k, i // k ** 2], 1) + 0.5) * s + rng.uniform(-0.2, 0.2, (n, 3)) * s
    spec = Scene(pos=pos, radius=r, material=Material(2600.0, 1e7, 0.3, 0.5), gravity=(0, 0, 0))
    g, o, dt = twin(spec)
    g.step(0)
    assert g.stats()["n_candidates"] == _count(pos, r, 0.5 * r.min())
    g.close()


@pytest.mark.parametrize("sizes,cells", [("equal", 9), ("uniform", 9), ("few large", 14)])
@pytest.mark.parametrize("spacing", [1.02, 1.6])
def test_candidates_periodic(sizes, cells, spacing):
    from paper_2301_00611_amd.scenes import Material, Scene
    rng = np.random.default_rng(5)
    n = cells ** 3
    r = {"equal": np.full(n, 1e-3), "uniform": rng.uniform(0.5e-3, 1.5e-3, n),
         "few large": np.where(np.arange(n) % 300 == 0, 3e-3, 1e-3)}[sizes]
    i = np.arange(n)
    s = 2e-3 * spacing
    pos = (np.stack([i % cells, i // cells % cells, i // cells ** 2], 1) + 0.5) * s + rng.uniform(-0.1, 0.1, (n, 3)) * s
    side = cells * s
    pos += side * rng.integers(-2, 3, (n, 3))  # periods away from the cell
    spec = Scene(pos=pos, radius=r, material=Material(2600.0, 1e7, 0.3, 0.5), gravity=(0, 0, 0))
    g, o, dt = twin(spec, periodic=True, hsize=np.eye(3) * side, velgrad=np.zeros((3, 3)))
    g.step(0)
    assert g.stats()["n_candidates"] == _count(pos, r, 0.5 * r.min(), side)
    g.close()


def test_contacts_through_runs_on_one_level():
    """A loose scene of size ratio 3 thrown at its floor: contacts and
    positions as the oracle's after several broad-phase runs."""
    from paper_2301_00611_amd.scenes import grid_column
    spec = grid_column(n=400, width=0.025, seed=3)
    v = np.tile([0.3, 0.1, -1.5], (400, 1))
    g, o, dt = twin(spec, vel=v)
    for _ in range(4):
        g.step(300)
        o.step(300)
        assert keyset(g.get_contacts()) == keyset(o.get_contacts())
    assert g.stats()["rebuilds"] > 3 and len(o.get_contacts()) > 0
    assert np.abs(g.get_state()["pos"] - o.get_state()["pos"]).max() <= 1e-9 * 0.025
