"""GPU test of the list build's candidate pruning where single precision is
coarse: a potential whose cutoff is 41,000 length units (the 4.1 A one scaled by
10,000), pairs at that distance less 1e-10 of it.  Rounded to single precision,
half of them lie beyond the radius by more than 0.001."""
import numpy as np
import pytest

from paper_1107_2619_amd import inputs
from tests.gpu_helpers import announce

pytestmark = pytest.mark.gpu
SCALE = 1e4


@pytest.fixture(scope="module")
def md():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_2619_amd import md as _md

    return _md


@pytest.mark.parametrize("nbr_mode", ["full", "half"])
def test_pairs_at_a_large_radius(md, nbr_mode):
    announce(f"pruning at a radius of 41,000, {nbr_mode} list")
    base = inputs.bcc_fe(4, seed=1)
    pot = dict(base.potential)
    for k in ("pair_r", "dens_R"):
        pot[k] = np.asarray(pot[k]) * SCALE
    for k in ("pair_a", "dens_A"):
        pot[k] = np.asarray(pot[k]) / SCALE**3
    rc = float(np.max(pot["pair_r"]))
    n = 2000
    rng = np.random.default_rng(7)
    u = rng.normal(size=(n, 3))
    u[:, 0] = np.abs(u[:, 0]) + 0.5
    u /= np.linalg.norm(u, axis=1)[:, None]
    first = np.tile(np.array([1.99, 1.99, 1.99]) * rc, (n, 1))  # the others lie in the next cells along x
    pos = np.stack([first, first + u * (rc * (1 - 1e-10))], 1).reshape(-1, 3)
    s = inputs.System(
        name="far pairs", pos=pos, vel=np.zeros_like(pos), species=np.zeros(2 * n, np.uint8),
        rigid=np.zeros(2 * n, np.uint8), atom_offset=np.arange(0, 2 * n + 1, 2, dtype=np.int64),
        box=np.full((n, 3), 4.0 * rc), origin=np.zeros((n, 3)), periodic=np.zeros((n, 3), np.uint8),
        rigid_velocity=np.zeros((n, 3)), potential=pot, dt_fs=1.0, skin=0.0, rebuild_every=10, steps=0,
        temperature=np.zeros(n), max_neighbours=4,
    )
    d = pos[1::2] - pos[0::2]
    assert np.all(np.einsum("ij,ij->i", d, d) < rc * rc)
    sim = md.Simulation(s, precision="fp64", nbr_mode=nbr_mode)
    sim.build_neighbours()
    counts, _ = sim.neighbours()
    assert counts.reshape(n, 2).sum() == (2 * n if nbr_mode == "full" else n)
