"""GPU tests of the split density and force kernels (the neighbours of 64 atoms
dealt to the waves of a workgroup; systems of at most 131,072 slots): parity
with the oracle where the deal has remainders, and bitwise agreement with the
one-thread kernels, which larger systems use, and with their staged form (own
records in LDS; one species in FP64 beyond 262,144 slots)."""
import numpy as np
import pytest

from paper_1107_2619_amd import inputs
from tests.gpu_helpers import TOL, announce, energy_error, force_error

pytestmark = pytest.mark.gpu
SPLIT_SLOTS = 2 * 1024 * 64
DIRECT_SLOTS = 4 * 1024 * 64


@pytest.fixture(scope="module")
def md():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_2619_amd import md as _md

    return _md


def _batch(parts):
    """One batch of one-replica systems of the same potential."""
    p0 = parts[0]
    cat = lambda k: np.concatenate([getattr(p, k) for p in parts])  # noqa: E731
    return inputs.System(
        name="batch", pos=cat("pos"), vel=cat("vel"), species=cat("species"), rigid=cat("rigid"),
        atom_offset=np.concatenate([[0], np.cumsum([p.n_atoms for p in parts])]).astype(np.int64), box=cat("box"),
        origin=cat("origin"), periodic=cat("periodic"), rigid_velocity=cat("rigid_velocity"), potential=p0.potential,
        dt_fs=p0.dt_fs, skin=p0.skin, rebuild_every=p0.rebuild_every, steps=p0.steps, temperature=cat("temperature"),
        max_neighbours=p0.max_neighbours)


def _take(s, n):
    """The first n atoms of a one-replica system in the same box."""
    s.pos, s.vel, s.species, s.rigid = (a[:n].copy() for a in (s.pos, s.vel, s.species, s.rigid))
    s.atom_offset = np.array([0, n], np.int64)
    return s


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("skin,cap,potential", [(0.05, 31, "fe_fs"), (0.4, 33, "fe_fs"), (0.9, 61, "fec_eam"),
                                                (1.6, 90, "fe_fs")])
def test_split_rounds_against_oracle(md, orc, precision, skin, cap, potential):
    """Lists of about 26 to 65 entries (one, two and three rounds of eight groups
    of four) at capacities that are no multiple of a group, 127 atoms (a ragged
    last wavefront): forces and per-atom energies at the parity tolerances."""
    announce(f"split rounds {precision} skin {skin} {potential}")
    s = _take(inputs.bcc_fe(4, seed=91, displace=0.06, skin=skin, potential=potential), 127)
    s.max_neighbours = cap
    if potential == "fec_eam":
        s.species[::5] = 1
    ref = orc.forces(s.pos, s.species, s.box[0], s.periodic[0], orc.Potential(s.potential))
    sim = md.Simulation(s, precision=precision)
    sim.eam_forces()
    en = sim.energy()
    assert 16 < sim.get_option(md.MD_OPT_MAX_COUNT) <= cap
    assert force_error(sim.forces(), ref.f) <= TOL[precision]["force"]
    assert energy_error(sim.atom_energies(), ref.e_atom) <= TOL[precision]["energy"]
    assert abs(en.pe[0] - ref.pe) <= TOL[precision]["energy"] * abs(ref.pe)


@pytest.mark.parametrize("precision,potential,slots", [
    ("fp64", "fe_fs", SPLIT_SLOTS), ("mixed", "fe_fs", SPLIT_SLOTS), ("fp64", "fec_eam", SPLIT_SLOTS),
    ("mixed", "fec_eam", SPLIT_SLOTS), ("fp64", "fe_fs", DIRECT_SLOTS)])
def test_forms_agree_bitwise(md, precision, potential, slots):
    """The same replicas (128, 127, 64, 65 and 1 atoms) in a batch that fills the
    largest size of one form and in one 64 slots larger: forces, energies, virial and
    12 steps with energies are bitwise equal, so a replica does not depend on
    the size of its batch."""
    announce(f"forms at {slots} slots {precision} {potential}")
    parts = []
    for k, n in enumerate((128, 127, 64, 65, 1)):
        p = _take(inputs.bcc_fe(4, seed=92 + k, pot_seed=92, displace=0.06, skin=0.8, potential=potential), n)
        if potential == "fec_eam":
            p.species[::7] = 1
        p.max_neighbours = 64
        parts.append(p)
    used = sum((p.n_atoms + 63) // 64 for p in parts)
    fill = _take(inputs.bcc_fe(4, seed=99, pot_seed=92, skin=0.8, potential=potential), 64)
    fill.max_neighbours = 64
    n = sum(p.n_atoms for p in parts)
    got = []
    for extra in (0, 1):
        s = _batch(parts + [fill] * (slots // 64 - used + extra))
        assert sum((int(v) + 63) // 64 * 64 for v in np.diff(s.atom_offset)) == slots + 64 * extra
        sim = md.Simulation(s, precision=precision, energy_ring=8)
        sim.set_option(md.MD_OPT_ENERGY_EVERY, 2)
        sim.eam_forces()
        e0 = sim.energy()
        f0, ea = sim.forces()[:n], sim.atom_energies()[:n]
        sim.step(12)
        e1 = sim.energy()
        hist = np.array([np.concatenate([h.pe[:5], h.ke[:5], h.virial[:5].ravel()]) for h in sim.energy_history()])
        got.append((f0, ea, e0.pe[:5], e0.virial[:5], sim.positions()[:n], sim.velocities()[:n], sim.forces()[:n],
                    e1.pe[:5], e1.ke[:5], e1.virial[:5], hist))
    for a, b in zip(*got):
        assert np.array_equal(a, b)
