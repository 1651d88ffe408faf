"""GPU tests of the forms of the density and force passes where the choice
changes: the split form (eight waves deal the neighbours of 64 atoms), one thread
per atom, and one thread per atom with the workgroup's records staged in LDS.  The
forms add the same terms in the same order, so a replica is bitwise the same on
either side of every limit.  In wavefronts of 64 slots per SIMD (65,536 slots) the
split form ends at 2 for plain passes and, for the force passes that also sum
energies or the virial, at 1.25 with one species and at 1.75 (FP64) or 2 (mixed)
with several; FP64 with one species stages beyond 4."""
import numpy as np
import pytest

from paper_1107_2619_amd import inputs
from tests.gpu_helpers import TOL, announce, energy_error, force_error
from tests.test_gpu_split import _batch, _take

pytestmark = pytest.mark.gpu
PER_SIMD = 64 * 1024
KB_EV = 8.617343e-5


@pytest.fixture(scope="module")
def md():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_2619_amd import md as _md

    return _md


def _parts(cells, sizes, potential, skin, cap):
    parts = []
    for k, n in enumerate((*sizes, 64)):  # the last one fills the batch
        p = _take(inputs.bcc_fe(cells, seed=92 + k, pot_seed=92, displace=0.06, temperature=300.0, skin=skin,
                                rebuild_every=2, potential=potential), n)
        if potential == "fec_eam":
            p.species[::7] = 1
        p.max_neighbours = cap
        parts.append(p)
    return parts[:-1], parts[-1]


def _filled(parts, fill, slots):
    """The replicas in a batch of so many slots."""
    used = sum((p.n_atoms + 63) // 64 for p in parts)
    s = _batch(parts + [fill] * (slots // 64 - used))
    assert sum((int(v) + 63) // 64 * 64 for v in np.diff(s.atom_offset)) == slots
    return s


def _integrator(mode, s):
    n = np.diff(s.atom_offset).astype(float)
    kw = {}
    if mode == "nvt":
        kw.update(nh_temperature=np.full(len(n), 400.0), nh_mass=np.maximum(3 * n - 3, 1) * KB_EV * 400.0 * 1e4)
    if mode in ("npt", "full_npt"):  # a box heavy enough for the nearly empty ones
        kw.update(pr_pressure_gpa=np.full(len(n), 2.0), pr_mass=1e4 * n)
    if mode == "full_npt":
        kw.update(box_matrix=np.stack([np.diag(b) for b in s.box]))
    if mode == "gear":
        kw.update(integrator="gear3")
    return kw


def _run(md, s, n, r, mode="nve", precision="fp64", evaluator=None, chunk=None, steps=12):
    """Everything the first n atoms (r replicas) show of one evaluation and a run."""
    kw = _integrator(mode, s)
    if mode == "nve":
        kw["energy_ring"] = 8
    sim = md.Simulation(s, precision=precision, **kw)
    if mode == "nve":
        sim.set_option(md.MD_OPT_ENERGY_EVERY, 2)
    if evaluator is not None:
        sim.set_option(md.MD_OPT_EVALUATOR, evaluator)
    if chunk is not None:
        sim.set_option(md.MD_OPT_NEIGHBOUR_CHUNK, chunk)
    sim.eam_forces()
    out = [sim.forces()[:n], sim.atom_energies()[:n]]
    energies = [sim.energy()]
    sim.eam_forces(want_energy=False)
    out.append(sim.forces()[:n])
    sim.step(steps)
    energies.append(sim.energy())
    if mode == "nve":
        energies += sim.energy_history()  # of the evaluation at step 0 too
        assert len(energies) == 3 + steps // 2
    out += [sim.positions()[:n], sim.velocities()[:n], sim.forces()[:n]]
    for e in energies:
        out += [e.pe[:r], e.ke[:r], e.virial[:r], e.nh_pi[:r], e.nh_energy[:r], e.box[:r], e.pr_energy[:r], e.h[:r]]
    assert all(np.all(np.isfinite(v)) for v in out)
    return out


def _both_sides(md, parts, fill, slots, **kw):
    n = sum(p.n_atoms for p in parts)
    one, other = (_run(md, _filled(parts, fill, slots + extra), n, len(parts), **kw) for extra in (0, 64))
    for a, b in zip(one, other):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("precision,potential,waves", [
    ("fp64", "fe_fs", 1.25), ("mixed", "fe_fs", 1.25), ("fp64", "fec_eam", 1.75), ("mixed", "fec_eam", 2)])
@pytest.mark.parametrize("mode", ["nve", "npt", "full_npt"])
def test_passes_with_sums(md, precision, potential, waves, mode):
    """The limits of the passes that sum energies (every second step) or the virial."""
    announce(f"passes with sums, {mode} {precision} {potential} at {waves}")
    parts, fill = _parts(5, (250, 127, 64, 65, 1), potential, 0.3, 64)
    _both_sides(md, parts, fill, int(waves * PER_SIMD), mode=mode, precision=precision)


@pytest.mark.parametrize("mode", ["nvt", "npt", "full_npt", "gear"])
@pytest.mark.parametrize("precision,potential,waves", [
    ("fp64", "fe_fs", 2), ("mixed", "fe_fs", 2), ("fp64", "fec_eam", 2), ("fp64", "fe_fs", 4), ("mixed", "fe_fs", 4)])
def test_integrators(md, precision, potential, waves, mode):
    """The sums a force pass takes per wavefront for the thermostat and the barostats
    (whose padding lanes stay to the end), and the Gear steps, in every form."""
    announce(f"{mode} {precision} {potential} at {waves}")
    parts, fill = _parts(5, (250, 127, 64, 65, 1), potential, 0.3, 64)
    _both_sides(md, parts, fill, waves * PER_SIMD, mode=mode, precision=precision)


@pytest.mark.parametrize("waves", [2, 4])
def test_knot_sums(md, waves):
    """The term-by-term evaluator, which needs no tables beside the staged records."""
    announce(f"knot sums at {waves}")
    parts, fill = _parts(5, (250, 127, 64, 65, 1), "fe_fs", 0.3, 64)
    _both_sides(md, parts, fill, waves * PER_SIMD, evaluator=1)


@pytest.mark.parametrize("precision,potential,waves", [
    ("fp64", "fe_fs", 2), ("mixed", "fe_fs", 2), ("fp64", "fec_eam", 2), ("mixed", "fec_eam", 2), ("fp64", "fe_fs", 4)])
def test_neighbour_chunk_beyond_the_split_form(md, precision, potential, waves):
    """Two, four or eight neighbour records in flight where they take effect: one
    thread per atom, from the caches and staged, with energies on every second step;
    rows whose lengths leave every remainder of a chunk."""
    announce(f"neighbour chunk {precision} {potential} at {waves}")
    parts, fill = _parts(5, (250, 127, 64, 65, 1), potential, 0.3, 64)
    s = _filled(parts, fill, int(waves * PER_SIMD) + 64)
    n = sum(p.n_atoms for p in parts)
    counts = md.Simulation(s, precision=precision)
    counts.build_neighbours()
    assert set(counts.neighbours()[0][:n] % 8) == set(range(8))
    runs = [_run(md, s, n, len(parts), precision=precision, chunk=c) for c in (4, 2, 8)]
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("potential,skin,cap,rounds,inner_rounds", [
    ("fe_fs", 1.6, 90, 2, 2), ("fe_fs", 2.8, 133, 4, 4), ("fec_eam", 2.0, 101, 3, 2)])
def test_rounds_of_the_split_form(md, orc, precision, potential, skin, cap, rounds, inner_rounds):
    """Rows of two to four rounds of eight groups of four, the inner entries (the
    density pass) of two or four: forces and per-atom energies against the oracle."""
    announce(f"split rounds {precision} {potential} skin {skin}")
    s = _take(inputs.bcc_fe(6, seed=95, displace=0.06, skin=skin, potential=potential), 431)
    s.max_neighbours = cap
    if potential == "fec_eam":
        s.species[::5] = 1
    d = s.pos[:, None] - s.pos[None]
    d -= s.box[0] * np.rint(d / s.box[0])
    r = np.sqrt(np.sum(d * d, 2)) + 1e9 * np.eye(s.n_atoms)
    inner = np.max(np.sum(r < float(np.max(s.potential["dens_R"])) + skin, 1))
    ref = orc.forces(s.pos, s.species, s.box[0], s.periodic[0], orc.Potential(s.potential))
    sim = md.Simulation(s, precision=precision)
    sim.eam_forces()
    en = sim.energy()
    longest = sim.get_option(md.MD_OPT_MAX_COUNT)
    assert longest <= cap and (longest + 31) // 32 == rounds and (inner + 31) // 32 == inner_rounds
    assert force_error(sim.forces(), ref.f) <= TOL[precision]["force"]
    assert energy_error(sim.atom_energies(), ref.e_atom) <= TOL[precision]["energy"]
    assert abs(en.pe[0] - ref.pe) <= TOL[precision]["energy"] * abs(ref.pe)


@pytest.mark.parametrize("knots", [{1: 2.59}, {0: 2.2071, 1: 2.2171}, {1: 2.585}])
def test_staging_beside_larger_tables(md, knots):
    """Tables of 412 and 822 bins, with and without knots inside bins: beside them
    the records of the density pass, the force pass, both or neither are staged."""
    announce(f"staging with knots {knots}")
    parts, fill = _parts(5, (250, 127, 64, 65, 1), "fe_fs", 0.3, 64)
    pot = dict(fill.potential, pair_r=np.array(fill.potential["pair_r"]))
    for k, r in knots.items():
        pot["pair_r"][..., k] = r
    for p in (*parts, fill):
        p.potential = pot
    for mode in ("nve", "nvt"):
        _both_sides(md, parts, fill, 4 * PER_SIMD, mode=mode)
