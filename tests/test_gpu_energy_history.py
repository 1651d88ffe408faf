"""GPU test of md_energy_history's host memory: a history of many replicas is
copied in pieces, so the call needs little beyond the caller's records; every
piece, across the end of the ring too, holds the energies of its steps."""
import ctypes
import resource

import numpy as np
import pytest

from paper_1107_2619_amd import inputs
from tests.gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def md():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_2619_amd import md as _md

    return _md


def _dimers(n):
    """n pairs of Fe atoms in open boxes, stretched by a little more each."""
    base = inputs.workload("bcc2000")
    pos = np.tile(np.array([[5.0, 5.0, 5.0], [7.4, 5.0, 5.0]]), (n, 1))
    pos[1::2, 0] += 0.2 * np.arange(n) / n
    return inputs.System(
        name="dimers", pos=pos, vel=np.zeros_like(pos), species=np.zeros(2 * n, np.uint8),
        rigid=np.zeros(2 * n, np.uint8), atom_offset=np.arange(0, 2 * n + 1, 2, dtype=np.int64),
        box=np.full((n, 3), 12.0), origin=np.zeros((n, 3)), periodic=np.zeros((n, 3), np.uint8),
        rigid_velocity=np.zeros((n, 3)), potential=base.potential, dt_fs=0.02, skin=0.3, rebuild_every=10, steps=0,
        temperature=np.zeros(n), max_neighbours=8,
    )


def test_history_copies_in_pieces(md):
    """4096 replicas, 256 steps into a ring of 250 entries (94 MiB, pieces of two
    entries): peak memory grows by less than 32 MiB over the call, and the entries
    equal those read after every step."""
    announce("energy history of 4096 replicas")
    n, ring, steps = 4096, 250, 256
    s = _dimers(n)
    each = md.Simulation(s, precision="fp64", energy_ring=4)
    each.set_option(md.MD_OPT_ENERGY_EVERY, 1)
    want = []
    for _ in range(steps):
        each.step(1)
        want += [(h.step, h.pe, h.ke) for h in each.energy_history()]
    want = want[-ring:]

    sim = md.Simulation(s, precision="fp64", energy_ring=ring)
    sim.set_option(md.MD_OPT_ENERGY_EVERY, 1)
    for _ in range(steps):
        sim.step(1)
    sim.energy()
    out = (md._Energies * (n * ring))()
    ctypes.memset(out, 1, ctypes.sizeof(out))  # the caller's records are paid for before
    got = ctypes.c_int64(0)
    before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
    sim.ctx._check(sim.ctx.lib.md_energy_history(sim.ctx.handle, out, ring, ctypes.byref(got), sim.stream))
    grown = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before
    assert got.value == ring
    rec = np.frombuffer(out, np.dtype(md._Energies)).reshape(ring, n)
    for k, (step, pe, ke) in enumerate(want):
        assert rec["step"][k, 0] == step
        assert np.array_equal(rec["pe"][k], pe) and np.array_equal(rec["ke"][k], ke)
    assert grown < 32 * 1024  # KiB
