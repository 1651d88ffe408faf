"""GPU tests of the list build's candidate handling: cells whose candidates are
pruned and held in registers at once, pruned but more than fit (a counting
sweep), more than the candidate table holds, more own atoms than a wavefront
has lanes, and pairs that take their minimum image one by one.  The list is
compared with every pair within r_c + skin, and the forces (whose density reads
only the front of each row) with the oracle."""
import numpy as np
import pytest

from paper_1107_2619_amd import inputs
from tests.gpu_helpers import TOL, announce, force_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def md():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_2619_amd import md as _md

    return _md


def _brute(s, rlist):
    from scipy.spatial import cKDTree

    tree = cKDTree(s.pos % s.box[0], boxsize=s.box[0])
    return [set(v) - {i} for i, v in enumerate(tree.query_ball_tree(tree, rlist))]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("cells,skin,cap,sheared", [
    (8, 0.4, 64, False),    # pruned, one or two register sets
    (8, 1.6, 96, False),    # ~16 atoms per cell: pruned, about 256 candidates left
    (8, 3.0, 160, False),   # ~38 atoms per cell, 1000 candidates: no table
    (11, 5.9, 400, False),  # ~85 atoms per cell: own atoms in two chunks
    (4, 1.5, 80, False),    # two link cells per axis: minimum images
    (10, 0.7, 64, True),    # a sheared cell
])
def test_list_and_forces(md, orc, precision, cells, skin, cap, sheared):
    announce(f"list build {precision} cells {cells} skin {skin} sheared {sheared}")
    s = inputs.bcc_fe(cells, seed=30 + cells, displace=0.08, skin=skin, vacancy_frac=0.02)
    s.max_neighbours = cap
    kw = {}
    if sheared:  # the same crystal in a cell whose third edge leans by the first
        h = np.diag(s.box[0]) @ np.array([[1.0, 0.0, 1.0], [0.0, 1.0, 0.0], [0.0, 0.0, 1.0]])
        kw["box_matrix"] = h
    sim = md.Simulation(s, precision=precision, **kw)
    sim.eam_forces()
    sim.energy()
    counts, lst = sim.neighbours()
    want = _brute(s, 4.1 + skin)
    for i, w in enumerate(want):
        assert counts[i] == len(w)
        assert set(lst[i, :counts[i]].tolist()) == w
    ref = orc.forces(s.pos, s.species, s.box[0], s.periodic[0], orc.Potential(s.potential))
    assert force_error(sim.forces(), ref.f) <= TOL[precision]["force"]
