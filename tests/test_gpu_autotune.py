"""GPU test of the autotuner's candidates: neighbour chunks of two and eight are
timed only where a pass runs one thread per atom (the split form of small systems
has no chunk, so its three candidates would be one, told apart by noise)."""
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


@pytest.mark.parametrize("precision,cells,candidates", [("mixed", 10, 1), ("mixed", 41, 3), ("fp64", 10, 2),
                                                        ("fp64", 41, 6)])
def test_chunk_candidates(md, precision, cells, candidates):
    """One list build per candidate and round, two rounds (automatic rebuilds leave
    out the brick kernels; FP64 times both evaluators)."""
    announce(f"autotune candidates {precision} {cells} cells")
    sim = md.Simulation(inputs.bcc_fe(cells, seed=63, displace=0.05), precision=precision)
    sim.set_option(md.MD_OPT_AUTO_REBUILD, 1)
    sim.eam_forces()
    sim.energy()
    before = sim.get_option(md.MD_OPT_N_BUILDS)
    choice = sim.autotune(trials=1)
    assert sim.get_option(md.MD_OPT_N_BUILDS) - before == 2 * candidates
    assert choice["kernel"] == 1 and choice["nchunk"] in ((4,) if cells == 10 else (2, 4, 8))
