"""The particle step's block numberings: FP32 plans of at most 12288 bricks deal contiguous
ranges to the XCDs, larger ones runs of four bricks (grids padded to whole runs).  Plans on
either side of the line, with brick counts that are and are not multiples of a run's 32 blocks,
give the bits of the hardware order, batched, in box groups and for subsets of the tiles."""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Np,per_side,buffer", [(32, 1, 24), (64, 4, 8), (64, 4, 16), (64, 1, 32)])
def test_numbering_changes_no_result(Np, per_side, buffer):
    import torch

    import paper_2003_04925_amd as S
    tiles = S.uniform_tiling(Np, per_side, buffer)
    if (Np, buffer) == (64, 16):
        tiles = tiles[:-1] + [(tiles[-1][0], tiles[-1][1], tiles[-1][2] + 8)]   # an odd class
    sim = S.Simulation(4.0 * Np, Np, tiles, 3)
    w = torch.from_numpy(synthetic.white_noise(Np, 6)).cuda()
    sched = sim.schedule()
    sim.set_graph(False)
    sim.set_schedule({M: dict(v, xcd_remap_particles=0) for M, v in sched.items()})
    want = sim.forward(w)["pos"].clone()
    sim.set_schedule({M: dict(v, xcd_remap_particles=1) for M, v in sched.items()})
    for groups in (1, 2):
        sim.groups = groups
        assert torch.equal(sim.forward(w)["pos"], want)
    sim.evolve([0])
    sim.output(tile_subset=[0])
    assert np.isfinite(sim.view("x_res").cpu().numpy()).all()
