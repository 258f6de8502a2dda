"""The reverse mode on tilings whose boxes overlap in other ways than the uniform ones: a box
longer than the lattice (it covers sites several times), boxes of two sizes, box origins at odd
sites and more boxes than a block has threads; with the segment lengths at which the ring and
the checkpoints meet (1, a divisor of the steps, a remainder, more than the steps).  FP64 bar
as in the other gradient tests: 1e-7 of the oracle's largest entry."""
import numpy as np
import pytest

import synthetic
from oracle.adjoint import loss_and_gradient
from oracle.tiling import Tile

pytestmark = pytest.mark.gpu

NP, L = 16, 150.0
MIXED = [((0, 0, 0), 12, 10)] + [((x, y, z), 4, 6) for x in range(0, 16, 4)
                                 for y in range(0, 16, 4) for z in range(0, 16, 4)
                                 if max(x, y, z) >= 12]
ODD = [((x, y, z), 2, 7) for x in range(0, 16, 2) for y in range(0, 16, 2)
       for z in range(0, 16, 2)]


@pytest.mark.parametrize("name,tiles,steps,every", [
    ("mixed", MIXED, 3, 2), ("odd", ODD, 2, 1), ("mixed", MIXED, 4, 2), ("mixed", MIXED, 2, 5),
    ("mixed", MIXED, 1, 1)])
@pytest.mark.parametrize("groups", [1, 4])
def test_gradient_on_overlapping_tilings(name, tiles, steps, every, groups):
    import torch

    import paper_2003_04925_amd as S
    sim = S.Simulation(L, NP, tiles, steps, precision="fp64", checkpoint_every=every)
    sim.groups = groups
    w = synthetic.white_noise(NP, 4)
    target = synthetic.loss_target(NP, 43)
    _, want, _ = loss_and_gradient(w, L, [Tile(*t) for t in tiles], target, n_steps=steps)
    plain = S.Simulation(L, NP, tiles, steps, precision="fp64")
    x = torch.from_numpy(w).cuda()
    ref = plain.forward(x)
    t = torch.from_numpy(target).cuda()
    for _ in range(3):                 # eager, then the recorded graph, then its replay
        out = sim.forward(x)
        assert torch.equal(out["pos"], ref["pos"])
        # the state and the last potential where the operator-level calls find them
        assert torch.equal(sim.view("x_res"), plain.view("x_res"))
        assert torch.equal(sim.view("p_res"), plain.view("p_res"))
        assert torch.equal(sim.view("phi"), plain.view("phi"))
        grad = sim.backward(2.0 * (out["density"] - t)).cpu().numpy()
        assert np.abs(grad - want).max() < 1e-7 * np.abs(want).max()
