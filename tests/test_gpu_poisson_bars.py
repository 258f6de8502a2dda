"""The FP32 Poisson passes at the block sizes of every box side, held to tighter bars: the wide
stencils' potentials to 3e-6 of the maximum, the bar of the order-2 passes (the transforms, where
FP32 rounds, are the same), and the reverse passes' gradient to a relative L2 of 1e-4 against the
FP64 plan's with at most three particles in another output cell there (2e-3 each: positions agree
to about 1e-6 cells, so of 32768 particles about 0.2 lie that close to a cell face)."""
import numpy as np
import pytest

import synthetic
from oracle.poisson import dirichlet_potential

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [4, 6])
@pytest.mark.parametrize("Np,buffer", [(16, 0), (16, 8), (16, 16), (32, 16), (32, 24), (32, 32),
                                       (32, 40), (32, 48)])
def test_wide_potential_to_the_order_2_bar(order, Np, buffer):
    import torch

    import paper_2003_04925_amd as S
    sim = S.Simulation(4.0 * Np, Np, S.uniform_tiling(Np, 1, buffer), 2, fda_order=order)
    M, side = Np + 2 * buffer, Np + 2 * buffer + 1 + order
    sim.setup(torch.from_numpy(synthetic.white_noise(Np, 17)).cuda())
    sim.op_deposit(2.0, -2.0)
    rho = sim.view("rho").cpu().numpy()[:(M - 1) ** 3].reshape((M - 1,) * 3)
    delta = rho / 2.0 ** sim.layout.fixed_bits - 1.0
    sim.op_poisson(2.0)
    got = sim.view("phi").double().cpu().numpy()[:side ** 3].reshape((side,) * 3)
    bc = sim.view("bc0").cpu().numpy()[:side ** 3].reshape((side,) * 3)
    want = dirichlet_potential(delta, 2.0 * bc, order=order)
    assert np.abs(got - want).max() < 3e-6 * np.abs(want).max()


@pytest.mark.parametrize("buffer", [8, 16, 24, 32, 40, 48])
def test_reverse_passes_with_few_cell_changes(buffer):
    import torch

    import paper_2003_04925_amd as S
    Np, L = 32, 200.0
    w = torch.from_numpy(synthetic.white_noise(Np, 9)).cuda()
    t = torch.from_numpy(synthetic.loss_target(Np, 45)).cuda()
    grad, pos = {}, {}
    for precision in ("fp32", "fp64"):
        sim = S.Simulation(L, Np, S.uniform_tiling(Np, 1, buffer), 2, precision=precision,
                           checkpoint_every=1)
        out = sim.forward(w)
        pos[precision] = out["pos"].double().cpu().numpy() * (Np / L)
        grad[precision] = sim.backward(2.0 * (out["density"] - t.to(out["density"].dtype))).cpu()
    moved = int((np.floor(pos["fp32"]) != np.floor(pos["fp64"])).any(axis=0).sum())
    assert moved <= 3
    rel = float((grad["fp32"] - grad["fp64"]).norm() / grad["fp64"].norm())
    assert rel < 1e-4 + 2e-3 * moved


def test_many_boxes_of_128_as_one_alone():
    """The pencils of many boxes of 128^3 take another block size than those of a few: the same
    bits for a box among 64 and by itself."""
    import torch

    import paper_2003_04925_amd as S
    sim = S.Simulation(128.0, 32, S.uniform_tiling(32, 4, 60), 2)
    sim.setup(torch.from_numpy(synthetic.white_noise(32, 11)).cuda())
    sim.evolve()
    P, h = 128 ** 3, 131 ** 3
    want = {k: sim.view(k)[:, 37 * P:38 * P].clone() for k in ("x_res", "p_res")}
    phi = sim.view("phi")[37 * h:38 * h].clone()
    for k in ("x_res", "p_res", "phi"):
        sim.view(k).fill_(-7.0)
    sim.evolve([37])
    for k in want:
        assert torch.equal(sim.view(k)[:, 37 * P:38 * P], want[k]), k
    assert torch.equal(sim.view("phi")[37 * h:38 * h], phi)
