"""The LDS windows of the periodic deposits (output density, tCOLA's mass) and of tCOLA's force
where a block's footprint fits, exceeds the window, or wraps round a grid smaller than itself.

Bars: a node's mass is a sum of integer weights each within three 2^-40 units of its exact
value, so the density of n particles on a node is within 3 n 2^-40 (N_out / N_p)^3 of the
oracle's; the mass of the grid is exactly one unit per particle; end to end FP64 runs are
within 1e-8 cell of the oracle, as in the other tests."""
import numpy as np
import pytest

import synthetic
from oracle.cosmology import Cosmology, cola_schedule
from oracle.run import output_density, setup_full_box
from oracle.scola import evolve_periodic, lattice_positions

pytestmark = pytest.mark.gpu

NP = 32


def _sim(L, N_out, order=2, steps=2, precision="fp64"):
    import paper_2003_04925_amd as S
    return S.Simulation(L, NP, S.uniform_tiling(NP, 2, 8), steps, precision=precision,
                        N_out=N_out, fda_order=order)


@pytest.mark.parametrize("call", ["forward", "tcola_forward"])
@pytest.mark.parametrize("N_out,L", [(32, 128.0), (8, 128.0), (3, 128.0), (45, 128.0),
                                     (100, 128.0), (32, 8.0), (50, 8.0)])
def test_output_density_in_every_window_form(call, N_out, L):
    """Grids from much coarser to three times finer than the lattice; at 8 Mpc/h the particles
    move tens of cells, so blocks exceed any window."""
    import torch
    sim = _sim(L, N_out)
    out = getattr(sim, call)(torch.from_numpy(synthetic.white_noise(NP, 5)).cuda())
    pos = out["pos"].cpu().numpy().reshape(3, -1) / (L / NP)
    want = output_density(pos, NP, N_out)
    scale = (N_out / NP) ** 3
    # positions in Mpc/h are rounded once more: 2^-50 of the box in each weight's slope
    bar = (want + 1.0).max() * (3 * 2.0 ** -40 * 8 + 2.0 ** -40) + scale * 1e-9
    got = out["density"].cpu().numpy()
    assert np.abs(got - want).max() <= bar
    if call == "forward":
        assert int(sim.view("outgrid").sum()) == NP ** 3 << 40


@pytest.mark.parametrize("order", [2, 4, 6])
@pytest.mark.parametrize("L", [128.0, 8.0])
def test_tcola_in_every_window_form(order, L):
    import torch
    w = synthetic.white_noise(NP, 6)
    sim = _sim(L, NP, order)
    out = sim.tcola_forward(torch.from_numpy(w).cuda())
    c = Cosmology()
    _, _, psi1, psi2 = setup_full_box(w, L, c, 0.05, order)
    steps, _ = cola_schedule(c, 0.05, 1.0, 2)
    ora = evolve_periodic(psi1, psi2, steps, fda_order=order)
    d = out["pos"].cpu().numpy() / (L / NP) - ora["u"]
    d = np.remainder(d + NP / 2, NP) - NP / 2
    assert np.abs(d).max() < 1e-8
