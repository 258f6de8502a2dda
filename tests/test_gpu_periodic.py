"""The periodic FP64 solves of the set-up (five fused passes, one kernel set per grid side)
through scola_setup, at every grid side: against the oracle up to 256, and on plane waves,
whose potentials have a closed form, at 512."""
import numpy as np
import pytest

import synthetic
from oracle.cosmology import Cosmology
from oracle.lpt import lagrangian_potentials, linear_power

pytestmark = pytest.mark.gpu

A_I = 0.05


def _sim(N, order, L):
    """A plan whose LPT grid has N nodes per side (a lattice of at least 32)."""
    import paper_2003_04925_amd as S
    Np = max(N, 32)
    per = max(1, Np // 64)
    buf = 0 if Np // per >= 16 else 4
    return S.Simulation(L, Np, S.uniform_tiling(Np, per, buf), 2, a_i=A_I, N_lpt=N,
                        fda_order=order)


@pytest.mark.parametrize("N,order", [(8, 2), (8, 6), (16, 2), (16, 4), (32, 2), (64, 4),
                                     (128, 2), (128, 6), (256, 2)])
def test_setup_potentials_at_every_grid_side(N, order):
    import torch
    L = 4.0 * N
    sim = _sim(N, order, L)
    w = synthetic.white_noise(N, 7)
    # the noise at an address that is no multiple of 16 bytes, as a slice of a larger array
    store = torch.empty(N ** 3 + 1, dtype=torch.float64, device="cuda")
    noise = store[1:].view(N, N, N)
    noise.copy_(torch.from_numpy(w))
    sim.setup(noise)
    c = Cosmology()
    ratio = 1.0 / c.growth(np.array([1.0]), A_I)[0][0]
    phi1, phi2 = lagrangian_potentials(w, L, c, ratio, order)
    for name, want in (("phi1", phi1), ("phi2", phi2)):
        got = sim.view(name).cpu().numpy()
        assert np.abs(got - want).max() < 1e-11 * np.abs(want).max(), name


@pytest.mark.parametrize("N", [64, 512])
def test_plane_waves_have_their_closed_form(N):
    """phi1 of a plane wave is the wave times sqrt(P N^3 / L^3) / symbol; the sum of three
    waves touches the zero column, the Nyquist column and the interior of the half spectrum."""
    import torch
    L = 4.0 * N
    sim = _sim(N, 2, L)
    c = Cosmology()
    ratio = 1.0 / c.growth(np.array([1.0]), A_I)[0][0]
    i = torch.arange(N, dtype=torch.float64, device="cuda")
    w = torch.zeros((N, N, N), dtype=torch.float64, device="cuda")
    want = torch.zeros_like(w)
    for m, amp in (((3, N // 2 - 1, 5), 1.0), ((N // 2, 1, 0), -0.5), ((2, 7, N // 2), 0.25)):
        ph = [torch.remainder(i * q, N) for q in m]
        wave = amp * torch.cos(2 * np.pi / N * (ph[0][:, None, None] + ph[1][None, :, None] +
                                                ph[2][None, None, :]))
        k = 2 * np.pi / L * np.sqrt(sum(q * q for q in m))
        f = np.sqrt(linear_power(np.array([k]), c)[0] * ratio ** 2 * N ** 3 / L ** 3)
        sym = -4.0 * sum(np.sin(np.pi * q / N) ** 2 for q in m)
        w += wave
        want += wave * (f / sym)
    sim.setup(w)
    got = sim.view("phi1")
    assert float((got - want).abs().max()) < 1e-11 * float(want.abs().max())
