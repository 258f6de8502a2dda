"""The largest grid sides of the periodic FP64 solves, on two crossed plane waves, whose
potentials of both orders have a closed form: with phi1 = A cos(a x) + B cos(b x), s = sin a,
t = sin b per axis (central differences), the second-order source is
A B cos(a x) cos(b x) |s x t|^2, whose product is a sum of two waves.  The waves and their sum
and difference touch the zero column, the Nyquist column and the interior of the half
spectrum.  Bar: 1e-10 of the maximum, ten times the bar of the smaller grids, since the
reference's P(k) and growth (quadratures to 1e-12 and 1e-11) enter the second order twice; a
wrong mode, twiddle or column changes the result by its own size."""
import numpy as np
import pytest

from oracle.cosmology import Cosmology
from oracle.lpt import linear_power

pytestmark = pytest.mark.gpu

A_I = 0.05


@pytest.mark.parametrize("N", [64, 512, 1024])
def test_crossed_plane_waves(N):
    import torch

    import paper_2003_04925_amd as S
    L = 4.0 * N
    per = N // 64 if N > 64 else 1
    sim = S.Simulation(L, N, S.uniform_tiling(N, per, 0), 2, a_i=A_I)
    c = Cosmology()
    ratio = 1.0 / c.growth(np.array([1.0]), A_I)[0][0]
    i = torch.arange(N, dtype=torch.float64, device="cuda")

    def add(out, m, amp):
        """out += amp cos(2 pi m x / N), from the products of the axes' cosines and sines."""
        f = [2.0 * np.pi / N * torch.remainder(i * q, N) for q in m]
        co, si = [torch.cos(p) for p in f], [torch.sin(p) for p in f]
        yz_c = torch.outer(co[1], co[2]) - torch.outer(si[1], si[2])
        yz_s = torch.outer(si[1], co[2]) + torch.outer(co[1], si[2])
        for x in range(N):
            out[x] += amp * (co[0][x] * yz_c - si[0][x] * yz_s)

    def symbol(m):
        return -4.0 * sum(np.sin(np.pi * q / N) ** 2 for q in m)

    def amplitude(m):
        k = 2.0 * np.pi / L * np.sqrt(sum(q * q for q in m))
        p = linear_power(np.array([k]), c)[0]
        return np.sqrt(p * ratio ** 2 * N ** 3 / L ** 3) / symbol(m)
    a, b = (N // 8 + 1, 3, N // 4), (2, N // 4 - 1, N // 4)
    w = torch.zeros((N, N, N), dtype=torch.float64, device="cuda")
    add(w, a, 1.0)
    add(w, b, 1.0)
    sim.setup(w)
    A, B = amplitude(a), amplitude(b)
    s, t = (np.sin(2.0 * np.pi * np.array(m) / N) for m in (a, b))
    half = 0.5 * A * B * float((np.cross(s, t) ** 2).sum())
    plus = tuple(p + q for p, q in zip(a, b))
    minus = tuple(p - q for p, q in zip(a, b))
    for name, waves in (("phi1", ((a, A), (b, B))),
                        ("phi2", ((plus, half / symbol(plus)), (minus, half / symbol(minus))))):
        w.zero_()
        for m, amp in waves:
            add(w, m, amp)
        top = float(w.abs().max())
        w.sub_(sim.view(name))
        assert float(w.abs_().max()) < 1e-10 * top, name
