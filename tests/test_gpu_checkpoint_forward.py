"""The forward results of a plan with and without checkpoints: the same bits in FP64.  FP32 plans
with the reverse mode form the Lagrangian potentials by other FP64 transforms, whose rounding
differs: phi1 and phi2 agree to twice the bars that each is held to against the oracle (1e-12 and
1e-11 of the maximum), positions to the FP32 bar of 1e-4 cell."""
import pytest

import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("every", [1, 4])
@pytest.mark.parametrize("Np,order,N_lpt", [(32, 2, 0), (64, 2, 0), (32, 4, 0), (32, 2, 16)])
def test_forward_with_and_without_checkpoints(precision, every, Np, order, N_lpt):
    import torch

    import paper_2003_04925_amd as S
    L, tiles = 4.0 * Np, S.uniform_tiling(Np, 2, 8)
    w = torch.from_numpy(synthetic.white_noise(N_lpt or Np, 8)).cuda()
    sims = [S.Simulation(L, Np, tiles, 6, precision=precision, fda_order=order, N_lpt=N_lpt,
                         want_momenta=True, checkpoint_every=c) for c in (0, every)]
    a, b = [s.forward(w) for s in sims]
    other = precision == "fp32" and order == 2 and not N_lpt
    for k, bar in (("phi1", 2e-12), ("phi2", 2e-11)):
        u, v = [s.view(k) for s in sims]
        if other:
            assert float((u - v).abs().max()) < bar * float(u.abs().max())
        else:
            assert torch.equal(u, v)
    if other:
        d = (a["pos"].double() - b["pos"].double()) * (Np / L)
        d = torch.remainder(d + Np / 2, Np) - Np / 2
        assert float(d.abs().max()) < 1e-4
    else:
        for k in ("pos", "mom", "density"):
            assert torch.equal(a[k], b[k])
