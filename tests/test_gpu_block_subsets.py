"""Tile subsets under each block numbering give the bits of the hardware order for every tile of
the subset and touch no other tile."""
import pytest

import synthetic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Np,per_side,buffer,subset", [
    (32, 1, 24, [0]), (64, 4, 8, [0]), (64, 4, 8, [63, 5, 17]), (64, 4, 16, [2, 40]),
    (64, 1, 32, [0])])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_subset_gives_the_bits_of_the_hardware_order(Np, per_side, buffer, subset, precision):
    import torch

    import paper_2003_04925_amd as S
    tiles = S.uniform_tiling(Np, per_side, buffer)
    sim = S.Simulation(4.0 * Np, Np, tiles, 3, precision=precision)
    w = torch.from_numpy(synthetic.white_noise(Np, 6)).cuda()
    sched = sim.schedule()
    sim.set_graph(False)
    sim.set_schedule({M: dict(v, xcd_remap_particles=0, xcd_remap_mesh=0)
                      for M, v in sched.items()})
    whole = sim.forward(w)["pos"].clone()
    want = {k: sim.view(k).clone() for k in ("x_res", "p_res")}
    for remap in (1, 0):
        sim.set_schedule({M: dict(v, xcd_remap_particles=remap, xcd_remap_mesh=remap)
                          for M, v in sched.items()})
        for k in want:
            sim.view(k).fill_(-7.0)
        sim.evolve(subset)
        for t, (po, M, go, ho) in enumerate(sim.box_slices()):
            for k in want:
                got = sim.view(k)[:, po:po + M ** 3]
                if t in subset:
                    assert torch.equal(got, want[k][:, po:po + M ** 3]), (t, k)
                else:
                    assert bool((got == -7.0).all()), (t, k)
        pos = torch.full_like(whole, -1.0)
        sim.output(pos=pos, tile_subset=subset)
        done = pos >= 0
        assert int(done[0].sum()) == sum(tiles[t][1] ** 3 for t in subset)
        assert torch.equal(pos[done], whole[done])
