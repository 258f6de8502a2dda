"""The per-tile schedule over several streams and its recorded graph: every call (eager, the one
that records, replays, with other work between them, and tile subsets of 1 to 5 tiles) gives
bitwise the batched run, on the current stream's order and on a side stream, and inside a
capture of the caller's."""
import pytest

import synthetic

pytestmark = pytest.mark.gpu

NP, L = 32, 100.0
MIXED = [((0, 0, 0), 24, 4)] + [((x, y, z), 8, 4) for x in range(0, 32, 8)
                                for y in range(0, 32, 8) for z in range(0, 32, 8)
                                if max(x, y, z) >= 24]


def _sim(schedule, precision):
    import paper_2003_04925_amd as S
    return S.Simulation(L, NP, MIXED, 3, precision=precision, schedule=schedule,
                        want_momenta=True)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_per_tile_calls_equal_the_batched_run(precision):
    import torch
    w = [torch.from_numpy(synthetic.white_noise(NP, s)).cuda() for s in (1, 2)]
    ref = [_sim("batched", precision).forward(x) for x in w]
    sim = _sim("per_tile", precision)
    side = torch.cuda.Stream()
    junk = torch.zeros(1 << 20, device="cuda")
    for call in range(5):
        which = call % 2
        if call == 3:
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                out = sim.forward(w[which])
            torch.cuda.current_stream().wait_stream(side)
        else:
            out = sim.forward(w[which])
        junk.add_(1.0).sum().item()
        for k in ("pos", "mom", "density"):
            assert torch.equal(out[k], ref[which][k]), (call, k)
    for n in range(1, 6):
        sim.setup(w[0])
        sub = list(range(0, 2 * n, 2))
        sim.evolve(sub)
        pos = torch.full((3, NP, NP, NP), -1.0, dtype=sim.real, device="cuda")
        sim.output(pos=pos, tile_subset=sub)
        done = pos >= 0
        assert int(done[0].sum()) == sum(MIXED[t][1] ** 3 for t in sub)
        assert torch.equal(pos[done], ref[0]["pos"][done])


@pytest.mark.parametrize("warm,graph", [(0, False), (3, False), (0, True), (3, True)])
def test_per_tile_evolution_inside_a_caller_capture(warm, graph):
    import torch
    w = torch.from_numpy(synthetic.white_noise(NP, 3)).cuda()
    ref = _sim("batched", "fp64").forward(w)
    sim = _sim("per_tile", "fp64")
    sim.set_graph(graph)
    sim.setup(w)
    for _ in range(warm):
        sim.evolve()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sim.evolve()
    for _ in range(3):
        sim.setup(w)
        g.replay()
        pos = torch.empty((3, NP, NP, NP), dtype=sim.real, device="cuda")
        sim.output(pos=pos)
        assert torch.equal(pos, ref["pos"])
