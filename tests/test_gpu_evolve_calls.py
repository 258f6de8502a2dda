"""scola_evolve called in other ways than once over all tiles in order: tile lists in any order,
eager calls while the caller records a graph, per-tile plans on either side of the number of
launches up to which they are recorded, the persistent step of a plan with checkpoints, and its
grid."""
import pytest

import synthetic

pytestmark = pytest.mark.gpu

NP, L = 32, 100.0


def _noise(Np, seed):
    import torch
    return torch.from_numpy(synthetic.white_noise(Np, seed)).cuda()


@pytest.mark.parametrize("schedule", ["batched", "per_tile"])
@pytest.mark.parametrize("order", [[5, 2, 7, 0, 1, 3, 6, 4], [0, 7, 6, 5, 4, 3, 2, 1], [3, 1], None])
def test_last_potential_for_any_tile_order(schedule, order):
    """A plan with checkpoints leaves the last force's potential of every evolved tile where the
    operator-level calls look for it, in whichever order the tiles are listed."""
    import torch

    import paper_2003_04925_amd as S
    tiles = S.uniform_tiling(NP, 2, 8)
    w = _noise(NP, 3)
    plain = S.Simulation(L, NP, tiles, 5, precision="fp64", schedule=schedule)
    plain.setup(w)
    plain.evolve()
    sim = S.Simulation(L, NP, tiles, 5, precision="fp64", schedule=schedule, checkpoint_every=2)
    sim.setup(w)
    for _ in range(3):                 # eager, then a recorded graph where one is taken
        sim.view("phi").fill_(float("nan"))
        sim.evolve(order)
        for t, (po, M, go, ho) in enumerate(sim.box_slices()):
            got, n = sim.view("phi")[ho:ho + (M + 3) ** 3], M ** 3
            if order is None or t in order:
                assert torch.equal(got, plain.view("phi")[ho:ho + (M + 3) ** 3]), t
                for k in ("x_res", "p_res"):
                    assert torch.equal(sim.view(k)[:, po:po + n], plain.view(k)[:, po:po + n])
            else:
                assert bool(got.isnan().all()), t


@pytest.mark.parametrize("graph", [False, True])
def test_eager_call_while_the_caller_records_another(graph):
    """Inside a caller's capture the per-tile schedule stays on the captured stream, so that an
    eager call on a stream that is not being captured still runs before the capture ends."""
    import torch

    import paper_2003_04925_amd as S
    tiles = S.uniform_tiling(NP, 2, 8)
    w = _noise(NP, 4)
    ref = S.Simulation(L, NP, tiles, 3, precision="fp64").forward(w)["pos"]
    sim = S.Simulation(L, NP, tiles, 3, precision="fp64", schedule="per_tile")
    sim.set_graph(graph)
    sim.setup(w)
    for _ in range(3):                 # the plan has its streams and events, and its graph
        sim.evolve()
    torch.cuda.synchronize()
    pos = torch.empty_like(ref)
    g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        sim.evolve()
        with torch.cuda.stream(side):
            sim.evolve([1, 2, 4, 7])
            sim.evolve()
            sim.output(pos=pos)
    torch.cuda.synchronize()
    assert torch.equal(pos, ref)
    for _ in range(3):
        sim.view("x_res").zero_()
        g.replay()
        sim.output(pos=pos)
        assert torch.equal(pos, ref)


@pytest.mark.parametrize("Np,per_side,buffer,steps,momenta,recorded", [
    (32, 2, 8, 4, False, True), (64, 8, 4, 3, False, True), (64, 8, 4, 4, False, False),
    (64, 8, 4, 2, True, True), (64, 8, 4, 3, True, False)])
def test_per_tile_recording_is_bounded(Np, per_side, buffer, steps, momenta, recorded):
    """At most 8192 launches of the per-tile schedule become a graph (512 tiles: 3 steps, 2 with
    momenta); plans beyond, which a graph slows down, launch their kernels on every call."""
    import torch
    from torch.profiler import ProfilerActivity, profile

    import paper_2003_04925_amd as S
    tiles, w = S.uniform_tiling(Np, per_side, buffer), _noise(Np, 5)
    ref = S.Simulation(4.0 * Np, Np, tiles, steps, want_momenta=momenta).forward(w)["pos"]
    sim = S.Simulation(4.0 * Np, Np, tiles, steps, want_momenta=momenta, schedule="per_tile")
    sim.setup(w)
    for _ in range(2):
        sim.evolve()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        sim.evolve()
        torch.cuda.synchronize()
    pos = torch.empty_like(ref)
    sim.output(pos=pos)
    assert torch.equal(pos, ref)
    calls = [e.name for e in prof.events() if e.name.startswith("hip")]
    if not calls:
        pytest.skip("the profiler saw no runtime calls")
    assert calls.count("hipGraphLaunch") == (1 if recorded else 0)


@pytest.mark.parametrize("every", [1, 2, 7])
@pytest.mark.parametrize("momenta", [False, True])
def test_persistent_step_with_checkpoints(every, momenta):
    """The persistent step leaves the state, the checkpoints and the last segment's positions and
    potentials, from which the reverse mode starts, bitwise as the default schedule does."""
    import torch

    import paper_2003_04925_amd as S
    n = 5
    w = _noise(NP, 6)
    sims = []
    for persistent in (False, True):
        sim = S.Simulation(L, NP, S.uniform_tiling(NP, 2, 8), n, checkpoint_every=every,
                           want_momenta=momenta)
        sim.set_persistent(persistent)
        sim.set_graph(False)
        sim.setup(w)
        sim.evolve()
        sims.append(sim)
    a, b = sims
    assert b.persistent()["enabled"] and b.persistent()["barrier_failures"] == 0
    for k in ("x_res", "p_res", "phi"):
        assert torch.equal(a.view(k), b.view(k)), k
    P, H = a.layout.n_particles, a.layout.n_padded

    def kept(sim, name, first, count):
        off = sim._ws_off + getattr(sim.layout, name) + 4 * first
        return sim.workspace[off:off + 4 * count].view(torch.float32)
    saved = (n + every - 1) // every
    assert torch.equal(kept(a, "ckpt", 0, saved * 6 * P), kept(b, "ckpt", 0, saved * 6 * P))
    last = (n - 1) // every * every
    for k in range(last, n):
        slot = k % (every + 1)
        assert torch.equal(kept(a, "seg_phi", slot * H, H), kept(b, "seg_phi", slot * H, H)), k
        if k > last:
            assert torch.equal(kept(a, "seg_x", slot * 3 * P, 3 * P),
                               kept(b, "seg_x", slot * 3 * P, 3 * P)), k


@pytest.mark.parametrize("Np,per_side,buffer", [(32, 1, 8), (64, 1, 16), (64, 1, 24), (32, 2, 8),
                                                (64, 2, 8)])
def test_persistent_grid(Np, per_side, buffer):
    """One block per CU where that holds every plane and pencil chunk of the class, else at most
    three; the state is the default schedule's, bitwise, on either side."""
    import torch

    import paper_2003_04925_amd as S
    tiles, w = S.uniform_tiling(Np, per_side, buffer), _noise(Np, 7)
    sims = []
    for persistent in (False, True):
        sim = S.Simulation(4.0 * Np, Np, tiles, 3)
        sim.set_persistent(persistent)
        sim.setup(w)
        sim.evolve()
        sims.append(sim)
    for k in ("x_res", "p_res", "phi"):
        assert torch.equal(sims[0].view(k), sims[1].view(k)), k
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    M = Np // per_side + 2 * buffer
    mesh = per_side ** 3 * max(M + 3, ((M - 1) ** 2 + 63) // 64)
    st = sims[1].persistent()
    assert st["barrier_failures"] == 0
    assert (st["grid"] <= cus) == (mesh <= cus) and st["grid"] <= 3 * cus


def test_subsets_of_a_persistent_plan():
    """Tile subsets of a plan with the persistent step, which run on one stream: the default
    schedule's bits, in the order of the caller's stream."""
    import torch

    import paper_2003_04925_amd as S
    tiles, w = S.uniform_tiling(NP, 2, 8), _noise(NP, 8)
    sims = [S.Simulation(L, NP, tiles, 3) for _ in range(2)]
    for sim in sims:
        sim.setup(w)
        sim.evolve()
    a, b = sims
    b.set_persistent(True)
    b.evolve()
    for _ in range(2):
        for k in ("x_res", "p_res"):
            b.view(k).fill_(-7.0)
        b.evolve([6, 0, 3])
        b.evolve([1, 2, 4, 5, 7])
        for k in ("x_res", "p_res"):
            assert torch.equal(a.view(k), b.view(k)), k
    assert b.persistent()["barrier_failures"] == 0


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("Np,buffer", [(16, 4), (32, 8), (32, 16)])
def test_single_step_subsets(precision, Np, buffer):
    """One step of fewer than eight boxes of up to 32^3 stays on one stream, others fork: every
    subset gives the batched run's bits."""
    import torch

    import paper_2003_04925_amd as S
    tiles, w = S.uniform_tiling(Np, 2, buffer), _noise(Np, 10)
    sim = S.Simulation(4.0 * Np, Np, tiles, 1, precision=precision)
    sim.setup(w)
    sim.evolve()
    want = {k: sim.view(k).clone() for k in ("x_res", "p_res")}
    for subset in ([7], [0, 6], [5, 1, 2], [0, 1, 2, 3, 4, 5, 7]):
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
