"""What a batch's pool holds.

sim_batch_world_bytes is the pool that one world takes: a pool of the tables
and n times that admits n worlds, whatever lists the worlds before them were
given.  Worlds with room beyond it get larger lists, from where no world is;
their results are the same.
"""
import pytest
import torch

from paper_2607_02954_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _mods():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_02954_amd import sim, batch
    return sim, batch


def _admit_all(sim, eng, jobs):
    slots = []
    try:
        for w, p in jobs:
            slots.append(eng.admit(w, p, 20))
    except sim.SimError as e:
        assert e.status == sim.SIM_E_WORKSPACE
    return slots


@pytest.mark.parametrize("n", [1, 4, 8, 12])
@pytest.mark.parametrize("side, chains", [(128, 60), (256, 250), (200, 1)])
def test_a_pool_admits_what_world_bytes_says(n, side, chains):
    sim, batch = _mods()
    w = wl.random_world(n, side, side, [48] * chains, amp=0.5)
    p = sim.Params(nx=side, ny=side)
    need = batch.BatchEngine.world_bytes(p, w.n_filaments, w.n_particles)
    # the tables are a fixed part of the pool and of the world count: below 8% here
    eng = batch.BatchEngine(max_worlds=n, pool_bytes=int(1.08 * n * need))
    slots = _admit_all(sim, eng, [(w, p)] * n)
    assert len(slots) == n
    eng.advance(20)
    W = sim.World(w, p)
    W.rollout(0, 20)
    for s in slots:
        got = eng.retire(s, w)
        for name in ("cell", "frac", "f", "u"):
            assert torch.equal(getattr(got, name), getattr(W.state, name)), name


def test_worlds_come_and_go_around_larger_lists():
    # uneven worlds in a pool that holds some of their larger lists: each
    # admission may take a place that larger lists lay in, each retirement
    # leaves one; every state equals the world's run alone
    sim, batch = _mods()
    worlds = [wl.random_world(60 + k, 96 + 32 * (k % 5), 96 + 16 * (k % 7), [40] * (8 + 23 * (k % 6)), amp=0.5)
              for k in range(14)]
    par = [sim.Params(nx=w.nx, ny=w.ny) for w in worlds]
    need = [batch.BatchEngine.world_bytes(p, w.n_filaments, w.n_particles) for w, p in zip(worlds, par)]
    eng = batch.BatchEngine(max_worlds=5, pool_bytes=int(1.3 * sum(sorted(need)[-5:])) + (1 << 20))
    alone = []
    for w, p in zip(worlds, par):
        W = sim.World(w, p)
        W.rollout(0, 24)
        W.sync()
        alone.append(W.state)
    waiting, inside, done = list(range(len(worlds))), {}, 0
    while waiting or inside:
        while waiting and len(inside) < 5:
            k = waiting[0]
            inside[eng.admit(worlds[k], par[k], 24)] = k
            waiting.pop(0)
            eng.advance(2)                        # (the others are partway)
        eng.advance(6)
        for s in [s for s in inside if eng.remaining(s) == 0]:
            k = inside.pop(s)
            got = eng.retire(s, worlds[k])
            for name in ("cell", "frac", "f", "u"):
                assert torch.equal(getattr(got, name), getattr(alone[k], name)), (name, k)
            done += 1
    assert done == len(worlds)
