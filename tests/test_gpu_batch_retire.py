"""Worlds taken out of a batch before their last step.

A slot can be retired after any sim_batch_advance; its state is then that of
the steps it has taken, the velocity of the last of them included.  Compared
bit for bit with the same world run alone for that many steps (the binned
transfer's sums do not depend on the order), for worlds with and without tile
lists and two-layer markers, after runs of captured pairs, of captured chunks
and both, and for a budget that ends inside the run.
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


@pytest.mark.parametrize("ran", [2, 10, 20, 26])
@pytest.mark.parametrize("unfused", [False, True])
def test_early_retire_equals_a_run_of_that_many_steps(ran, unfused):
    sim, batch = _mods()
    worlds = [(wl.random_world(31, 72, 50, [20, 9, 40], amp=0.5), 0.0, 100),
              (wl.random_world(32, 130, 97, [48] * 30, amp=0.5), 0.0, 31),
              (wl.random_world(33, 96, 110, [40] * 20, amp=0.5), 0.75, 90),
              (wl.random_world(34, 64, 64, [12] * 8, amp=0.5), 0.0, 7)]      # ends on an odd step
    eng = batch.BatchEngine(max_worlds=6, pool_bytes=128 << 20)
    if unfused:                              # forcing iterations: the separate kernels run for all
        w = wl.random_world(35, 64, 64, [12] * 8, amp=0.5)
        eng.admit(w, sim.Params(nx=64, ny=64, mdf_iters=2), 200)
    par = lambda w, off: sim.Params(nx=w.nx, ny=w.ny, marker_offset=off)
    slots = [eng.admit(w, par(w, off), steps) for w, off, steps in worlds]
    eng.advance(ran)
    for (w, off, steps), slot in zip(worlds, slots):
        taken = min(steps, ran)
        assert eng.remaining(slot) == steps - taken
        got = eng.retire(slot, w)
        W = sim.World(w, par(w, off))
        W.rollout(0, taken)
        W.sync()
        for name in ("cell", "frac", "f", "u"):
            assert torch.equal(getattr(got, name), getattr(W.state, name)), (name, w.nx, taken)


@pytest.mark.parametrize("kind", [dict(mdf_iters=3), dict(transfer="sorted"), dict(transfer="direct"),
                                  dict(transfer="sorted", tile=64), dict(marker_offset=0.75)])
def test_a_retired_kind_of_world_leaves_no_launches_behind(kind):
    # a world of another kind adds launches to every step, or takes the
    # one-kernel step away; some admissions after it has gone the others run as
    # in a batch that never had one (before, never again: 1.5 times the step
    # after a world with forcing iterations), and with the same results
    import time
    sim, batch = _mods()
    w = wl.random_world(41, 128, 110, [40] * 20, amp=0.5)
    other = wl.random_world(42, 64, 64, [12] * 8, amp=0.5)
    us = {}
    for had in (False, True):
        eng = batch.BatchEngine(max_worlds=3, pool_bytes=128 << 20)
        if had:
            s = eng.admit(other, sim.Params(nx=64, ny=64, **kind), 4)
            eng.advance(4)
            eng.retire(s, other)
        for _ in range(6):
            s = eng.admit(w, sim.Params(nx=w.nx, ny=w.ny), 4)
            eng.advance(4)
            got = eng.retire(s, w)
        s = eng.admit(w, sim.Params(nx=w.nx, ny=w.ny), 10 ** 8)
        eng.advance(40)
        best = float("inf")
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            eng.advance(40)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t)
        us[had] = best / 40 * 1e6
        eng.close()
        W = sim.World(w, sim.Params(nx=w.nx, ny=w.ny))
        W.rollout(0, 4)
        for name in ("cell", "frac", "f", "u"):
            assert torch.equal(getattr(got, name), getattr(W.state, name)), name
    print({k: round(v, 1) for k, v in us.items()})
    assert us[True] <= 1.25 * us[False]
