"""Worlds around the size from which a binned world has tile lists (512 nodes).

Worlds of up to 512 nodes test every node in every tile, larger ones read lists.
Alone or side by side in a batch, where both kinds share the launches, each
world's state is bitwise the same.
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


@pytest.mark.parametrize("nx,ny,offset", [(75, 50, 0.0), (640, 610, 0.0), (96, 130, 0.75)])
def test_worlds_around_the_limit_alone_and_in_a_batch(nx, ny, offset):
    sim, batch = _mods()
    sizes = [511, 512, 513, 514]
    worlds = [wl.random_world(80 + n, nx, ny, [n // 8] * 7 + [n - 7 * (n // 8)], amp=0.5) for n in sizes]
    par = sim.Params(nx=nx, ny=ny, marker_offset=offset)
    assert [w.n_particles for w in worlds] == sizes
    eng = batch.BatchEngine(max_worlds=4, pool_bytes=512 << 20)
    slots = [eng.admit(w, par, 22) for w in worlds]
    eng.advance(22)
    for k, w in enumerate(worlds):
        got = eng.retire(slots[k], w)
        W = sim.World(w, par)
        W.rollout(0, 22)
        W.sync()
        for name in ("cell", "frac", "f", "u"):
            assert torch.equal(getattr(got, name), getattr(W.state, name)), (name, sizes[k])
