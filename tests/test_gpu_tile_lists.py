"""Tile lists of the binned transfer against every tile testing every node.

The sums of the binned transfer are exact in fixed point, so a step's result
does not depend on how its tiles find their nodes: a world whose workspace
leaves its lists too short (segments overflow and the tiles test every node),
and one without lists, equal the same world with full lists bit for bit.  The
worlds cross the places where the lists can go wrong: axes of one to six
tiles, a last tile narrower than the reach of a node, crowded tiles, every
tile side, radius and marker layer.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2607_02954_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _sim():
    from paper_2607_02954_amd import sim
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sim


def _run(sim, w, p, nbytes, steps):
    """State after `steps` steps with a workspace of nbytes (None if refused)."""
    st = sim.DeviceState(w)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    arr, cp, h = st.arrays(), p.c(), ctypes.c_void_p()
    L = sim.lib()
    if L.sim_create(ctypes.byref(cp), ctypes.byref(arr), sim._ptr(ws), nbytes, sim._stream_handle(),
                    ctypes.byref(h)) == sim.SIM_E_WORKSPACE:
        return None
    for n in (steps - 1, 1):                     # an odd run, then a single step
        sim.check(L.sim_rollout(h, 0, n, 0, None, 0))
    assert L.sim_sync(h) in (sim.SIM_OK, sim.SIM_E_UNSTABLE)   # (a crowd may trip the Mach guard)
    L.sim_destroy(h)
    return [t.clone().view(torch.int32) for t in (st.cell, st.frac, st.f, st.u)]


def _crowd(seed, nx, ny, n, spread):
    """n short chains around the middle of the world (crowded tiles)."""
    w = wl.random_world(seed, nx, ny, [12] * n, amp=0.3)
    x = w.positions64()
    c = np.array([[nx / 2.0], [ny / 2.0]])
    mid = np.repeat(np.stack([x[:, k * 12:(k + 1) * 12].mean(1) for k in range(n)], 1), 12, axis=1)
    w.cell, w.frac = wl.split_position(x - mid + c + spread * (mid - c))
    return w


CASES = [
    # nx, ny, chains, spread of the crowd, tile side, radius, marker offset
    (200, 170, 90, 1.0, 32, 4, 0.0),
    (200, 170, 120, 0.1, 32, 4, 0.0),            # most nodes in a few tiles
    (97, 65, 60, 1.0, 32, 4, 0.0),               # last tiles one cell wide
    (100, 40, 60, 1.0, 32, 8, 0.0),
    (33, 20, 50, 1.0, 16, 8, 0.0),
    (24, 24, 50, 1.0, 32, 6, 0.0),               # one tile
    (150, 330, 90, 0.4, 64, 2, 0.0),
    (117, 100, 90, 0.5, 16, 1, 0.75),
    (200, 99, 90, 0.3, 32, 4, 1.0),
    # two tiles along an axis, the last narrower than a node's reach; three with a narrow last one
    (50, 18, 60, 1.0, 16, 4, 0.0),
    (19, 66, 60, 1.0, 16, 2, 0.5),
    (72, 50, 60, 1.0, 16, 4, 0.0),
    # enough 32-cell tiles to keep that side, last ones one and three cells wide
    (641, 547, 90, 1.0, 32, 4, 0.0),
    (641, 547, 90, 0.2, 32, 8, 0.5),
    (353, 1100, 300, 0.15, 32, 3, 0.0),
]


@pytest.mark.parametrize("nx, ny, chains, spread, tile, radius, offset", CASES)
def test_lists_equal_testing_every_node(nx, ny, chains, spread, tile, radius, offset):
    sim = _sim()
    w = _crowd(nx + ny, nx, ny, chains, spread)
    p = sim.Params(nx=nx, ny=ny, tile=tile, repulse_radius=radius, marker_offset=offset)
    nb, cp = ctypes.c_size_t(), p.c()
    sim.check(sim.lib().sim_workspace_size(ctypes.byref(cp), w.n_filaments, w.n_particles, ctypes.byref(nb)))
    full = int(nb.value)
    ref = _run(sim, w, p, full, 8)
    sizes = [int(full * k / 40) // 256 * 256 for k in range(39, 9, -1)]
    ran = 0
    for nbytes in sizes[::3] + sizes[-1:]:
        got = _run(sim, w, p, nbytes, 8)
        if got is None:
            break
        ran += 1
        for a, b, name in zip(got, ref, ("cell", "frac", "f", "u")):
            assert torch.equal(a, b), (name, nbytes, full)
    assert int(ref[3].abs().max()) > 0
    print(f"{nx}x{ny} tile {tile}: {ran} smaller workspaces of {full} bytes equal")


def test_node_count_around_the_list_limit():
    """Worlds of 511 to 514 nodes (no lists up to 512) match a batch of them and each other's common part."""
    sim = _sim()
    for n in (511, 512, 513):
        w = wl.random_world(7, 120, 90, [n - 500, 250, 250], amp=0.5)
        p = sim.Params(nx=w.nx, ny=w.ny)
        W = sim.World(w, p)
        W.rollout(0, 5)
        W.sync()
        D = sim.World(w, sim.Params(nx=w.nx, ny=w.ny, transfer="sorted"))
        D.rollout(0, 5)
        D.sync()
        a, b = W.positions(), D.positions()
        # FP32 rounding of five steps' displacements in cells of about 100
        assert float((a - b).abs().max()) <= 1e-5
