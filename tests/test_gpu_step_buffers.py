"""The per-step buffers after an ordinary step.

The binned step of few tiles runs its last four sub-steps in one kernel that
keeps the grid force in LDS.  After the call the buffers hold what the same
step run sub-step by sub-step leaves, bit for bit (the arithmetic is the
same), and the adjoint hook of the fluid update, which reads the world's grid
force, returns the same.
"""
import pytest
import torch

from paper_2607_02954_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0.0, 0.75])
@pytest.mark.parametrize("nx, ny, lens", [(72, 50, [20, 9, 31]), (130, 97, [48] * 30)])
def test_buffers_after_a_step_are_the_sub_steps(nx, ny, lens, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_02954_amd import sim
    w = wl.random_world(nx, nx, ny, lens, amp=0.5)
    p = sim.Params(nx=nx, ny=ny, marker_offset=offset)
    A, B = sim.World(w, p), sim.World(w, p)
    A.rollout(0, 7)
    B.rollout(0, 6)
    B.sync()
    for k in range(5):
        B.substep(k, 6)
    A.sync()
    B.sync()
    N = w.n_particles
    for which, shape in ((1, (ny, nx, 2)), (2, (ny, nx, 2)), (3, (2, N)), (4, (2, N))):
        a, b = A.buffer(which, shape), B.buffer(which, shape)
        assert float(b.abs().max()) > 0 and torch.equal(a, b), which
    for name in ("cell", "frac", "f", "u"):
        assert torch.equal(getattr(A.state, name), getattr(B.state, name)), name
    g = torch.randn(9, ny, nx, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    outs = []
    for W in (A, B):
        out = torch.zeros_like(g)
        W.adjoint_substep(2, g, out, torch.zeros(4 * nx * ny, device="cuda"))
        torch.cuda.synchronize()
        outs.append(out)
    assert torch.equal(*outs)


@pytest.mark.parametrize("nx, n, kw, own_kernels", [
    (72, 3, {}, (0, 4)),                             # S0 - S3 and S4 - S7 in a kernel each
    (200, 100, {"energy_rate": 0.05}, (0, 4, 5)),
    (200, 100, {"mdf_iters": 2}, (0, 3, 4, 5)),      # S4 - S7 apart
    (96, 40, {"transfer": "sorted"}, (0, 1, 2, 3, 4, 5)),
])
def test_profile_times_the_kernels_a_step_runs(nx, n, kw, own_kernels):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np
    from paper_2607_02954_amd import sim
    w = wl.random_world(3, nx, nx, [24] * n, amp=0.5)
    if "energy_rate" in kw:
        w.energy = np.ones((nx, nx), dtype=np.float32)
    p = sim.Params(nx=nx, ny=nx, **kw)
    A, B = sim.World(w, p), sim.World(w, p)
    ms = A.profile(0, 7)
    B.rollout(0, 7)
    B.sync()
    print([round(1e3 * v, 1) for v in ms], "us")
    assert [k for k, v in enumerate(ms) if v > 0] == list(own_kernels)
    for name in ("cell", "frac", "f", "u") + (("energy", "energy_collected") if "energy_rate" in kw else ()):
        assert torch.equal(getattr(A.state, name), getattr(B.state, name)), name
