"""The work that users of the framework have it do, as cases that can be timed.

Each case is one call of a user's program: a step, a rollout from a start
state, a rollout with its gradient (one world, or a set of worlds), a queue of
rollout jobs through the batch server, or the folding objective.  Sizes are
those of the workloads module and of the benchmark, and generic ones between
them.  ``exact`` repeats each case in 64 bits with plain torch.
"""
import math

import numpy as np
import torch

from paper_2607_02954_amd import batch, serve, sim
from paper_2607_02954_amd import workloads as wl

F64 = torch.float64
TWO_PI = 2.0 * math.pi


def _case(kind, name=None, **kw):
    c = {"kind": kind, "nx": 64, "ny": 64, "nodes": 32, "lo": 32, "hi": 32, "steps": 1, "amp": 0.5, "radius": 4,
         "pbd": 4, "mdf": 1, "offset": 0.0, "packets": 0, "shape": "chains", "worlds": 1, "every": 0, "tile": 32}
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one step of one creature: an interactive caller, or a controller in the loop
        _case("step", "step 64x64", nx=64, ny=64, nodes=32, lo=32, hi=32),
        # a few short creatures in a small odd box: one evaluation of a search
        _case("rollout", "rollout 72x50", nx=72, ny=50, nodes=150, lo=3, hi=40, steps=50),
        # the uniform population of 1024 x 64 nodes
        _case("rollout", "rollout 512x512", nx=512, ny=512, nodes=65536, lo=64, hi=64, steps=40),
        # the million-node scaling workload
        _case("rollout", "rollout 2048x2048", nx=2048, ny=2048, nodes=1048576, lo=16, hi=256, steps=20),
        # swimmers that sense and collect an energy field
        _case("rollout", "energy 512x384", nx=512, ny=384, nodes=12000, lo=48, hi=48, steps=40, packets=96),
        # branched creatures (chains and loops with chains hanging from them)
        _case("rollout", "branched 400x400", nx=400, ny=400, nodes=12000, steps=40, shape="branched"),
        # the coupling's leakage fixes on the quarter-density population
        _case("rollout", "mdf two-layer 1024x1024", nx=1024, ny=1024, nodes=65536, lo=16, hi=256, steps=20, mdf=4,
              offset=0.75),
        # folding: gradient of a position loss in the rest angles
        _case("grad", "gradient 256x256", nx=256, ny=256, nodes=3072, lo=48, hi=48, steps=60, every=20, amp=0.0),
        # the same for a population of worlds at once
        _case("grad", "gradient of 16 worlds 256x256", nx=256, ny=256, nodes=3072, lo=48, hi=48, steps=20, every=20,
              amp=0.0, worlds=16),
        # the gradient of a large population
        _case("grad", "gradient 1024x1024", nx=1024, ny=1024, nodes=262144, lo=16, hi=256, steps=10, every=5),
        # uneven jobs through the batch server, all arrived at once
        _case("serve", "serve 12 jobs", worlds=12, nodes=12000, lo=8, hi=128, nx=128, ny=320, steps=80),
        # the folding objective on its own: image, loss and gradient at the paper's sizes
        _case("loss", "density loss 1000 nodes", nx=256, ny=256, nodes=1000, lo=128, hi=128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "rollout", "rollout", "rollout", "rollout", "grad", "grad", "set", "serve", "loss"])
    if kind == "loss":
        side = _log(rng, 64, 512)
        px = _log(rng, 32, 256)                               # pixels per side
        return _case("loss", nx=side, ny=side, nodes=_log(rng, 100, 20000), lo=px, hi=px)
    if kind == "serve":
        return _case("serve", worlds=rng.randint(2, 12), nodes=_log(rng, 300, 12000), lo=8, hi=128,
                     nx=128, ny=rng.choice([192, 256, 320]), steps=rng.randint(20, 80))
    # (the side's logarithm is spread evenly; the two sides differ, and are seldom multiples of a tile)
    top = {"step": 700, "rollout": 2048, "grad": 1000, "set": 200}[kind]
    nx = _log(rng, 48, top)
    ny = max(48, min(top, int(nx * rng.uniform(0.6, 1.6))))
    shape = rng.choice(["chains", "chains", "chains", "general", "branched"]) if nx <= 600 else "chains"
    mdf, offset = rng.choice([(1, 0.0), (1, 0.0), (1, 0.0), (3, 0.0), (1, 0.75), (4, 0.5)])
    density = rng.uniform(0.02, 0.06) if mdf > 1 or shape == "branched" else rng.uniform(0.02, 0.25)
    nodes = max(32, int(density * nx * ny))
    hi = min(rng.choice([24, 48, 128, 256, 256, 1000]), nodes)
    lo = min(rng.choice([1, 3, 8, 16]), hi)
    big = nx * ny > 300 * 300
    c = _case("grad" if kind == "set" else kind, nx=nx, ny=ny, nodes=nodes, lo=lo, hi=hi, shape=shape,
              radius=rng.choice([4, 4, 4, 2, 6]), pbd=rng.choice([4, 4, 4, 2, 8]), mdf=mdf, offset=offset)
    if kind == "step":
        c.update(mdf=1)
        return c
    if kind == "rollout":
        c["steps"] = rng.randint(8, 20) if big else rng.randint(20, 60)
        c["packets"] = rng.choice([0, 0, 0, 20])
        return c
    c["amp"] = rng.choice([0.0, 0.5])
    c["steps"] = rng.randint(4, 8) if big else rng.randint(10, 40)
    c["every"] = rng.choice([2, 4]) if big else rng.choice([5, 10, 20])
    if kind == "set":
        c["worlds"] = rng.randint(2, 12)
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _lengths(total, lo, hi):
    """Lengths U{lo..hi} that sum to about `total` (at least one filament); the
    same for every seed, so that all inputs of a case have its sizes."""
    g = np.random.Generator(np.random.PCG64(total + 7919 * lo + 104729 * hi))
    n = g.integers(lo, hi + 1, size=max(1, int(2 * total / (lo + hi)) + 16))
    k = int(np.searchsorted(np.cumsum(n), total))
    return [int(v) for v in n[:max(1, k)]]


def _world(c, seed):
    """The start state of one world of the case (host arrays)."""
    nx, ny = c["nx"], c["ny"]
    if c["shape"] == "branched":
        # (a creature holds about 38 nodes); the same creatures for every
        # seed, at other places, with other rest angles and phases
        w = wl.branched_world(c["nodes"], nx, ny, max(1, c["nodes"] // 38), amp=c["amp"])
        g = np.random.Generator(np.random.PCG64(seed))
        fil = np.repeat(np.arange(w.n_filaments), np.diff(w.fil_offset))
        creature = np.cumsum(w.parent < 0)[fil]
        shift = g.uniform(0, 1, (2, creature[-1] + 1)) * [[nx], [ny]]
        w.cell, w.frac = wl.split_position(w.positions64() + shift[:, creature])
        w.rest_angle = (w.rest_angle + g.normal(0, 0.1, w.n_particles)).astype(np.float32)
        w.act_phase = g.uniform(0, TWO_PI, w.n_filaments).astype(np.float32)
    elif c["shape"] == "general":
        ls = _lengths(c["nodes"], c["lo"], c["hi"])
        w = wl.generality_world(seed, nx, ny, ls, [3 + (k * 7) % 40 for k in range(max(1, len(ls) // 8))],
                                amp=c["amp"])
    else:
        w = wl.random_world(seed, nx, ny, _lengths(c["nodes"], c["lo"], c["hi"]), amp=c["amp"])
    if c["packets"]:
        g = np.random.Generator(np.random.PCG64(seed + 77))
        P = c["packets"]
        w.meta["packets"] = (g.uniform(0, 1, (2, P)) * [[nx], [ny]], g.uniform(0.5, 2, P), g.uniform(3, 12, P))
        w.energy = np.zeros((ny, nx), dtype=np.float32)
    return w


def _worlds(c, seed):
    return [_world(c, 1000003 * (k + 1) + seed) for k in range(c["worlds"])]


def _jobs(c, seed):
    """Uneven jobs: node counts log-uniform, sides in steps of 32, steps uniform
    (as the served workload); their sizes are the same for every seed."""
    g = np.random.Generator(np.random.PCG64(c["nodes"]))
    jobs = []
    for k in range(c["worlds"]):
        nodes = int(round(math.exp(g.uniform(math.log(8), math.log(c["nodes"])))))
        side = int(g.choice(np.arange(c["nx"], c["ny"] + 1, 32)))
        d = dict(c, nx=side, ny=side, nodes=nodes)
        jobs.append(wl.Job(job_id=k, arrival=0.0, steps=int(g.integers(c["steps"] // 2, c["steps"] + 1)),
                           world=_world(d, 1000003 * (k + 1) + seed)))
    return jobs


def _params(c, nx=None, ny=None):
    return sim.Params(nx=nx or c["nx"], ny=ny or c["ny"], pbd_iters=c["pbd"], repulse_radius=c["radius"],
                      mdf_iters=c["mdf"], marker_offset=c["offset"], energy_rate=0.05 if c["packets"] else 0.0,
                      tile=c["tile"])


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _targets(worlds, seed):
    """Target positions near the start ([2, N_w] blocks one after another, flat)."""
    g = np.random.Generator(np.random.PCG64(seed + 13))
    return np.concatenate([(w.positions64() + g.normal(0, 2, (2, w.n_particles))).ravel() for w in worlds])


def _target_image(c, seed):
    g = np.random.Generator(np.random.PCG64(seed + 5))
    x = np.linspace(-1, 1, c["lo"])
    r = np.hypot(x[None, :], x[:, None]) - g.uniform(0.3, 0.7)
    return np.exp(-(r / 0.08) ** 2).astype(np.float32)


def _curled(c, seed):
    """One curled filament (a persistent random walk) in the middle of the world."""
    g = np.random.Generator(np.random.PCG64(seed))
    return wl.split_position(wl.curled_chain(g, c["nodes"], (c["nx"] / 2.0, c["ny"] / 2.0), 0.5))


def prepare(case, seed):
    c = case
    if c["kind"] == "loss":
        cell, frac = _curled(c, seed)
        return {"case": c, "cell": torch.from_numpy(cell).cuda(), "frac": torch.from_numpy(frac).cuda(),
                "target": torch.from_numpy(_target_image(c, seed)).cuda()}
    if c["kind"] == "serve":
        jobs = _jobs(c, seed)
        engine = batch.BatchEngine(max_worlds=c["worlds"], pool_bytes=1 << 30)
        x0 = [torch.from_numpy(j.world.positions64()).cuda() for j in jobs]
        server = serve.Server(serve.GpuExecutor(engine, lambda job: _params(c, job.world.nx, job.world.ny)),
                              chunk_steps=20)
        return {"case": c, "jobs": jobs, "server": server, "engine": engine, "x0": x0}
    worlds = _worlds(c, seed)
    p = _params(c)
    if c["worlds"] > 1:
        W = sim.WorldSet(worlds, p)
        states = W.states
    else:
        W = sim.World(worlds[0], p)
        states = [W.state]
    s = {"case": c, "W": W, "states": states, "t": 0,
         "cell": [st.cell.clone() for st in states], "frac": [st.frac.clone() for st in states]}
    if c["packets"]:
        st = states[0]
        packets = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda", torch.float32)
                   for a in worlds[0].meta["packets"]]
        s["energy"] = sim.energy_packets(c["nx"], c["ny"], *packets)
        st.energy.copy_(s["energy"])
    x0 = W.positions()
    s["x0"] = x0
    if c["kind"] == "grad":
        s["target"] = torch.from_numpy(_targets(worlds, seed)).cuda().reshape(x0.shape)
        rest = W.rest_angles() if c["worlds"] > 1 else W.state.rest_angle
        s["rest"] = rest.clone()
    return s


def _restart(s):
    """The start state again: nodes at their first positions, fluid at rest."""
    for st, cell, frac in zip(s["states"], s["cell"], s["frac"]):
        st.cell.copy_(cell)
        st.frac.copy_(frac)
        st.f.zero_()


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "step":
        W = s["W"]
        W.step(s["t"])                                   # the simulation goes on from call to call
        s["t"] += 1
        return {"cell": W.state.cell, "frac": W.state.frac, "u": W.state.u, "f": W.state.f}
    if c["kind"] == "rollout":
        W = s["W"]
        _restart(s)
        if c["packets"]:
            W.state.energy.copy_(s["energy"])
            W.state.energy_collected.zero_()
        W.rollout(0, c["steps"])
        out = {"moved": (W.positions() - s["x0"]).float(), "u": W.state.u, "f": W.state.f}
        if c["packets"]:
            out.update(energy=W.state.energy, collected=W.state.energy_collected, sensed=W.state.energy_sensed)
        return out
    if c["kind"] == "grad":
        W = s["W"]
        _restart(s)
        rest = s["rest"].detach().requires_grad_(True)
        fn = sim.SetRollout if c["worlds"] > 1 else sim.Rollout
        x = fn.apply(rest, W, 0, c["steps"], c["every"])
        loss = ((x - s["target"]) ** 2).sum() / (x.numel() // 2)
        (g,) = torch.autograd.grad(loss, rest)
        return {"moved": (x.detach() - s["x0"]).float(), "gradient": g, "f": [st.f for st in s["states"]]}
    if c["kind"] == "serve":
        stats = s["server"].run(s["jobs"])
        return [{"moved": (r.state.cell.double() + r.state.frac.double() - x0).float(), "u": r.state.u,
                 "f": r.state.f} for r, x0 in zip(stats.results, s["x0"])]
    loss, image, g = sim.density_loss(c["nx"], c["ny"], s["cell"], s["frac"], s["target"], 2.0, 0.1)
    return {"loss": loss, "image": image, "gradient": g}


def work(case):
    """Per step: populations read and written, positions and rest values read,
    positions written; the reverse mode reads and writes the populations'
    adjoint and reads the populations once more, after a second forward."""
    c = case
    if c["kind"] == "loss":
        P = c["lo"] * c["lo"]
        h = c["nx"] / c["lo"]
        cover = min(P, math.pi * (10.0 / h) ** 2)
        return {"bytes": 24.0 * c["nodes"] + 8.0 * P, "flops": 40.0 * c["nodes"] * cover}
    cells, nodes, steps = c["nx"] * c["ny"] * c["worlds"], c["nodes"] * c["worlds"], c["steps"]
    if c["kind"] == "serve":
        side = 0.5 * (c["nx"] + c["ny"])
        cells = side * side * c["worlds"]
        nodes = c["worlds"] * (c["nodes"] - 8) / max(1e-9, math.log(c["nodes"] / 8.0))
        steps = 0.75 * c["steps"]
    b, f = 72.0 * cells + 40.0 * nodes, 200.0 * cells + 1000.0 * nodes
    if c["packets"]:
        b += 8.0 * cells
    b *= steps
    f *= steps * (1.0 + 0.3 * (c["mdf"] - 1))
    if c["kind"] == "grad":
        b, f = 3.5 * b, 4.0 * f
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The same in 64 bits: plain torch, one vectorised expression per index set
# ---------------------------------------------------------------------------

class _Body:
    """Index sets and constants of one world's filaments (as the header of the
    C interface states them), on the device."""

    def __init__(self, w, dev):
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
        off = np.asarray(w.fil_offset, dtype=np.int64)
        n = np.diff(off)
        fil = np.repeat(np.arange(len(n)), n)
        N = int(off[-1])
        k = np.arange(N) - off[fil]
        closed = np.zeros(len(n), bool) if w.closed is None else np.asarray(w.closed, bool)
        ring = (closed & (n >= 3))[fil]
        odd_last = ring & (n[fil] % 2 == 1) & (k == n[fil] - 1)
        first, last = off[fil], off[fil] + n[fil] - 1
        i = np.arange(N)
        nxt = np.where(ring & (i == last), first, i + 1)
        prv = np.where(ring & (i == first), last, i - 1)
        edge = ring | (k < n[fil] - 1)
        joint = ring | ((k >= 1) & (k <= n[fil] - 2))
        jl = np.where(ring, k, k - 1)
        ecol = np.where(odd_last, 2, k % 2)
        jcol = np.where(odd_last, 2, jl % 2)
        self.N, self.F = N, len(n)
        self.nxt, self.prv, self.fil = t(nxt), t(prv), t(fil)
        self.edge = t(np.nonzero(edge)[0])
        self.joint = t(np.nonzero(joint)[0])
        self.edges = [t(np.nonzero(edge & (ecol == q))[0]) for q in range(3)]
        self.joints = [t(np.nonzero(joint & (jcol == q))[0]) for q in range(3)]
        self.phase_j = t((jl / np.maximum(np.where(ring, n[fil], n[fil] - 2), 1))[joint])
        # the nodes that a node's tangent joins
        self.ta = t(np.where(ring | (k > 0), prv, i))
        self.tb = t(np.where(ring | (k < n[fil] - 1), nxt, i))
        f64 = lambda a: t(np.asarray(a, dtype=np.float64))
        self.rest, self.length = f64(w.rest_angle), f64(w.rest_length)
        self.amp, self.period, self.phase = f64(w.act_amp), f64(w.act_period), f64(w.act_phase)
        self.stiff = None if w.stiffness is None else [f64(a) for a in w.stiffness]
        par = np.full(len(n), -1) if w.parent is None else np.asarray(w.parent, dtype=np.int64)
        kid = np.nonzero(par >= 0)[0]
        self.any_att = len(kid) > 0
        if self.any_att:
            att = np.asarray(np.asarray(w.attach, dtype=np.float32), dtype=np.float64)[:, kid]
            self.ap, self.ac, self.ain = t(par[kid]), t(off[kid]), t(prv[par[kid]])
            self.aL, self.aa, self.ab = (t(a) for a in att)
            two = np.nonzero(n[kid] >= 2)[0]
            self.a2 = t(two)


def _f32(v):
    return float(np.float32(v))


def _wrap(d):
    return d - TWO_PI * torch.ceil((d - math.pi) / TWO_PI)


def _edge_move(v, th, L, ks, ksh):
    ell = torch.sqrt(v[0] * v[0] + v[1] * v[1])
    st = (ell - L) * v / ell
    return 0.5 * ks * (st + ksh * (v - L * torch.stack([torch.cos(th), torch.sin(th)]) - st))


def _elastic(x, b, rest, t, c):
    hat = rest
    if b.joint.numel():
        f = b.fil[b.joint]
        arg = TWO_PI * t / b.period[f] + b.phase[f] - TWO_PI * b.phase_j
        hat = rest.index_add(0, b.joint, b.amp[f] * torch.sin(arg))
    kb, ks, ksh = (0.5, 1.0, 0.5) if b.stiff is None else b.stiff
    at = lambda k, i: k[i] if torch.is_tensor(k) else k
    y, th = x, torch.zeros(b.N, dtype=F64, device=x.device)
    if b.edge.numel():
        v = x[:, b.nxt[b.edge]] - x[:, b.edge]
        th = th.index_add(0, b.edge, torch.atan2(v[1], v[0]))
    if b.any_att:
        v = x[:, b.ac] - x[:, b.ap]
        tha = torch.atan2(v[1], v[0])
    for _ in range(c["pbd"]):
        for j in b.joints:
            if j.numel():
                a = b.prv[j]
                e = 0.5 * at(kb, j) * (_wrap(th[j] - th[a]) - hat[j])
                th = th.index_add(0, a, e).index_add(0, j, -e)
        if b.any_att:
            e = 0.25 * (_wrap(tha - th[b.ain]) - b.aa)
            th, tha = th.index_add(0, b.ain, e), tha - e
            n0 = b.ac[b.a2]
            e = 0.25 * (_wrap(th[n0] - tha[b.a2]) - b.ab[b.a2])
            th, tha = th.index_add(0, n0, -e), tha.index_add(0, b.a2, e)
        for e in b.edges:
            if e.numel():
                d = _edge_move(y[:, b.nxt[e]] - y[:, e], th[e], b.length[e], at(ks, e), at(ksh, e))
                y = y.index_add(1, e, d).index_add(1, b.nxt[e], -d)
        if b.any_att:
            d = _edge_move(y[:, b.ac] - y[:, b.ap], tha, b.aL, 1.0, 0.5)
            y = y.index_add(1, b.ap, d).index_add(1, b.ac, -d)
    return _f32(0.05) * (y - x)


def _phi(r):
    a = torch.abs(r)
    i, o = torch.clamp(a, max=1.0), torch.clamp(a, min=1.0, max=2.0)
    inner = (3 - 2 * i + torch.sqrt(1 + 4 * i - 4 * i * i)) / 8
    outer = (5 - 2 * o - torch.sqrt(-7 + 12 * o - 4 * o * o)) / 8
    return torch.where(a <= 1, inner, torch.where(a < 2, outer, torch.zeros_like(a)))


def _stencil(x, nx, ny):
    m = torch.arange(-1, 3, dtype=F64, device=x.device)
    cx = torch.floor(x[0].detach())[:, None] + m
    cy = torch.floor(x[1].detach())[:, None] + m
    wx, wy = _phi(cx - x[0][:, None]), _phi(cy - x[1][:, None])
    at = torch.remainder(cy.long(), ny)[:, :, None] * nx + torch.remainder(cx.long(), nx)[:, None, :]
    return at.reshape(-1, 16), (wy[:, :, None] * wx[:, None, :]).reshape(-1, 16)


def _spread(sts, v, nx, ny):
    out = torch.zeros(v.shape[0], ny * nx, dtype=F64, device=v.device)
    for at, w in sts:
        out = out.index_add(1, at.reshape(-1), (w * v[:, :, None] / len(sts)).reshape(v.shape[0], -1))
    return out.reshape(-1, ny, nx)


def _gather(sts, g):
    g = g.reshape(g.shape[0], -1)
    return sum((g[:, at] * w).sum(2) for at, w in sts) / len(sts)


_CX = [0, 1, 0, -1, 0, 1, -1, -1, 1]
_CY = [0, 0, 1, 0, -1, 1, 1, -1, -1]
_WQ = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
_OPP = [0, 3, 4, 1, 2, 7, 8, 5, 6]


def _step(x, g, t, b, c, rest, nx, ny):
    """One step: positions x and shifted populations g; returns both and u."""
    q = lambda a: torch.tensor(a, dtype=F64, device=x.device).reshape(9, 1, 1)
    cx, cy, wq = q(_CX), q(_CY), q(_WQ)
    R = c["radius"]
    one = [_stencil(x, nx, ny)]
    st = one
    if c["offset"] > 0:
        tan = x[:, b.tb] - x[:, b.ta]
        n2 = tan[0] ** 2 + tan[1] ** 2
        tan = torch.where(n2 > 0, tan / torch.sqrt(torch.where(n2 > 0, n2, torch.ones_like(n2))),
                          torch.zeros_like(tan))
        d = _f32(c["offset"]) * torch.stack([-tan[1], tan[0]])
        st = [_stencil(x + d, nx, ny), _stencil(x - d, nx, ny)]
    s = _spread(one, torch.ones(1, x.shape[1], dtype=F64, device=x.device), nx, ny)[0]
    taps = torch.exp(-torch.arange(-R, R + 1, dtype=F64) ** 2 / 2)
    taps = (taps / taps.sum()).tolist()
    s = sum(taps[k + R] * torch.roll(s, k, 1) for k in range(-R, R + 1))
    s = sum(taps[k + R] * torch.roll(s, k, 0) for k in range(-R, R + 1))
    D = 0.5 * torch.stack([torch.roll(s, -1, 1) - torch.roll(s, 1, 1), torch.roll(s, -1, 0) - torch.roll(s, 1, 0)])
    F = _elastic(x, b, rest, t, c) - _f32(0.1) * _gather(one, D)
    Fg = _spread(st, F, nx, ny)
    rho = 1 + g.sum(0)
    j = torch.stack([(g * cx).sum(0), (g * cy).sum(0)])
    if c["mdf"] > 1:
        Ud = _gather(st, j / rho) + 0.5 * F
        for _ in range(c["mdf"] - 1):
            Fg = Fg + _spread(st, 2 * (Ud - _gather(st, (j + 0.5 * Fg) / rho)), nx, ny)
    u = (j + 0.5 * Fg) / rho
    cu, us = cx * u[0] + cy * u[1], (u * u).sum(0)
    eq = wq * (rho * (3 * cu + 4.5 * cu * cu - 1.5 * us) + rho - 1)
    S = wq * ((3 * (cx - u[0]) + 9 * cu * cx) * Fg[0] + (3 * (cy - u[1]) + 9 * cu * cy) * Fg[1])
    sym, anti = lambda a: 0.5 * (a + a[_OPP]), lambda a: 0.5 * (a - a[_OPP])
    ne = g - eq                                            # tau = 1, Lambda = 1/4: both rates are 1
    out = g - sym(ne) - anti(ne) + 0.5 * sym(S) + 0.5 * anti(S)
    out = torch.stack([torch.roll(out[k], (_CY[k], _CX[k]), (0, 1)) for k in range(9)])
    return x + _gather(st, u), out, u


def _start(w, dev):
    x = torch.from_numpy(w.positions64()).to(dev)
    return x, torch.zeros(9, w.ny, w.nx, dtype=F64, device=dev), _Body(w, dev)


def _exact_rollout(w, c, steps, dev):
    x0, g, b = _start(w, dev)
    x, nx, ny = x0, w.nx, w.ny
    out = {}
    if c["packets"]:
        ctr, amp, wid = (torch.from_numpy(np.asarray(a, dtype=np.float32).astype(np.float64)).to(dev)
                         for a in w.meta["packets"])
        E = torch.zeros(ny, nx, dtype=F64, device=dev)
        ax, ay = (torch.arange(n, dtype=F64, device=dev) for n in (nx, ny))
        image = lambda d, n: d - n * torch.floor(d / n + 0.5)
        for k in range(len(amp)):
            r2 = image(ay - ctr[1, k], ny)[:, None] ** 2 + image(ax - ctr[0, k], nx)[None, :] ** 2
            E = E + amp[k] * torch.exp(-r2 / (2 * wid[k] ** 2))
        got = torch.zeros(b.F, dtype=F64, device=dev)
    for t in range(steps):
        if c["packets"]:
            one = [_stencil(x, nx, ny)]
            e = _gather(one, E[None])
            got = got.index_add(0, b.fil, _f32(0.05) * e[0])
            E = E - _spread(one, _f32(0.05) * e, nx, ny)[0]
        x, g, u = _step(x, g, t, b, c, b.rest, nx, ny)
    if c["packets"]:
        out.update(energy=E, collected=got, sensed=e[0])
    out.update(moved=x - x0, u=u.permute(1, 2, 0), f=g)
    return out, x


def _exact_grad(w, c, target, share, dev):
    """The final positions and populations, and dL/d(rest angle) of L = share * |x_T - target|^2."""
    x, g, b = _start(w, dev)
    x0, kept = x, []
    with torch.no_grad():
        for t in range(c["steps"]):
            kept.append((x, g))
            x, g, _ = _step(x, g, t, b, c, b.rest, w.nx, w.ny)
    end = g
    gx, gg, gr = 2 * share * (x - target), torch.zeros_like(g), torch.zeros_like(b.rest)
    for t in reversed(range(c["steps"])):
        xs, gs = (a.clone().requires_grad_(True) for a in kept.pop())
        r = b.rest.clone().requires_grad_(True)
        xe, ge, _ = _step(xs, gs, t, b, c, r, w.nx, w.ny)
        gx, gg, d = torch.autograd.grad([xe, ge], [xs, gs, r], [gx, gg], allow_unused=True)
        gr = gr if d is None else gr + d
    return x - x0, end, gr


def _exact_loss(c, seed, dev):
    cell, frac = _curled(c, seed)
    x = torch.from_numpy(cell.astype(np.float64) + frac.astype(np.float64)).to(dev)
    T = torch.from_numpy(_target_image(c, seed).astype(np.float64)).to(dev)
    P, nx, ny, amp = c["lo"], c["nx"], c["ny"], _f32(0.1)
    px = -0.5 + (torch.arange(P, dtype=F64, device=dev) + 0.5) * (nx / P)
    py = -0.5 + (torch.arange(P, dtype=F64, device=dev) + 0.5) * (ny / P)
    image = lambda d, n: d - n * torch.floor(d / n + 0.5)

    def parts(lo, hi):
        dx = image(x[0, lo:hi, None, None] - px[None, None, :], nx)
        dy = image(x[1, lo:hi, None, None] - py[None, :, None], ny)
        r2 = dx * dx + dy * dy
        return dx, dy, torch.where(r2 <= 100.0, amp * torch.exp(-r2 / 8.0), torch.zeros_like(r2))

    cut = list(range(0, x.shape[1], 256)) + [x.shape[1]]
    I = sum(parts(lo, hi)[2].sum(0) for lo, hi in zip(cut, cut[1:]))
    res = 2 * (I - T) / (P * P)
    g = [torch.stack([-(res * v * dx / 4).sum((1, 2)), -(res * v * dy / 4).sum((1, 2))])
         for dx, dy, v in (parts(lo, hi) for lo, hi in zip(cut, cut[1:]))]
    return {"loss": ((I - T) ** 2).mean().reshape(1), "image": I, "gradient": torch.cat(g, 1)}


def exact(case, seed):
    c, dev = case, _dev()
    if c["kind"] == "loss":
        return _exact_loss(c, seed, dev)
    if c["kind"] == "serve":
        with torch.no_grad():
            return [_exact_rollout(j.world, c, j.steps, dev)[0] for j in _jobs(c, seed)]
    worlds = _worlds(c, seed)
    if c["kind"] == "grad":
        total = sum(w.n_particles for w in worlds)
        target = torch.from_numpy(_targets(worlds, seed)).to(dev)
        moved, grads, ends, at = [], [], [], 0
        for w in worlds:
            m = 2 * w.n_particles
            d, end, g = _exact_grad(w, c, target[at:at + m].reshape(2, -1), 1.0 / total, dev)
            moved.append(d)
            grads.append(g)
            ends.append(end)
            at += m
        if c["worlds"] == 1:
            return {"moved": moved[0], "gradient": grads[0], "f": ends}
        return {"moved": torch.cat([d.reshape(-1) for d in moved]), "gradient": torch.cat(grads), "f": ends}
    with torch.no_grad():
        out, x = _exact_rollout(worlds[0], c, 1 if c["kind"] == "step" else c["steps"], dev)
    if c["kind"] == "step":
        del out["moved"]
        cell = torch.floor(x)
        out.update(cell=cell.int(), frac=x - cell)
    return out
