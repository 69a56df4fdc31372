"""Workloads by which the engine's speed is judged, each through the package's
public entry points (mpcd.Context, mpcd.mpcd_moments_noalloc,
serve.LibraryEngine).

Six kinds of work, with sizes from the tests, the benchmark's workloads or of
generic shape:

  dump        steps, then the whole particle state to the host
  observe     steps, then the observables (momentum, energy, temperature,
              VACF): how long runs of boxes of 10^6 to 10^8 particles are read
  ensemble    many boxes stepped together, then every box observed
  serve       requests admitted, stepped in chunks, observed and released
  checkpoint  a saved state loaded, stepped, and saved again
  moments     momentum and energy of caller arrays already on the GPU

Cell sums are exact, so a box's trajectory is the same bits whatever the order
of the particles in memory, and every output here is reproducible.
"""
import math

import numpy as np
import torch

from paper_2212_11878_amd import inputs, mpcd, serve


# ---------------------------------------------------------------------------
# the cases

def _box(L, density, steps, **more):
    """A box of L[0] x L[1] x L[2] cells and how it is run; `more` replaces the defaults."""
    case = dict(L0=L[0], L1=L[1], L2=L[2], density=density, steps=steps, dt=0.1, alpha_deg=130.0, a=1.0,
                ids=True, masses=False, conserve_l=False, sort=False, vacf_stride=0)
    case.update(more)
    return case


def listed():
    return [
        # a solvent box coupled to other code that reads every particle after
        # each step: the smallest call, all latency
        dict(name="couple_8cube", kind="dump", **_box((8, 8, 8), 5.0, 1)),
        # the 10^3 test box, 100 steps between dumps: launches and host calls
        dict(name="small_10cube", kind="dump", **_box((10, 10, 10), 10.0, 100)),
        # the benchmark's 100^3 box with the velocity autocorrelation sampled
        dict(name="vacf_100cube", kind="observe", **_box((100, 100, 100), 10.0, 100, vacf_stride=10)),
        # the default benchmark: 256^3 cells, no particle ids
        dict(name="bench_256cube", kind="observe", **_box((256, 256, 256), 10.0, 40, ids=False)),
        # a box that no brick, block or tile divides, other density, cell edge,
        # angle and time step, ids kept
        dict(name="ragged_ids", kind="observe",
             **_box((203, 167, 131), 7.5, 50, dt=0.17, alpha_deg=95.0, a=1.25)),
        # embedded-particle runs: every particle carries its own mass
        dict(name="masses_96cube", kind="observe", **_box((96, 96, 96), 10.0, 50, masses=True)),
        # the angular-momentum-conserving rule
        dict(name="angmom_96cube", kind="observe", **_box((96, 96, 96), 10.0, 30, conserve_l=True)),
        # counting-sort binning: the form boxes too large for buckets take
        dict(name="sort_128cube", kind="observe", **_box((128, 128, 128), 10.0, 30, ids=False, sort=True)),
        # the paper's small systems in a batch: 512 boxes, edges 8..48,
        # densities 5..20, one launch sequence for all
        dict(name="ensemble_512", kind="ensemble", boxes=512, edge_lo=8, edge_hi=48, steps=50),
        # a serving round: requests of edges 8..64 arrive, run, are read, leave
        dict(name="serve_32", kind="serve", requests=32, edge_lo=8, edge_hi=64, chunks=4, chunk_steps=50),
        # resume from a checkpoint, run a little, checkpoint again
        dict(name="checkpoint_32cube", kind="checkpoint", **_box((32, 32, 32), 10.0, 10)),
        # diagnostics of a caller's own arrays, an odd count, with masses
        dict(name="moments_12M", kind="moments", n=12345677, masses=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dump", "observe", "observe", "observe", "ensemble", "serve", "checkpoint", "moments"])
    if kind == "moments":
        return dict(kind=kind, n=_log_int(rng, 1000, 60000000), masses=rng.random() < 0.5)
    if kind == "ensemble":
        lo = rng.randint(6, 16)
        return dict(kind=kind, boxes=_log_int(rng, 12, 400), edge_lo=lo, edge_hi=lo + rng.randint(8, 30),
                    steps=rng.randint(10, 50))
    if kind == "serve":
        lo = rng.randint(6, 16)
        return dict(kind=kind, requests=_log_int(rng, 3, 40), edge_lo=lo, edge_hi=lo + rng.randint(8, 46),
                    chunks=rng.randint(1, 5), chunk_steps=rng.randint(10, 50))
    density = round(rng.uniform(4.0, 18.0), 2)
    more = dict(dt=round(rng.uniform(0.05, 0.2), 3), alpha_deg=round(rng.uniform(80.0, 150.0), 1),
                a=rng.choice([1.0, 1.0, 1.25, 0.8]))
    if kind == "observe":
        edge = lambda: _log_int(rng, 24, 200)  # noqa: E731
        option = rng.choice(["plain", "plain", "ids", "vacf", "masses", "conserve_l", "sort"])
        more["ids"] = option not in ("plain", "sort")
        if option == "vacf":
            more["vacf_stride"] = rng.randint(1, 12)
        elif option != "ids" and option != "plain":
            more[option] = True
        limit = 1.0e9 if option in ("conserve_l", "sort") else 3.0e9
    else:
        edge = lambda: _log_int(rng, 4, 44)  # noqa: E731
        limit = 1.0e7
    L = (edge(), edge(), edge())
    n = density * L[0] * L[1] * L[2]
    steps = max(1, min(_log_int(rng, 1 if kind == "dump" else 5, 120), int(limit / n)))
    return dict(kind=kind, **_box(L, density, steps, **more))


# ---------------------------------------------------------------------------
# inputs

def _edges(case):
    return (case["L0"], case["L1"], case["L2"])


def _count(case):
    return int(round(case["density"] * case["L0"] * case["L1"] * case["L2"]))


def _thermal(case, seed):
    """Uniform positions and Maxwellian velocities (kT = m = 1, no net
    momentum) as float32 (3, N) arrays on the host."""
    n = _count(case)
    rng = np.random.default_rng([seed, 1])
    pos = np.empty((3, n), np.float32)
    for d, edge in enumerate(_edges(case)):
        size = np.float32(edge * case["a"])
        pos[d] = rng.random(n, dtype=np.float32) * size
        pos[d][pos[d] >= size] = 0.0
    vel = rng.standard_normal((3, n), dtype=np.float32)
    vel -= vel.mean(axis=1, keepdims=True, dtype=np.float64).astype(np.float32)
    return pos, vel


def _desc(case, seed, init):
    return mpcd.make_desc(_edges(case), _count(case), dt=case["dt"], alpha_deg=case["alpha_deg"], seed=seed + 1,
                          a=case["a"], init=init, vacf_stride=case["vacf_stride"],
                          vacf_capacity=1 << 16 if case["vacf_stride"] else 0, particle_mass=case["masses"],
                          conserve_l=case["conserve_l"], unordered=not case["ids"])


def _requests(case, seed, count):
    """Boxes of cubic shape, edges and densities uniform, each with its own
    parameters and seed."""
    rng = np.random.default_rng([seed, 2])
    boxes = []
    for _ in range(count):
        L = int(rng.integers(case["edge_lo"], case["edge_hi"] + 1))
        boxes.append(dict(L=L, n=int(round(rng.uniform(5.0, 20.0) * L ** 3)), dt=float(rng.uniform(0.05, 0.2)),
                          alpha_deg=float(rng.uniform(90.0, 150.0)), seed=int(rng.integers(1, 2 ** 62))))
    return boxes


def prepare(case, seed):
    kind = case["kind"]
    if kind == "moments":
        g = torch.Generator(device="cuda").manual_seed(seed)
        v = torch.randn((3, case["n"]), generator=g, device="cuda")
        m = 0.5 + torch.rand(case["n"], generator=g, device="cuda") if case["masses"] else None
        return dict(kind=kind, n=case["n"], v=v, m=m, out=torch.empty(5, dtype=torch.float64, device="cuda"))
    if kind == "serve":
        requests = [dict(r, steps=case["chunks"] * case["chunk_steps"])
                    for r in _requests(case, seed, case["requests"])]
        return dict(kind=kind, engine=serve.LibraryEngine(hbm_budget=64 << 30), requests=requests,
                    chunks=case["chunks"], chunk_steps=case["chunk_steps"])
    if kind == "ensemble":
        ctx = mpcd.Context()
        boxes = inputs.ensemble_boxes(case["boxes"], seed=seed + 1, edge=(case["edge_lo"], case["edge_hi"]))
        slots = [ctx.admit(mpcd.make_desc(b["L"], b["n"], dt=b["dt"], alpha_deg=b["alpha_deg"], seed=b["seed"]))
                 for b in boxes]
        return dict(kind=kind, ctx=ctx, slots=slots, steps=case["steps"])
    ctx = mpcd.Context(binning=mpcd.MPCD_BIN_SORT if case["sort"] else mpcd.MPCD_BIN_AUTO)
    if kind == "observe":
        slot = ctx.admit(_desc(case, seed, "maxwell"))
        if case["masses"]:
            ctx.set_mass(slot, np.random.default_rng([seed, 3]).uniform(0.5, 2.0, _count(case)).astype(np.float32))
        return dict(kind=kind, ctx=ctx, slot=slot, steps=case["steps"])
    state = _thermal(case, seed)
    slot = ctx.admit(_desc(case, seed, "external"), state)
    return dict(kind=kind, ctx=ctx, slot=slot, steps=case["steps"], saved=state)


# ---------------------------------------------------------------------------
# one pass

def _observed(o):
    return dict(step=int(o["step"]), P=o["P"], E=o["E"], T=o["T"], vacf=o["vacf"])


def run(state):
    kind = state["kind"]
    if kind == "moments":
        v, m = state["v"], state["m"]
        rc = mpcd.mpcd_moments_noalloc(v[0].data_ptr(), v[1].data_ptr(), v[2].data_ptr(),
                                       m.data_ptr() if m is not None else 0, state["n"], state["out"].data_ptr(),
                                       torch.cuda.current_stream().cuda_stream)
        if rc != mpcd.MPCD_OK:
            raise mpcd.MPCDError(rc, "mpcd_moments_noalloc")
        return state["out"]
    if kind == "serve":
        engine = state["engine"]
        slots = [engine.admit(r) for r in state["requests"]]
        for _ in range(state["chunks"]):
            engine.step(state["chunk_steps"])
        seen = []
        for slot in slots:
            seen.append(engine.observe(slot))
            engine.release(slot)
        return dict(T=np.array([o["T"] for o in seen]), vacf=np.concatenate([o["vacf"] for o in seen]),
                    step=np.array([o["step"] for o in seen]), status=np.array([o["status"] for o in seen]))
    ctx = state["ctx"]
    if kind == "ensemble":
        ctx.step(state["steps"])
        seen = [ctx.observe(slot) for slot in state["slots"]]
        return dict(P=np.array([o["P"] for o in seen]), E=np.array([o["E"] for o in seen]),
                    T=np.array([o["T"] for o in seen]), step=np.array([o["step"] for o in seen]))
    if kind == "observe":
        ctx.step(state["steps"])
        return _observed(ctx.observe(state["slot"]))
    if kind == "checkpoint":
        ctx.set_state(state["slot"], state["saved"], 0)
    ctx.step(state["steps"])
    pos, vel, step = ctx.get_state(state["slot"])
    return dict(pos=pos, vel=vel, step=step)


# ---------------------------------------------------------------------------
# what a pass cannot do without

def work(case):
    """Bytes: every particle's x, v (and id, mass where kept) read and written
    once a step; the state read and written once for a dump or a load; v read
    once for the observables.  Operations: streaming, cell index, sums and the
    affine collision map, about 60 a particle-step."""
    kind = case["kind"]
    if kind == "moments":
        return dict(bytes=case["n"] * (16 if case["masses"] else 12), flops=case["n"] * 12)
    if kind in ("ensemble", "serve"):
        # the mean of uniform edges cubed, densities of mean 12.5
        edges = range(case["edge_lo"], case["edge_hi"] + 1)
        n = 12.5 * sum(e ** 3 for e in edges) / len(edges)
        if kind == "ensemble":
            n, steps, extra = n * case["boxes"], case["steps"], 12
        else:   # admission writes x, v and id
            n, steps, extra = n * case["requests"], case["chunks"] * case["chunk_steps"], 12 + 28
        return dict(bytes=n * (56 * steps + extra), flops=60.0 * n * steps)
    n, steps = _count(case), case["steps"]
    step_bytes = 48 + (8 if case["ids"] else 0) + (8 if case["masses"] else 0)
    extra = dict(observe=12, dump=48, checkpoint=96)[kind]
    return dict(bytes=n * (step_bytes * steps + extra), flops=60.0 * n * steps * (8 if case["conserve_l"] else 1))


# ---------------------------------------------------------------------------
# 64-bit values

def _philox(k, cell, stream, seed):
    """Philox4x32-10 (Salmon et al., SC'11) of counters (k_lo, cell, k_hi, stream), key = seed."""
    low = np.uint64(0xFFFFFFFF)
    word = lambda v: np.broadcast_to(np.asarray(v, np.uint64), np.shape(cell)).copy()  # noqa: E731
    x, y, z, w = word(k & 0xFFFFFFFF), np.asarray(cell, np.uint64).copy(), word(k >> 32), word(stream)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        a, b = x * np.uint64(0xD2511F53), z * np.uint64(0xCD9E8D57)
        x, y, z, w = ((b >> np.uint64(32)) ^ y ^ np.uint64(k0), b & low, (a >> np.uint64(32)) ^ w ^ np.uint64(k1),
                      a & low)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x, y, z, w


def _unit(word):
    return (word >> np.uint64(8)).astype(np.float64) / (1 << 24)


def _step64(case, seed, k, pos, vel):
    """Step k of equal-mass particles in float64: stream, shifted cells, rotation about the cell mean."""
    L, a = np.array(_edges(case)), case["a"]
    pos = np.mod(pos + vel * case["dt"], (L * a)[:, None])
    shift = a * (np.array([_unit(w) for w in _philox(k, np.zeros(1, np.uint64), 0, seed)[:3]])[:, 0] - 0.5)
    c = np.floor((pos - shift[:, None]) / a).astype(np.int64) % L[:, None]
    cell = c[0] + L[0] * (c[1] + L[1] * c[2])
    ncell = int(L.prod())
    count = np.maximum(np.bincount(cell, minlength=ncell), 1)
    u = np.array([np.bincount(cell, weights=vel[d], minlength=ncell) / count for d in range(3)])
    q = _philox(k, np.arange(ncell), 1, seed)
    z, phi = 2.0 * _unit(q[0]) - 1.0, 2.0 * np.pi * _unit(q[1])
    rho = np.sqrt(1.0 - z * z)
    n = np.array([rho * np.cos(phi), rho * np.sin(phi), z])[:, cell]
    w = vel - u[:, cell]
    ca, sa = math.cos(math.radians(case["alpha_deg"])), math.sin(math.radians(case["alpha_deg"]))
    along = n * (n * w).sum(axis=0)
    return pos, u[:, cell] + along + ca * (w - along) + sa * np.cross(n, w, axis=0)


def exact(case, seed):
    """Positions and velocities where a pass is a step or two of a small box
    (later, rounding decides which side of a cell face a particle is on, and
    trajectories part); elsewhere the kinetic energy and temperature, which
    the plain collision conserves."""
    kind = case["kind"]
    if kind == "moments":
        s = prepare(case, seed)
        v = s["v"].double()
        m = s["m"].double() if s["m"] is not None else torch.ones(1, dtype=torch.float64, device="cuda")
        p = (v * m).sum(dim=1)
        return torch.cat([p, (m * v * v).sum()[None], torch.zeros(1, dtype=torch.float64, device="cuda")])
    if kind in ("dump", "checkpoint"):
        if case["steps"] > 2 or _count(case) > 200000:
            return None
        pos, vel = (x.astype(np.float64) for x in _thermal(case, seed))
        for k in range(case["steps"]):
            pos, vel = _step64(case, seed + 1, k, pos, vel)
        return dict(pos=pos, vel=vel, step=None)
    if kind == "ensemble":
        n = np.array([b["n"] for b in inputs.ensemble_boxes(case["boxes"], seed=seed + 1,
                                                            edge=(case["edge_lo"], case["edge_hi"]))], np.float64)
        return dict(P=None, E=1.5 * (n - 1.0), T=np.ones(len(n)), step=None)
    if kind == "serve":
        return dict(T=np.ones(case["requests"]), vacf=None, step=None, status=None)
    if case["masses"] or case["conserve_l"]:
        return None
    return dict(step=None, P=None, E=1.5 * (_count(case) - 1.0), T=1.0, vacf=None)
