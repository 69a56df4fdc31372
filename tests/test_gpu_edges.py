"""Kernels at the sizes where their tiles, remainders and ranges end."""
import numpy as np
import pytest

from paper_2212_11878_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2212_11878_amd import mpcd
    return mpcd


def exact_moments(vel, mass):
    """(sum m v, sum m v^2): each term rounded to the quantum 2^-32, the
    integers added exactly, each total rounded once."""
    def total(term):
        t = np.rint(term * 2.0 ** 32).astype(np.int64)
        hi, lo = int((t >> 32).sum()), int((t & 0xFFFFFFFF).sum())
        return float((hi << 32) + lo) * 2.0 ** -32
    v, m = vel.astype(np.float64), mass.astype(np.float64)
    return [total(m * v[d]) for d in range(3)] + [total(m * (v[0] * v[0] + v[1] * v[1] + v[2] * v[2]))]


@pytest.mark.parametrize("tiles,extra", [(63, 1), (64, 0), (64, 1), (65, -1), (1025, 17)])
def test_moments_over_record_counts(mp, tiles, extra):
    """Bit for bit at particle counts around one fold of the partial records."""
    import torch
    n = tiles * 4096 + extra
    rng = np.random.default_rng(n)
    vel = (rng.normal(size=(3, n)) * 8.0).astype(np.float32)
    mass = rng.uniform(0.01, 200.0, n).astype(np.float32)
    v, m = torch.from_numpy(vel).cuda(), torch.from_numpy(mass).cuda()
    out = torch.zeros(5, dtype=torch.float64, device="cuda")
    rc = mp.mpcd_moments_noalloc(v[0].data_ptr(), v[1].data_ptr(), v[2].data_ptr(), m.data_ptr(), n, out.data_ptr())
    torch.cuda.synchronize()
    assert rc == mp.MPCD_OK
    # (the energy term's FP64 products may be contracted on the device: each
    # then differs by at most one quantum, a few parts in 2^53 of the term)
    got, want = out.cpu().numpy(), exact_moments(vel, mass)
    assert list(got[:3]) == want[:3] and got[4] == 0
    v2 = float((mass.astype(np.float64) * (vel.astype(np.float64) ** 2).sum(axis=0)).sum())
    assert abs(got[3] - want[3]) <= n * 2.0 ** -32 + 4.0 * 2.0 ** -53 * v2


@pytest.mark.parametrize("n", [1, 255, 4096, 9000])
def test_moments_at_the_edges_of_their_fast_range(mp, n):
    """Energies on both sides of 2^18 and velocities and masses on both sides
    of their limits, in multiples of 2^-8 or 2^-4: every product is exact, so
    the sums are those of integers, and each particle out of range counts once."""
    import torch
    rng = np.random.default_rng(n)
    edge = np.array([[32.0, 0, 0], [31.9375, 0, 0], [0, -32.0625, 0], [0, 255.9375, -255.9375], [256.0, 1, 1],
                     [0, 0, -256.0], [-255.9375, 255.9375, 255.9375], [0.0625, -0.0625, 0], [0, 0, 0], [300.0, 2, 3]])
    vel = edge[rng.integers(0, len(edge), n)].T.astype(np.float32)
    mass = np.array([256.0, 256.0625, 2.0 ** -8, 2.0 ** -9, 1.0, 255.9375])[rng.integers(0, 6, n)].astype(np.float32)
    v, m = torch.from_numpy(np.ascontiguousarray(vel)).cuda(), torch.from_numpy(mass).cuda()
    out = torch.zeros(5, dtype=torch.float64, device="cuda")
    rc = mp.mpcd_moments_noalloc(v[0].data_ptr(), v[1].data_ptr(), v[2].data_ptr(), m.data_ptr(), n, out.data_ptr())
    torch.cuda.synchronize()
    assert rc == mp.MPCD_OK
    out_of_range = (np.abs(vel) >= 256.0).any(axis=0) | (mass < 2.0 ** -8) | (mass > 256.0)
    assert list(out.cpu().numpy()) == exact_moments(vel, mass) + [float(out_of_range.sum())]


@pytest.mark.parametrize("L,density", [((60, 60, 61), 8.6), ((100, 90, 91), 8.1)])
def test_observe_over_record_counts(mp, L, density):
    """Boxes on both sides of the reduction's second level: the observables
    are those of the state read back."""
    n = int(density * L[0] * L[1] * L[2])
    pos, vel = inputs.thermal_state(L, n, seed=n)
    with mp.Context() as ctx:
        slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3))
        ctx.set_state(slot, (pos, vel))
        ctx.step(2)
        obs = ctx.observe(slot)
        _, v, _ = ctx.get_state(slot)
    want = exact_moments(v, np.ones(n))
    assert list(obs["P"]) == want[:3]
    assert abs(2.0 * obs["E"] - want[3]) <= n * 2.0 ** -32 + 4.0 * 2.0 ** -53 * want[3]


@pytest.mark.parametrize("L,n,brick,steps,more", [
    ((24, 23, 25), 700, 2, 3, {}),                          # many buckets a tile, most of them nearly empty
    ((9, 8, 7), 6001, 2, 2, dict(unordered=True)),
    ((16, 16, 16), 40960, 8, 0, {}),                        # not yet bucketed: one bucket holds everything
    ((16, 16, 16), 40960, 8, 2, dict(particle_mass=True)),
    ((5, 5, 5), 1, 0, 2, {}),
    ((5, 5, 5), 0, 0, 2, {}),
])
def test_observe_sees_every_particle_once(mp, L, n, brick, steps, more):
    pos, vel = inputs.thermal_state(L, n, seed=n + 1) if n else (np.zeros((3, 0), np.float32),) * 2
    mass = np.ones(n)
    with mp.Context(brick=brick) as ctx:
        slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3, **more))
        ctx.set_state(slot, (pos, vel))
        if "particle_mass" in more:
            mass = np.random.default_rng(5).uniform(0.5, 2.0, n).astype(np.float32)
            ctx.set_mass(slot, mass)
        ctx.step(steps) if steps else None
        obs = ctx.observe(slot)
        _, v, _ = ctx.get_state(slot)
    want = exact_moments(v, mass)
    assert list(obs["P"]) == want[:3] and obs["status"] == 0
    assert abs(2.0 * obs["E"] - want[3]) <= n * 2.0 ** -32 + 4.0 * 2.0 ** -53 * want[3]


@pytest.mark.parametrize("n", [43690, 43691])   # the last state that fits the pinned staging, the first that does not
@pytest.mark.parametrize("binning,more", [(1, {}), (2, {}), (1, dict(particle_mass=True))])
def test_state_round_trip_at_the_staging_limit(mp, n, binning, more):
    L = (17, 16, 16)
    pos, vel = inputs.thermal_state(L, n, seed=n)
    with mp.Context(binning=binning) as ctx:
        slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3, **more))
        ctx.set_state(slot, (pos, vel), 7)
        ctx.step(1)
        p1, v1, step = ctx.get_state(slot)
        assert step == 8
        ctx.set_state(slot, (p1, v1), step)      # from either buffer
        p2, v2, step = ctx.get_state(slot)
        assert step == 8 and np.array_equal(p1, p2) and np.array_equal(v1, v2)
        # a bad value anywhere is refused and changes nothing
        for field, i, value in ((0, 0, -1.0), (2, n - 1, 16.0), (1, n // 2, np.nan), (3, n - 1, np.inf),
                                (5, 0, np.nan)):
            bad = np.concatenate([p1, v1])
            bad[field, i] = value
            with pytest.raises(mp.MPCDError) as e:
                ctx.set_state(slot, (bad[:3], bad[3:]), 3)
            assert e.value.status == mp.MPCD_EINVAL
        p2, v2, step = ctx.get_state(slot)
        assert step == 8 and np.array_equal(p1, p2) and np.array_equal(v1, v2)
        ctx.step(1)
        p3, v3, _ = ctx.get_state(slot)
        ctx.set_state(slot, (p1, v1), 8)
        ctx.step(1)
        p4, v4, _ = ctx.get_state(slot)
        assert np.array_equal(p3, p4) and np.array_equal(v3, v4)


@pytest.mark.parametrize("binning", [1, 2])
def test_graph_blocks_and_single_steps(mp, binning):
    """Calls of fewer steps than a graph holds, of whole graphs and of both,
    with the host reading the box in between, against eager launches."""
    L, n = (12, 11, 10), 13000
    pos, vel = inputs.thermal_state(L, n, seed=8)
    states = []
    for graph in (True, False):
        seen = []
        with mp.Context(binning=binning, use_graph=graph) as ctx:
            slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3, vacf_stride=5))
            ctx.set_state(slot, (pos, vel))
            for steps in (1, 16, 15, 33, 48, 1, 64):
                ctx.step(steps)
                obs = ctx.observe(slot)
                p, v, k = ctx.get_state(slot)
                seen.append((obs["E"], tuple(obs["P"]), tuple(obs["vacf"]), k, p.tobytes(), v.tobytes()))
        states.append(seen)
    assert states[0] == states[1]


@pytest.mark.parametrize("per_brick", [1, 180, 195, 400, 425, 880, 905, 1370, 1390, 1850, 1900])
@pytest.mark.parametrize("more", [{}, dict(unordered=True), dict(particle_mass=True)])
def test_small_grid_shapes_equal_sort(mp, per_brick, more):
    """Brick loads on both sides of every launch shape's capacity (mean plus
    four standard deviations: 256, 512, 1024, 1536, 2048), in a grid of eight
    bricks: the bits of counting-sort binning."""
    from gpu_util import same_particle_set
    L, n = (8, 8, 8), 8 * per_brick
    pos, vel = inputs.thermal_state(L, n, seed=n)
    mass = np.random.default_rng(n).uniform(0.5, 2.0, n).astype(np.float32)
    out = []
    for binning in (mp.MPCD_BIN_ATOMIC, mp.MPCD_BIN_SORT):
        with mp.Context(binning=binning, brick=4) as ctx:
            slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3, **more))
            ctx.set_state(slot, (pos, vel))
            if "particle_mass" in more:
                ctx.set_mass(slot, mass)
            ctx.step(20)
            out.append(ctx.get_state(slot))
    if "unordered" in more:
        assert same_particle_set(out[0][0], out[0][1], out[1][0], out[1][1])
    else:
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_small_bricks_only_while_they_fit(mp):
    """A box alone gets bricks for one step's latency (at most one per CU);
    boxes admitted to a filled batch, or under a memory budget, the density
    rule's; all run to the same bits."""
    L, n = (16, 16, 16), 40960
    pos, vel = inputs.thermal_state(L, n, seed=2)
    desc = mp.make_desc(L, n, init="external", seed=3)
    with mp.Context() as ctx, mp.Context(hbm_budget=1 << 30) as tight:
        slots = [ctx.admit(desc, (pos, vel)) for _ in range(2)]
        slots_tight = [tight.admit(desc, (pos, vel))]
        bricks = [int(np.prod(ctx.observe(s)["brick"])) for s in slots]
        rule = int(np.prod(tight.observe(slots_tight[0])["brick"]))
        assert bricks[0] < rule and 4096 // bricks[0] <= 256 and bricks[1] == rule
        ctx.step(20)
        tight.step(20)
        a, b, c = ctx.get_state(slots[0]), ctx.get_state(slots[1]), tight.get_state(slots_tight[0])
    for x in (b, c):
        assert np.array_equal(a[0], x[0]) and np.array_equal(a[1], x[1])


@pytest.mark.parametrize("scale", [1.0, 32.0, 200.0])
@pytest.mark.parametrize("density", [1, 9, 300])
def test_sort_sums_beyond_their_fast_range(mp, scale, density):
    """Momenta below, around and above 2^10 (the range that counting-sort
    binning sums in FP64): the bits of bricks, which sum integers throughout."""
    L, n = (9, 8, 7), density * 504
    rng = np.random.default_rng(density)
    pos = inputs.thermal_state(L, n, seed=n)[0]
    vel = rng.uniform(-scale, scale, (3, n)).astype(np.float32)
    mass = rng.uniform(min(scale, 30.0), scale + 1.0, n).astype(np.float32)
    out = []
    for binning in (mp.MPCD_BIN_ATOMIC, mp.MPCD_BIN_SORT):
        with mp.Context(binning=binning, brick=2) as ctx:
            slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3, dt=0.003, particle_mass=True))
            ctx.set_state(slot, (pos, vel))
            ctx.set_mass(slot, mass)
            ctx.step(3)
            out.append(ctx.get_state(slot))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("n", [1, 4095, 4097, 70001])
@pytest.mark.parametrize("more", [{}, dict(unordered=True), dict(particle_mass=True)])
def test_bucketed_state_is_the_state(mp, n, more):
    """Bucketing moves whole particles, ids and masses with them, from either
    buffer: the observables of a step, and the state by id, are those of
    counting-sort binning."""
    from gpu_util import same_particle_set
    L = (19, 8, 13)
    pos, vel = inputs.thermal_state(L, n, seed=n)
    mass = np.random.default_rng(n).uniform(0.5, 2.0, n).astype(np.float32)
    out = []
    for binning in (mp.MPCD_BIN_ATOMIC, mp.MPCD_BIN_SORT):
        with mp.Context(binning=binning, brick=4) as ctx:
            slot = ctx.admit(mp.make_desc(L, n, init="external", seed=3, **more))
            seen = []
            for steps in (1, 2):
                ctx.set_state(slot, (pos, vel), 5)
                if "particle_mass" in more:
                    ctx.set_mass(slot, mass)
                ctx.step(steps)
                obs = ctx.observe(slot)
                seen.append((obs["E"], tuple(obs["P"]), ctx.get_state(slot)))
            out.append(seen)
    for a, b in zip(*out):
        assert a[:2] == b[:2]
        if "unordered" in more:
            assert same_particle_set(a[2][0], a[2][1], b[2][0], b[2][1])
        else:
            assert np.array_equal(a[2][0], b[2][0]) and np.array_equal(a[2][1], b[2][1])


@pytest.mark.parametrize("tiles", [1025, 1026, 1030, 1281])
def test_observing_a_large_box_leaves_its_neighbours_alone(mp, tiles):
    """Tile counts whose last run of the first reduction level would hold one
    tile: the record of its sums stays inside the box's own memory."""
    n = 4096 * tiles
    small = mp.make_desc((10, 9, 8), 7000, seed=5)
    with mp.Context(binning=mp.MPCD_BIN_SORT) as ctx, mp.Context(binning=mp.MPCD_BIN_SORT) as alone:
        big = ctx.admit(mp.make_desc((128, 128, 64), n, seed=2, unordered=True))
        slots = [ctx.admit(small) for _ in range(4)]
        one = alone.admit(small)
        for _ in range(3):
            ctx.step(1)
            alone.step(1)
            assert abs(ctx.observe(big)["T"] - 1.0) < 1e-6
        _, want_v, _ = alone.get_state(one)
        for slot in slots:
            assert np.array_equal(ctx.get_state(slot)[1], want_v)
