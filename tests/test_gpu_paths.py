"""GPU parity of the kernels' rarer paths against the CPU oracle: pools that
spill and waves that hand over (bank schedule), stacks that leave LDS and time
grids that are not uniform (both seedings), generators of every size, distances
below the refined quotients' range, rows of uniforms that start inside lines,
and automatic work units.  Integer tallies and bits throughout, so every
comparison is exact."""
import math
import sys

import numpy as np
import pytest

import workloads as W
from helpers import diag_dict, raw_ints, u64_np

pytestmark = pytest.mark.gpu
LCG = W.Lcg()


def say(*a):
    print("[gpu]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def M():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    import paper_2403_06362_amd as M
    M.lib()
    return M


@pytest.fixture(scope="module")
def ctx(M):
    c = M.Context(0)
    yield c
    c.close()


def slab(M, ctx, probs, lcg=LCG, **opts):
    import torch
    raw, flux, diag = M.transport(probs, lcg, ctx=ctx, opts=M.make_opts(**opts))
    torch.cuda.synchronize()
    return raw_ints(raw), flux.cpu().numpy(), diag_dict(diag, M.DIAG_NAMES)


def pulse(M, ctx, prob, lcg=LCG, **opts):
    import torch
    counts, flux, diag = M.pulse(prob, lcg, ctx=ctx, opts=M.make_pulse_opts(**opts))
    torch.cuda.synchronize()
    return u64_np(counts).reshape(prob.n_batches, -1), dict(zip(M.PULSE_DIAG_NAMES, (int(v) for v in u64_np(diag))))


GROWING = W.pulse(W.hash_seeding(), n_batches=3, per_batch=90).with_(time_edges=np.arange(31, dtype=np.float64))
WIDE = W.pulse(W.hash_seeding(), n_batches=2, per_batch=50).with_(
    nu=13.5, scatter=0.3, time_edges=np.array([0.0, 0.5, 1.0, 1.5]))


@pytest.mark.parametrize("prob", [GROWING, WIDE], ids=["growing", "wide"])
@pytest.mark.parametrize("private,budget,tail", [(1024, 0, 1), (0, 0, 32), (64, 1, 32), (0, 1, 1), (128, 500, 100000)])
def test_pool_spills_and_hand_over(M, ctx, orc, monkeypatch, prob, private, budget, tail):
    """Every place a full pool's particles go: the private stack, the output
    bank, a hand-over of all a wave holds (with items not taken yet), after one
    iteration or never."""
    monkeypatch.setenv("MCRNG_PULSE_PRIVATE", str(private))
    monkeypatch.setenv("MCRNG_PULSE_TAIL", str(tail))
    if budget:
        monkeypatch.setenv("MCRNG_PULSE_BUDGET", str(budget))
    ref = orc.pulse(prob, LCG, threads=8)
    say("pool", prob.nu, private, budget, tail)
    c, d = pulse(M, ctx, prob, schedule=M.PULSE_BANK)
    assert np.array_equal(c, ref.counts) and d == ref.diag


@pytest.mark.parametrize("budget,private", [(1, 0), (3000, 64)])
def test_pool_many_ranges_handed_back(M, ctx, orc, monkeypatch, budget, private):
    """Every wave hands back the rest of its share at its first full pool: the
    next launch takes thousands of ranges of sources, or of census copies."""
    import torch
    monkeypatch.setenv("MCRNG_PULSE_PRIVATE", str(private))
    monkeypatch.setenv("MCRNG_PULSE_BUDGET", str(budget))
    p = W.pulse(W.hash_seeding(), n_batches=211, per_batch=1003)
    ref = orc.pulse(p, LCG, threads=8)
    say("ranges of sources", budget, private)
    c, d = pulse(M, ctx, p)
    assert np.array_equal(c, ref.counts) and d == ref.diag
    p = W.pulse_pc(n_batches=300, per_batch=1000, census_every=8)
    ref = orc.pulse_pc(p, LCG, threads=8)
    say("ranges of copies", budget, private)
    counts, flux, diag, pop = M.pulse_pc(p, LCG, ctx=ctx)
    torch.cuda.synchronize()
    assert np.array_equal(u64_np(counts).reshape(p.n_batches, -1), ref.counts)
    assert np.array_equal(u64_np(pop.contiguous()).reshape(ref.pop.shape), ref.pop)
    assert dict(zip(M.PULSE_DIAG_NAMES, (int(v) for v in u64_np(diag)))) == ref.diag


@pytest.mark.parametrize("budget,tail", [(0, 1), (1, 32), (300, 3)])
def test_pool_hand_over_with_population_control(M, ctx, orc, monkeypatch, budget, tail):
    """Census arrivals past their budget end a launch too; copies and sources
    not taken by then are taken by a later launch."""
    import torch
    monkeypatch.setenv("MCRNG_PULSE_TAIL", str(tail))
    if budget:
        monkeypatch.setenv("MCRNG_PULSE_BUDGET", str(budget))
    p = W.pulse_pc(n_batches=40, per_batch=300, census_every=4)
    ref = orc.pulse_pc(p, LCG, threads=8)
    say("pool with population control", budget, tail)
    counts, flux, diag, pop = M.pulse_pc(p, LCG, ctx=ctx)
    torch.cuda.synchronize()
    assert np.array_equal(u64_np(counts).reshape(p.n_batches, -1), ref.counts)
    assert np.array_equal(u64_np(pop.contiguous()).reshape(ref.pop.shape), ref.pop)
    assert dict(zip(M.PULSE_DIAG_NAMES, (int(v) for v in u64_np(diag)))) == ref.diag


@pytest.mark.parametrize("kind", ["hash", "stride"])
@pytest.mark.parametrize("edges", [np.array([0.0, 1.0]), np.array([0.5, 0.75, 7.0, 7.125, 12.0]),
                                   np.linspace(2.0, 9.0, 600), np.array([0.0, 0.9, 2.1, 3.0, 4.2, 5.0]) * 3.0],
                         ids=["one", "uneven", "many", "nearly-uniform"])
def test_pulse_time_grids(M, ctx, orc, kind, edges):
    """One bin, bins of very different widths, more bins than are staged in
    LDS, edges off a uniform grid by up to a fifth of a bin; a first edge
    after the pulse."""
    sd = W.hash_seeding() if kind == "hash" else W.stride_seeding()
    p = W.pulse(sd, n_batches=31, per_batch=70).with_(time_edges=edges)
    ref = orc.pulse(p, LCG, threads=8)
    say("time grid", kind, len(edges))
    for block in (64, 256):
        c, d = pulse(M, ctx, p, block=block)
        assert np.array_equal(c, ref.counts) and d == ref.diag, block


@pytest.mark.parametrize("nu", [0.7, 1.0, 1.6, 3.0])
def test_stride_multiplicities(M, ctx, orc, nu):
    """At most one particle, exactly one, one or two, always three emerging:
    lines without siblings and stacks deeper than their LDS part."""
    p = W.pulse(W.stride_seeding(), n_batches=9, per_batch=64).with_(
        nu=nu, scatter=min(0.95, 1.1 / nu), time_edges=np.arange(16, dtype=np.float64))
    ref = orc.pulse(p, LCG, threads=8)
    say("stride multiplicity", nu)
    c, d = pulse(M, ctx, p)
    assert np.array_equal(c, ref.counts) and d == ref.diag


@pytest.mark.parametrize("m", [53, 60, 64])
def test_generator_sizes(M, ctx, orc, m):
    """Top-aligned states of generators of 53, 60 and 64 bits: slab in both
    precisions and seedings, pulse in both seedings, uniforms."""
    import torch
    lcg = W.Lcg(m=m)
    for kind in ("hash", "stride"):
        sd = W.hash_seeding() if kind == "hash" else W.stride_seeding()
        p = W.homogeneous(10.0, 1.3, 0.9, 11, 3001, sd, n_batches=2)
        for precision in (0, 1):
            say("generator", m, kind, precision)
            ref = orc.transport(p, lcg, float_mode=bool(precision), threads=8)
            raw, _, diag = slab(M, ctx, [p], lcg, precision=precision)
            assert raw == ref.raw and diag[0] == ref.diag
        q = W.pulse(sd, n_batches=3, per_batch=100)
        ref = orc.pulse(q, lcg, threads=8)
        c, d = pulse(M, ctx, q, lcg)
        assert np.array_equal(c, ref.counts) and d == ref.diag
        u = torch.empty((5, 1003), dtype=torch.float64, device="cuda:0")
        M.uniforms(lcg, sd, u)
        torch.cuda.synchronize()
        assert np.array_equal(u.cpu().numpy(), orc.uniforms(lcg, sd, 1003, 5))


@pytest.mark.parametrize("c", [0.0, 2.0 ** -53, 0.5, 1.0 - 2.0 ** -53, 1.0])
def test_absorption_bounds(M, ctx, orc, c):
    """The absorption test as an integer bound, at its ends."""
    p = W.homogeneous(3.0, 1.0, c, 7, 4001, W.hash_seeding())
    ref = orc.transport(p, LCG, threads=8)
    say("absorption", c)
    raw, _, diag = slab(M, ctx, [p])
    assert raw == ref.raw and diag[0] == ref.diag


@pytest.mark.parametrize("precision,width", [(0, 1e-213), (1, 1e-10), (1, 3e-30)])
@pytest.mark.parametrize("regions", [1, 2])
def test_distances_below_the_quotients_range(M, ctx, orc, precision, width, regions):
    """Cells so thin that flight distances lie below the range of the refined
    quotients (2^-700, single 2^-36): plain divisions, the oracle's bits."""
    p = W.homogeneous(1.0, 1.0, 0.9, 8, 2003, W.hash_seeding())
    edges = np.linspace(0.0, width, 9)
    re = edges[[0, 8]] if regions == 1 else edges[[0, 4, 8]]
    p = p.with_(region_edges=re, sigma_t=np.full(regions, 1.5), scatter=np.full(regions, 0.9), bin_edges=edges)
    ref = orc.transport(p, LCG, float_mode=bool(precision), threads=8)
    say("thin cells", precision, width, regions)
    raw, _, diag = slab(M, ctx, [p], precision=precision)
    assert raw == ref.raw and diag[0] == ref.diag


def test_automatic_units_of_sets(M, ctx, orc):
    """Problems of very different sizes and costs in one set, one of them of no
    histories, steady and time-dependent, one and several regions: scheduled by
    expected time, reduced in one launch."""
    probs = [W.homogeneous(20.0, 1.0, 0.99, 40, 30_011, W.hash_seeding(group_key=1), n_batches=3),
             W.homogeneous(2.0, 0.5, 0.3, 9, 5, W.hash_seeding(group_key=2)),
             W.homogeneous(5.0, 2.0, 0.5, 200, 0, W.stride_seeding()),
             W.multi_region(n_histories=9_001, n_space_bins=8, n_time_bins=4)]
    say("automatic units")
    raw, _, diag = slab(M, ctx, probs)
    off = 0
    for p, d in zip(probs, diag):
        ref = orc.transport(p, LCG, threads=8)
        n = len(ref.raw)
        assert raw[off:off + n] == ref.raw and d == ref.diag
        off += n


@pytest.mark.parametrize("mode", ["hash", "stride", "load"])
@pytest.mark.parametrize("n,k", [(1_000_003, 3), (3_000_017, 17), (65_537, 800)])
def test_uniforms_rows_inside_lines(M, orc, mode, n, k):
    """Rows that start inside a 128-byte line, below and above the size where
    they are stored by runs; final states."""
    import torch
    sd = W.hash_seeding(5) if mode == "hash" else W.stride_seeding(5)
    st = torch.empty(n, dtype=torch.uint64, device="cuda:0")
    u = torch.empty((k, n), dtype=torch.float64, device="cuda:0")
    u.fill_(-1.0)
    say("uniforms rows", mode, n, k)
    if mode == "load":
        M.init_streams(LCG, sd, n, st)
    M.uniforms(LCG, None if mode == "load" else sd, u, st)
    torch.cuda.synchronize()
    assert float(u.min()) > 0.0 and float(u.max()) <= 1.0
    idx = np.concatenate([np.arange(40), np.arange(1000, 1050), np.arange(n - 40, n),
                          np.random.default_rng(3).integers(0, n, 150)])
    got = u[:, torch.from_numpy(idx).to("cuda:0")].cpu().numpy()
    end = u64_np(st)
    for c, i in enumerate(idx):
        one = W.hash_seeding(5 + int(i)) if mode == "hash" else W.stride_seeding(5 + int(i))
        assert np.array_equal(got[:, c], orc.uniforms(LCG, one, 1, k)[:, 0]), i
        x = orc.stream_start(LCG, one, 0)
        if c < 5:
            for _ in range(k):
                x = (LCG.g * x + LCG.c) % (1 << 63)
            assert int(end[i]) == x


@pytest.mark.parametrize("block", [256, 1024])
@pytest.mark.parametrize("bins", [50, 200, 400, 512])
def test_pulse_tally_rows(M, ctx, orc, bins, block):
    """Counters that are not in LDS, in 4 and 2 tally rows per wave, and in as
    many as the largest block has LDS for: hash and stride seeding, population
    control."""
    import torch
    edges = np.linspace(0.0, 12.0, bins + 1)
    n_batches = 1024 // bins + 2
    for kind in ("hash", "stride"):
        sd = W.hash_seeding() if kind == "hash" else W.stride_seeding()
        p = W.pulse(sd, n_batches=n_batches, per_batch=45).with_(time_edges=edges)
        ref = orc.pulse(p, LCG, threads=8)
        say("tally rows", kind, bins, block)
        c, d = pulse(M, ctx, p, block=block)
        assert np.array_equal(c, ref.counts) and d == ref.diag
    p = W.pulse_pc(n_batches=n_batches, per_batch=45, census_every=bins // 3).with_(time_edges=edges)
    ref = orc.pulse_pc(p, LCG, threads=8)
    say("tally rows, population control", bins, block)
    counts, flux, diag, pop = M.pulse_pc(p, LCG, ctx=ctx, opts=M.make_pulse_opts(block=block))
    torch.cuda.synchronize()
    assert np.array_equal(u64_np(counts).reshape(p.n_batches, -1), ref.counts)
    assert np.array_equal(u64_np(pop.contiguous()).reshape(ref.pop.shape), ref.pop)
    assert dict(zip(M.PULSE_DIAG_NAMES, (int(v) for v in u64_np(diag)))) == ref.diag


ONE_BIN = lambda bins: np.concatenate([[0.0], np.linspace(19.0, 20.0, bins)])   # all but a few collisions in bin 0


@pytest.mark.parametrize("n_batches,bins", [(1, 600), (3, 682), (4, 512), (4, 600), (20, 300), (129, 17)])
def test_pulse_counters_beyond_lds(M, ctx, orc, n_batches, bins):
    """About as many counters as LDS holds and more, with and without rows, few
    batches and more, the lanes of a wave in one counter or in many."""
    for kind in ("hash", "stride"):
        for spread in (False, True):
            sd = W.hash_seeding() if kind == "hash" else W.stride_seeding()
            p = W.pulse(sd, n_batches=n_batches, per_batch=900 // n_batches + 1)
            p = p.with_(time_edges=np.linspace(0.0, 20.0, bins + 1) if spread else ONE_BIN(bins), x_lo=-30.0, x_hi=30.0)
            ref = orc.pulse(p, LCG, threads=8)
            say("counters", n_batches, bins, kind, spread)
            c, d = pulse(M, ctx, p)
            assert np.array_equal(c, ref.counts) and d == ref.diag


@pytest.mark.parametrize("n_batches", [1, 4])
def test_pulse_counts_in_one_bin_do_not_queue(M, ctx, n_batches):
    """A run whose collisions nearly all fall into one of 600 bins against the
    same run with none of them scored: 9e5 wave flights of at most four atomics
    per batch, 10 ns each, at most double it; an atomic per collision on one
    address takes 11 to 36 times as long."""
    ms = {}
    for scored in (False, True):
        p = W.pulse(W.hash_seeding(), n_batches=n_batches, per_batch=800_000 // n_batches)
        p = p.with_(time_edges=ONE_BIN(600), x_lo=-50.0 if scored else 1000.0, x_hi=50.0 if scored else 1001.0)
        say("one bin", n_batches, scored)
        t = []
        for _ in range(3):
            pulse(M, ctx, p)
            t.append(ctx.last_run_ms())
        ms[scored] = min(t)
    say(ms)
    assert ms[True] < 4 * ms[False]


@pytest.mark.parametrize("precision,kernel", [(0, "k_transport"), (1, "k_transport_chain")])
def test_timed_runs_with_large_units(M, ctx, orc, monkeypatch, precision, kernel):
    """Time-dependent runs with units large enough for the chained kernel: FP64
    ones stay on the per-unit kernel, which has more waves per SIMD; both give
    the oracle's bits."""
    p = W.multi_region(n_histories=30_011, n_space_bins=20, n_time_bins=20)
    ref = orc.transport(p, LCG, float_mode=bool(precision), threads=8)
    say("timed, large units", precision)
    raw, _, diag = slab(M, ctx, [p], precision=precision, unit_histories=5120)
    assert ctx.last_run_kernel() == kernel
    assert raw == ref.raw and diag[0] == ref.diag
    monkeypatch.setenv("MCRNG_TRANSPORT_CHAIN", "2")
    raw, _, diag = slab(M, ctx, [p], precision=precision, unit_histories=5120)
    assert ctx.last_run_kernel() == "k_transport_chain"
    assert raw == ref.raw and diag[0] == ref.diag


@pytest.mark.parametrize("c,kernel", [(0.5, "k_transport"), (0.99, "k_transport_chain")])
def test_automatic_units_choose_the_kernel(M, ctx, monkeypatch, c, kernel):
    """A large run of one problem: long histories are chained, short ones run
    per unit; the other kernel gives the same bits."""
    p = W.homogeneous(30.0, 1.0, c, 100, 20_000_000, n_batches=2)
    say("automatic units", c)
    raw, flux, diag = slab(M, ctx, [p])
    assert ctx.last_run_kernel() == kernel
    monkeypatch.setenv("MCRNG_TRANSPORT_CHAIN", "0" if kernel == "k_transport_chain" else "2")
    other = slab(M, ctx, [p])
    assert ctx.last_run_kernel() != kernel
    assert other[0] == raw and other[2] == diag and np.array_equal(other[1], flux)


def test_pool_buffers_of_a_small_run(M):
    """A new context's first run of 4096 sources: at most 4096 waves, each with
    a private stack of 1024 entries and, in one full and one smaller bank, room
    for 1408, 32 bytes each and a quarter more: 525 MiB."""
    import torch
    p = W.pulse(W.hash_seeding(), n_batches=1, per_batch=4096)
    counts = torch.empty((1, 20), dtype=torch.uint64, device="cuda:0")
    pulse(M, M.Context(0), p)   # code objects and tables of the process
    torch.cuda.synchronize()
    c = M.Context(0)
    before = torch.cuda.mem_get_info()[0]
    say("buffers of a small run")
    c.run_pulse(LCG, p, counts)
    torch.cuda.synchronize()
    used = (before - torch.cuda.mem_get_info()[0]) >> 20
    c.close()
    say(used, "MiB")
    assert used < 600


@pytest.mark.parametrize("div", [0xFFFFFFFF, 1, 2, 3, 4, 16, 64])
def test_event_schedule_finish_points(M, ctx, orc, div):
    """The event schedule's tail, run depth first per lane by a finish launch
    (with its budget per particle and spills to the next generation), switched
    to at every point, never, and at the first shrinking generation of a growing
    population; its census arrivals with population control."""
    import torch
    for p in (W.pulse(W.hash_seeding(), n_batches=8, per_batch=400), W.pulse_few_sources(n_sources=256, t_end=40)):
        ref = orc.pulse(p, LCG, threads=8)
        say("event finish", div, p.n_batches)
        c, d = pulse(M, ctx, p, schedule=M.PULSE_EVENT, finish_div=div)
        assert np.array_equal(c, ref.counts) and d == ref.diag
    p = W.pulse_pc(n_batches=6, per_batch=500, census_every=4, target=700)
    ref = orc.pulse_pc(p, LCG, threads=6)
    say("event finish, population control", div)
    counts, flux, diag, pop = M.pulse_pc(p, LCG, ctx=ctx,
                                         opts=M.make_pulse_opts(schedule=M.PULSE_EVENT, finish_div=div))
    torch.cuda.synchronize()
    assert np.array_equal(u64_np(counts).reshape(p.n_batches, -1), ref.counts)
    assert np.array_equal(u64_np(pop.contiguous()).reshape(ref.pop.shape), ref.pop)
    assert dict(zip(M.PULSE_DIAG_NAMES, (int(v) for v in u64_np(diag)))) == ref.diag


def family_depth(orc, p):
    """Most entries (scatterings with siblings still to start) that a family of
    the stride-seeded problem holds at once."""
    mask = (1 << LCG.m) - 1
    deepest = 0
    for j in range(p.n_sources):
        x = orc.stream_start(LCG, p.seeding, j)

        def draw():
            nonlocal x
            x = (LCG.g * x + LCG.c) & mask
            return ((x >> (LCG.m - 53)) + 1) * 2.0 ** -53

        t, stack = 0.0, []
        while True:
            draw()                                   # direction
            t -= math.log(draw()) / p.sigma_t
            n = 0
            if t < p.time_edges[-1] and draw() < p.scatter:
                n = int(p.nu) + (draw() < p.nu - int(p.nu))
            if n > 1:
                stack.append([t, n - 1])
                deepest = max(deepest, len(stack))
            if n == 0:
                if not stack:
                    break
                t = stack[-1][0]
                stack[-1][1] -= 1
                if stack[-1][1] == 0:
                    stack.pop()
    return deepest


@pytest.mark.parametrize("t_end,n,depth", [(1, 30, 1), (3, 30, 4), (6, 30, 5), (6, 60, 6), (10, 30, 13)])
def test_stride_stack_depths(M, ctx, orc, t_end, n, depth):
    """Families as deep as opts.stack_depth: less than the entries a lane keeps
    in LDS, just as many, one and two more, and many more; one entry less is
    reported."""
    p = W.pulse(W.stride_seeding(), n_batches=1, per_batch=n).with_(time_edges=np.linspace(0.0, t_end, 5))
    assert family_depth(orc, p) == depth
    ref = orc.pulse(p, LCG, threads=4)
    for block in (64, 256):
        for extra in (0, 1, 40):
            say("stride stack", depth, block, extra)
            c, d = pulse(M, ctx, p, block=block, stack_depth=depth + extra)
            assert np.array_equal(c, ref.counts) and d == ref.diag
        if depth > 1:
            with pytest.raises(M.McrngError) as e:
                pulse(M, ctx, p, block=block, stack_depth=depth - 1)
            assert e.value.code == -4


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("space,time", [(50, 100), (20, 250), (4095, 0), (4, 2048)])
def test_slices_that_fill_lds(M, ctx, orc, precision, space, time):
    """Tally slices of which LDS holds one but not the chained kernel's two: with
    automatic units, with units large enough for that kernel, and without
    allocation."""
    import torch
    p = W.homogeneous(6.0, 1.0, 0.7, space, 1503, W.hash_seeding(), n_batches=2)
    if time:
        p = p.with_(time_edges=np.linspace(0.0, 40.0, time + 1))
    ref = orc.transport(p, LCG, float_mode=bool(precision), threads=8)
    for unit in (0, 6000):
        say("large slice", precision, space, time, unit)
        raw, _, diag = slab(M, ctx, [p], precision=precision, unit_histories=unit)
        assert raw == ref.raw and diag[0] == ref.diag
    nb = M.tally_bins([p])
    raw = torch.zeros((nb, 2), dtype=torch.uint64, device="cuda:0")
    flux = torch.zeros(nb, dtype=torch.float64, device="cuda:0")
    M.run_histories_noalloc(LCG, [p], raw, flux, opts=M.make_opts(precision=precision))
    torch.cuda.synchronize()
    assert raw_ints(raw) == ref.raw


@pytest.mark.parametrize("hist_per_lane", [1, 4])
def test_automatic_units_of_large_blocks(M, ctx, hist_per_lane):
    """A small run on large blocks keeps a unit for each of many of them: about
    the time of units of 256 histories (within the 1.3 of neighbouring sizes),
    not the two to three times of a few large ones."""
    p = W.homogeneous(42.0, 1.0, 0.95, 200, 50_000)
    ms = {}
    for unit in (0, 256):
        say("units of large blocks", hist_per_lane, unit)
        t = []
        for _ in range(5):
            slab(M, ctx, [p], block=1024, hist_per_lane=hist_per_lane, unit_histories=unit)
            t.append(ctx.last_run_ms())
        ms[unit] = min(t)
    say(ms)
    assert ms[0] < 1.6 * ms[256]


def test_small_blocks_of_few_flights(M, ctx):
    """Sources of little more than one flight each on 64-thread blocks: about as
    fast as on 256-thread ones (a wave per block costs the ends of four times as
    many blocks on the run's counters, which made it 1.6 times as long)."""
    p = W.pulse(W.hash_seeding(), n_batches=1, per_batch=247_334).with_(
        nu=0.5, scatter=0.5, time_edges=np.linspace(0.0, 5.0, 21))
    ms = {}
    for block in (64, 256):
        say("few flights", block)
        t = []
        for _ in range(10):
            pulse(M, ctx, p, block=block)
            t.append(ctx.last_run_ms())
        ms[block] = min(t)
    say(ms)
    assert ms[64] < 1.25 * ms[256]
