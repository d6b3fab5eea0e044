"""Rounds that one workgroup takes whole (k_round_few): job counts and amounts around the lines that lead there, against
the oracle's greedy on the same drawn curves, record for record.  Values are coarse, so slopes tie exactly."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def drawn_curves(orc, wl, ot, rng):
    n_rows = len(wl.grid.cpu_levels) * len(wl.grid.mem_levels_gb)
    n = ot.n_segments(n_rows)
    g_of = np.concatenate([np.tile(ot.seg_g[ot.seg_off[j]:ot.seg_off[j + 1]], n_rows) for j in range(wl.n_jobs)])
    bt = (g_of ** rng.uniform(0.3, 1.0, n)) * rng.uniform(0.5, 1.5, n)
    bt = np.round(bt * 8) / 8
    bt[rng.uniform(size=n) < 0.15] = 0
    bt = bt.astype(np.float32)
    bp = rng.integers(0, 1000, n).astype(np.uint32)
    bp[bt == 0] = 0xFFFFFFFF
    return bt, bp, orc.curves(ot, wl.grid, bt, bp)[0]


@pytest.mark.parametrize("n_jobs,g_max,most", [(1, 16, 16), (3, 256, 64), (31, 256, 64), (33, 256, 64), (63, 64, 32), (65, 64, 32),
                                               (127, 16, 16), (128, 16, 16), (129, 16, 16)])
@pytest.mark.parametrize("n_cpu,per_gpu", [(1, 1), (5, 1), (16, 0), (17, 1), (33, 0), (64, 1)])
def test_rounds_of_few_jobs(orc, n_jobs, g_max, most, n_cpu, per_gpu):
    import paper_2408_08586_amd as rk
    from gpu_harness import DeviceRun
    rng = np.random.default_rng(1000 * n_jobs + n_cpu)
    base = workloads.tiny()
    kinds = np.array([[96, 1680, 1], [24, 64, 1], [12, 32, 1], [32, 128, 2]], np.uint32)
    ints = kinds[rng.integers(0, len(kinds), n_jobs)]
    ints[0] = kinds[0]
    coef = np.tile(base.coef[:1], (n_jobs, 1))
    coef[:, 16] = rng.uniform(0.5, 4.0, n_jobs).astype(np.float32)
    grid = workloads.Grid(np.arange(1, n_cpu + 1, dtype=np.uint32), per_gpu, np.array([64.0, 256.0], np.float32), 0)
    wl = workloads.Workload("few", coef, ints, workloads.Bounds(g_max=g_max), grid, workloads.Env(), workloads.Cluster(8, 8, 64.0))
    ot = orc.enumerate_plans(wl.ints, wl.bounds)
    assert most // 2 < np.diff(ot.seg_off).max() <= most
    bt, bp, ct = drawn_curves(orc, wl, ot, rng)
    run = DeviceRun(wl)
    run.enumerate()
    d_bt, d_bp, d_ct = run.dev_f32(bt), run.dev_u32(bp), run.dev_f32(ct)
    for G, C, M in ((n_jobs, 3 * n_jobs, 1e9), (4 * n_jobs, 10 ** 6, 1e9), (7, 40, 300.0), (40 * n_jobs, 5 * n_jobs, 1e4), (0, 5, 64.0),
                    (2 ** 20, 2 ** 32 - 1, 1e9)):
        cl = workloads.Cluster(G, C, M)
        e_assign, e_total, _ = orc.greedy(wl.coef[:, 16], ot, wl.grid, cl, bt, bp, ct)
        assign, total = run.allocate(d_bt, d_bp, d_ct, cluster=rk.make_cluster(cl))
        assert np.array_equal(assign, e_assign), (G, C, M)
        assert total == pytest.approx(e_total, rel=1e-6, abs=1e-12)
    run.close()


@pytest.mark.parametrize("n_jobs,n_ticks", [(1, 1), (2, 129), (300, 127), (300, 128), (700, 257), (1024, 40), (1025, 40)])
@pytest.mark.parametrize("scarce", [False, True])
def test_ticks_in_one_launch(orc, n_jobs, n_ticks, scarce):
    """k_sim_few: job counts whose walks lie in LDS and beyond, ticks around the end of a launch, memory decided in job
    order.  Nearly everybody queues."""
    from gpu_harness import DeviceRun
    from test_gpu_sim import run_on_gpu, same
    base = workloads.trace_scale()
    coef, ints = np.resize(base.coef, (n_jobs, base.coef.shape[1])), np.resize(base.ints, (n_jobs, base.ints.shape[1]))
    grid = workloads.Grid(np.array([1, 2, 4, 8, 16], np.uint32), 1, np.array([64.0, 256.0], np.float32), 0)
    cluster = workloads.Cluster(24 if scarce else 96, 100 if scarce else 2000, 700.0 if scarce else 1e6)
    wl = workloads.Workload("few", coef, ints, base.bounds, grid, base.env, cluster)
    r = orc.schedule_round(wl, n_threads=16)
    rng = np.random.default_rng(n_jobs)
    arrival = np.sort(rng.uniform(0.0, 60.0 * n_ticks * 0.3, n_jobs))
    arrival[: 1 + n_jobs // 2] = 0.0
    work = coef[:, 16] * rng.uniform(60.0, 4000.0, n_jobs)
    delta = rng.uniform(0.0, 90.0, n_jobs)
    run = DeviceRun(wl)
    run.enumerate()
    assert np.diff(run.table_numpy()["seg_off"].astype(np.int64)).max() <= 16
    want = orc.simulator.simulate(coef[:, 16], r["table"], grid, cluster, r["best_thr"], r["best_plan"], r["curve_thr"], arrival, work,
                                  delta, 60.0, n_ticks, gate=0.9)
    same(run_on_gpu(run, r, arrival, work, delta, 60.0, n_ticks, 0.9), want)
    run.close()


def long_walks(orc, n_jobs, kind, g_max, n_cpu, per_gpu, rng):
    """Curves that gain at every amount and every CPU level, less and less: walks as long as they can be."""
    ot = orc.enumerate_plans(np.repeat(np.array([kind], np.uint32), n_jobs, axis=0), workloads.Bounds(g_max=g_max))
    g = ot.seg_g[:ot.seg_off[1]].astype(np.float64)[None, None, :]
    c = np.arange(1, n_cpu + 1)[None, :, None]
    a, b = rng.uniform(0.5, 0.9, (n_jobs, 1, 1)), rng.uniform(0.5, 0.9, (n_jobs, 1, 1))
    bt = (g ** a * (1 + 0.05 * c ** b)).astype(np.float32).reshape(-1)
    grid = workloads.Grid(np.arange(1, n_cpu + 1, dtype=np.uint32), per_gpu, np.array([64.0], np.float32), 0)
    return ot, grid, bt, np.ones(bt.size, np.uint32)


# n_jobs, kind of job, g_max, GPU counts per job, CPU levels, per GPU, GPUs per job of the cluster, ways: k_sim_few, launches
TURNS = [(320, (96, 1680, 1), 16, 16, 5, 1, 1.0, "f"), (321, (96, 1680, 1), 16, 16, 5, 1, 0.25, "fl"), (128, (96, 1680, 1), 64, 32, 5, 1, 2.0, "f"),
         (129, (96, 1680, 1), 64, 32, 16, 0, 1.0, "fl"), (64, (96, 1680, 1), 256, 64, 16, 0, 8.0, "f"), (65, (96, 1680, 1), 256, 64, 17, 0, 8.0, "fl"),
         (256, (96, 1680, 1), 16, 16, 64, 0, 8.0, "fl"), (64, (96, 1680, 1), 64, 32, 64, 0, 8.0, "fl"), (30, (96, 1680, 1), 256, 64, 33, 0, 0.4, "f"),
         (700, (96, 1680, 1), 16, 16, 33, 0, 0.5, "fl"), (1024, (96, 1680, 1), 16, 16, 5, 1, 0.5, "fl"), (1025, (96, 1680, 1), 16, 16, 5, 1, 0.5, "l"),
         (40, (96, 50400, 1), 512, 128, 5, 1, 4.0, "l")]


@pytest.mark.parametrize("n_jobs,kind,g_max,counts,n_cpu,per_gpu,gpus,ways_want", TURNS)
@pytest.mark.parametrize("thaw", [False, True])
def test_ticks_take_turns(orc, n_jobs, kind, g_max, counts, n_cpu, per_gpu, gpus, ways_want, thaw):
    """Simulations around the lines between k_sim_few and ticks as launches: 16, 32, 64 lanes per job in either pass, per-lane
    words in LDS and beyond.  All jobs come at the start, of more than 400 a quarter later, so that rounds get small, and large
    again; thaw: nobody is ever frozen."""
    from gpu_harness import DeviceRun, ways
    from test_gpu_sim import run_on_gpu, same
    rng = np.random.default_rng(n_jobs + n_cpu)
    ot, grid, bt, bp = long_walks(orc, n_jobs, kind, g_max, n_cpu, per_gpu, rng)
    assert counts // 2 < np.diff(ot.seg_off).max() <= counts
    base = workloads.tiny()
    coef = np.tile(base.coef[:1], (n_jobs, 1))
    coef[:, 16] = rng.uniform(0.5, 4.0, n_jobs).astype(np.float32)
    G = int(gpus * n_jobs)
    cluster = workloads.Cluster(G, 6 * G if per_gpu else n_cpu * n_jobs // 2, 1e9)
    wl = workloads.Workload("turns", coef, np.repeat(np.array([kind], np.uint32), n_jobs, axis=0), workloads.Bounds(g_max=g_max), grid,
                            base.env, cluster)
    n_ticks = 90
    arrival = np.where((n_jobs > 400) & (np.arange(n_jobs) % 4 == 0), 60.0 * 60, 0.0)
    work = np.median(bt) * 60.0 * rng.uniform(0.5, 30.0, n_jobs)
    delta = np.zeros(n_jobs) if thaw else rng.uniform(0.0, 90.0, n_jobs)
    want = orc.simulator.simulate(coef[:, 16], ot, grid, cluster, bt, bp, bt, arrival, work, delta, 60.0, n_ticks, gate=0.9)
    run = DeviceRun(wl)
    run.enumerate()
    curves = (run.dev_f32(bt), run.dev_u32(bp), run.dev_f32(bt))
    for _ in range(2):                                          # (the second one finds the first one's working memory)
        same(run_on_gpu(run, None, arrival, work, delta, 60.0, n_ticks, 0.9, curves=curves), want)
    got = ways(run.ctx)
    assert (got["sim_few"] > 0, got["sim_launches"] > 0) == ("f" in ways_want, "l" in ways_want), got
    run.close()


@pytest.mark.parametrize("n_jobs,n_ticks,gpn", [(1, 1, 8), (30, 64, 4), (60, 200, 8), (256, 65, 6), (257, 130, 8), (700, 60, 16), (1600, 20, 8), (1416, 20, 8),
                                                (1417, 20, 8)])
@pytest.mark.parametrize("scarce", [False, True])
def test_ticks_over_nodes_in_one_launch(orc, n_jobs, n_ticks, gpn, scarce):
    """k_sim_nodes: rounds around the end of a launch, one job per thread and more, jobs whose values fit LDS and (1,600 of
    them) do not; jobs that finish, thaw and lose their memory between the rounds."""
    from gpu_harness import DeviceRun, ways
    from test_gpu_sim import run_on_gpu, same
    base = workloads.trace_scale()
    coef, ints = np.resize(base.coef, (n_jobs, base.coef.shape[1])), np.resize(base.ints, (n_jobs, base.ints.shape[1]))
    grid = workloads.Grid(np.array([1, 2, 4, 8, 16], np.uint32), 1, np.array([64.0, 256.0], np.float32), 0)
    n_nodes = 3 if scarce else 10
    nodes = (n_nodes, gpn, (5 if scarce else 16) * gpn, 300.0 if scarce else 4096.0)
    cluster = workloads.Cluster(n_nodes * gpn, n_nodes * nodes[2], n_nodes * nodes[3])
    wl = workloads.Workload("few", coef, ints, base.bounds, grid, base.env, cluster)
    r = orc.schedule_round(wl, n_threads=16)
    rng = np.random.default_rng(n_jobs + n_ticks)
    arrival = np.sort(rng.uniform(0.0, 60.0 * n_ticks * 0.6, n_jobs))
    arrival[: 1 + n_jobs // 4] = 0.0
    work = coef[:, 16] * rng.uniform(60.0, 4000.0, n_jobs)
    delta = rng.uniform(0.0, 90.0, n_jobs)
    run = DeviceRun(wl)
    run.enumerate()
    want = orc.simulator.simulate(coef[:, 16], r["table"], grid, cluster, r["best_thr"], r["best_plan"], r["curve_thr"], arrival, work,
                                  delta, 60.0, n_ticks, gate=0.9, policy="nodes", nodes=nodes)
    for _ in range(2):                                          # (the second one finds the first one's working memory)
        same(run_on_gpu(run, r, arrival, work, delta, 60.0, n_ticks, 0.9, policy=2, nodes=nodes), want)
    got = ways(run.ctx)                                         # (1,416 jobs on 10 nodes of 8 GPUs are the last that fit LDS, 1,421 on 3)
    fits = n_jobs <= (1421 if scarce else 1416)
    assert (got["sim_nodes"], got["sim_launches"]) == ((2, 0) if fits else (0, 2))
    run.close()


@pytest.mark.parametrize("n_jobs,spread", [(511, 0.0), (512, 1.0), (513, 1.0), (1024, 1.0), (1025, 0.3), (2049, 0.0), (2049, 3.0),
                                           (3000, 1.0), (12288, 0.3)])
def test_thresholds_of_many_jobs(orc, n_jobs, spread):
    """Rounds around the lines between 512 and 1,024 threads and one and two jobs a thread, and rounds whose histograms are
    in memory (more than 2,048 jobs): slopes in few bins (spread 0: a handful of values) and
    over many groups of them, capacities that cut in the first group, in the middle, at the last step, and not at all."""
    import paper_2408_08586_amd as rk
    from gpu_harness import DeviceRun
    rng = np.random.default_rng(n_jobs)
    base = workloads.tiny()
    coef = np.tile(base.coef[:1], (n_jobs, 1))
    coef[:, 16] = (2.0 ** np.round(rng.normal(0.0, 4.0 * spread, n_jobs))).astype(np.float32)
    grid = workloads.Grid(np.array([1, 2, 4], np.uint32), 1, np.array([64.0], np.float32), 0)
    wl = workloads.Workload("many", coef, np.tile(np.array([[96, 128, 1]], np.uint32), (n_jobs, 1)), workloads.Bounds(g_max=64), grid,
                            workloads.Env(), workloads.Cluster(8, 8, 64.0))
    ot = orc.enumerate_plans(wl.ints, wl.bounds)
    bt, bp, ct = drawn_curves(orc, wl, ot, rng)
    # half of the jobs gain from every amount, less and less: walks as long as their lists (12 steps)
    n_rows = len(grid.cpu_levels)
    whole = int(ot.seg_off[n_jobs // 2])
    g_of = np.concatenate([np.tile(ot.seg_g[ot.seg_off[j]:ot.seg_off[j + 1]], n_rows) for j in range(n_jobs // 2)])
    bt[:whole * n_rows] = (np.sqrt(g_of) * 4).astype(np.float32)
    bp[:whole * n_rows] = 1
    ct = orc.curves(ot, wl.grid, bt, bp)[0]
    run = DeviceRun(wl)
    run.enumerate()
    d_bt, d_bp, d_ct = run.dev_f32(bt), run.dev_u32(bp), run.dev_f32(ct)
    for G, C in ((0, 0), (1, 1), (n_jobs // 3, 10 ** 7), (2 * n_jobs, 3 * n_jobs), (20 * n_jobs, 10 ** 7), (64 * n_jobs, 64 * n_jobs),
                 (2 ** 31, 2 ** 32 - 1)):
        cl = workloads.Cluster(G, C, 1e9)
        e_assign, e_total, _ = orc.greedy(wl.coef[:, 16], ot, wl.grid, cl, bt, bp, ct)
        assign, total = run.allocate(d_bt, d_bp, d_ct, cluster=rk.make_cluster(cl))
        assert np.array_equal(assign, e_assign), (G, C)
        assert total == pytest.approx(e_total, rel=1e-6, abs=1e-12)
    run.close()


def test_equal_jobs_are_found_again_in_later_calls(orc):
    """The table of equal jobs is left empty by every call for the next one: calls of growing and shrinking size on one
    context, each with kinds of jobs of its own, and one that ends in an error between them."""
    import torch
    import paper_2408_08586_amd as rk
    ctx = rk.rk_create(0)
    bounds = workloads.Bounds(g_max=64)
    for i, n_jobs in enumerate((2048, 5000, 2048, 9000, 0, 3000)):
        rng = np.random.default_rng(i)
        kinds = np.stack([rng.integers(1, 97, 40), rng.integers(1, 200, 40), np.ones(40)], 1).astype(np.uint32)
        ints = kinds[rng.integers(0, 40, max(n_jobs, 2500))]
        jobs = rk.Jobs(np.tile(workloads.tiny().coef[:1], (len(ints), 1)), ints, "cuda:0")
        if n_jobs == 0:                                         # a table without room
            small = rk.PlanTable(len(ints), 8, 8, "cuda:0")
            with pytest.raises(rk.RkError):
                rk.rk_enumerate_plans(ctx, jobs, rk.make_bounds(bounds), small.c)
            continue
        t = rk.enumerate_to_table(ctx, jobs, rk.make_bounds(bounds), "cuda:0")
        ot = orc.enumerate_plans(ints, bounds)
        torch.cuda.synchronize()
        assert np.array_equal(rk.u32(t.seg_off), ot.seg_off) and np.array_equal(rk.u32(t.seg_g)[:t.n_segs], ot.seg_g)
        assert np.array_equal(rk.u32(t.triple_off), ot.triple_off)
    rk.rk_destroy(ctx)


def test_small_rounds_sent_before_their_table_is_known():
    """Rounds on one context whose tables resemble the last two, are larger, smaller, wider than the parked words, in error
    and of the first kind again: every one is what a fresh context makes of it, and a round in error leaves its records
    alone."""
    import torch
    import paper_2408_08586_amd as rk
    from gpu_harness import ways
    ctx = rk.rk_create(0)
    base = workloads.tiny()
    small, wide, wider = np.array([[12, 32, 1]], np.uint32), np.array([[96, 128, 1]], np.uint32), np.array([[96, 1680, 1]], np.uint32)
    bad = np.array([[4095, 720720, 1]], np.uint32)
    plan = [(small, 64)] * 4 + [(wide, 64)] * 3 + [(small, 64)] * 3 + [(wider, 256), (wider, 256), (small, 64), (small, 64), (small, 64),
                                                                       (bad, 65535), (small, 64), (small, 16), (small, 16), (small, 64)]
    for i, (kind, g_max) in enumerate(plan):
        n_jobs = (20, 33, 7, 64)[i % 4]
        rng = np.random.default_rng(i)
        coef = base.coef[rng.integers(0, base.n_jobs, n_jobs)]
        ints = np.repeat(kind, n_jobs, axis=0)
        wl = workloads.Workload("seq", coef, ints, workloads.Bounds(g_max=g_max), base.grid, base.env,
                                workloads.Cluster(3 * n_jobs, 12 * n_jobs, 1e4))
        def on(c):
            assign, total = rk.new_assign(n_jobs, "cuda:0"), torch.full((1,), -1.0, device="cuda:0")
            assign.fill_(77)
            try:
                rk.rk_schedule_round(c, rk.Jobs(coef, ints, "cuda:0"), rk.make_bounds(wl.bounds), rk.make_grid(wl.grid),
                                     rk.make_env(wl.env), rk.make_cluster(wl.cluster), assign, total)
                code = 0
            except rk.RkError as e:
                code = e.code
            rk.rk_sync(c)
            return code, assign.cpu().numpy().copy(), float(total[0])
        got = on(ctx)
        fresh = rk.rk_create(0)
        want = on(fresh)                                       # (a context that has seen no table sends nothing ahead)
        rk.rk_destroy(fresh)
        assert got[0] == want[0] and np.array_equal(got[1], want[1]) and got[2] == want[2], i
        if kind is bad:
            bad_at = ways(ctx)["ahead"]
            assert got[0] == rk.RK_ERR_UNSUPPORTED and (got[1] == 77).all() and got[2] == -1.0
        else:
            assert got[0] == 0 and got[2] > 0
    seen = ways(ctx)
    assert bad_at > 0 and seen["ahead_taken"] >= 4 and seen["ahead"] - seen["ahead_taken"] >= 3      # sent and taken, sent and refused
    rk.rk_destroy(ctx)


def test_a_steady_round_is_sent_ahead_and_its_buffers_stay():
    """Calls of one kind: the first makes the working buffers, none after it does, and from the third on rounds go out before
    their table is known.  A round of another kind after them is refused once and launched again."""
    import torch
    import paper_2408_08586_amd as rk
    from gpu_harness import ways
    ctx = rk.rk_create(0)
    base = workloads.tiny()

    def call(kind, n_jobs, g_max):
        wl = workloads.Workload("steady", np.tile(base.coef[:1], (n_jobs, 1)), np.tile(np.array([kind], np.uint32), (n_jobs, 1)),
                                workloads.Bounds(g_max=g_max), base.grid, base.env, workloads.Cluster(3 * n_jobs, 12 * n_jobs, 1e4))
        assign, total = rk.new_assign(n_jobs, "cuda:0"), torch.zeros(1, device="cuda:0")
        rk.rk_schedule_round(ctx, rk.Jobs(wl.coef, wl.ints, "cuda:0"), rk.make_bounds(wl.bounds), rk.make_grid(wl.grid), rk.make_env(wl.env),
                             rk.make_cluster(wl.cluster), assign, total)
        rk.rk_sync(ctx)
        return ways(ctx)
    kinds = [((12, 32, 1), 60, 64), ((96, 1680, 1), 30, 64), ((96, 1680, 1), 30, 256), ((12, 32, 1), 60, 64)]
    ahead = taken = 0
    for i, kind in enumerate(kinds):
        grew = None
        for k in range(6):
            w = call(*kind)
            ahead += 0 if (i == 0 and k < 2) or (i > 0 and k == 1) else 1       # (the last two calls were of one kind)
            taken += 0 if k < 2 else 1
            assert (w["ahead"], w["ahead_taken"]) == (ahead, taken) or (i > 0 and k == 0), (i, k)
            if i > 0 and k == 0:                                # sent for the kind before, when its buffers had room for these jobs
                assert w["ahead"] in (ahead, ahead - 1) and w["ahead_taken"] == taken
                ahead = w["ahead"]
            assert grew is None or w["grew"] == grew, (i, k)
            grew = w["grew"]
    assert ahead > taken > 0                                    # (one guess at least was refused)
    rk.rk_destroy(ctx)


@pytest.mark.parametrize("n_jobs,n_cpu,gpus,few", [(64, 32, 8.0, True), (128, 32, 8.0, True), (128, 33, 0.5, True), (128, 33, 8.0, False),
                                                   (65, 64, 8.0, False), (64, 64, 8.0, True), (129, 17, 8.0, False)])
def test_rounds_from_descriptors_at_the_cpu_line(orc, n_jobs, n_cpu, gpus, few):
    """Rounds whose jobs may only offload, so that every job that holds GPUs walks all CPU levels, at the most lanes that one
    launch takes and beyond: the records are the oracle's greedy on the device's own curves."""
    import paper_2408_08586_amd as rk
    from gpu_harness import DeviceRun, ways
    coef, ints = workloads.draw_jobs(7, 11, 0, np.arange(n_jobs), param_buckets=[(1.0, 1e9, 4e9)], layer_choices=(12, 24, 32, 40))
    G = int(gpus * n_jobs)
    wl = workloads.Workload("offload", coef, ints, workloads.Bounds(g_max=16 if n_jobs > 64 else 64, off_mask=2),
                            workloads.Grid(np.arange(1, n_cpu + 1, dtype=np.uint32), 0, np.array([64.0, 1024.0], np.float32), 0),
                            workloads.Env(gpu_mem_cap=16e9), workloads.Cluster(G, n_cpu * n_jobs // 3, 3e4))
    run = DeviceRun(wl)
    for _ in range(3):
        assign, total = run.schedule_round()
    assert ways(run.ctx)["ahead_taken"] == (1 if few else 0)    # (what is sent ahead takes the one launch)
    run.enumerate()
    bt, bp, ct, _, _, n = run.fused()
    ot = orc.enumerate_plans(wl.ints, wl.bounds)
    assert np.diff(ot.seg_off.astype(np.int64)).max() <= 16
    want, want_total, _ = orc.greedy(coef[:, 16], ot, wl.grid, wl.cluster, run.host(bt, n), run.host(bp, n).view(np.uint32), run.host(ct, n))
    assert np.array_equal(assign, want) and total == pytest.approx(want_total, rel=1e-6)
    assert (want["g"] > 0).sum() > 4 and want["c"].max() == n_cpu
    run.close()
