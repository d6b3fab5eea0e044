"""Rounds whose evaluation goes out before the host knows the plan table's size: from the third call of a kind on, the
evaluation makes the table's content itself from what the search left.  The same records, bit for bit, as a context that has
seen nothing before finds them, also after a guess that was wrong."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def eval_ways(ctx):
    """Rounds of the context whose evaluation alone went out ahead, and those of them that it was right for."""
    import ctypes
    import paper_2408_08586_amd as rk
    counts = (ctypes.c_uint32 * 2)()
    assert rk.load_library().rk_ctx_ways_eval(ctx, counts) == 2
    return tuple(counts)


def _workload(seed, jobs, g_max, mu_mask, per_gpu, tiers):
    coef, ints = workloads.draw_jobs(seed, 11, 0, np.arange(jobs), param_buckets=[(1.0, 0.1e9, 70e9)], layer_choices=(12, 24, 32, 48))
    levels = np.array([1, 2, 4, 8, 16], np.uint32) if per_gpu else np.arange(1, 9, dtype=np.uint32)
    gpus = max(8, jobs // 2 // 8 * 8)
    return workloads.Workload("ahead", coef, ints, workloads.Bounds(g_max=g_max, mu_mask=mu_mask),
                              workloads.Grid(levels, int(per_gpu), np.array(tiers, np.float32), 0), workloads.Env(),
                              workloads.Cluster(gpus, 16 * gpus, 256.0 * gpus))


class Call:
    """One of the three entry points that evaluate by themselves, on a context."""

    def __init__(self, wl, kind):
        import torch
        import paper_2408_08586_amd as rk
        self.rk, self.wl, self.kind = rk, wl, kind
        self.jobs, self.grid, self.env = rk.Jobs(wl.coef, wl.ints), rk.make_grid(wl.grid), rk.make_env(wl.env)
        self.bounds, self.cluster = rk.make_bounds(wl.bounds), rk.make_cluster(wl.cluster)
        n = wl.cluster.G // 8
        self.nodes = rk.rk_nodes(n, 8, wl.cluster.C // n, wl.cluster.host_mem_gb / n)
        self.i32 = lambda k: torch.zeros(k, dtype=torch.int32, device="cuda:0")
        self.total = torch.zeros(2, dtype=torch.float32, device="cuda:0")

    def __call__(self, ctx):
        import torch
        rk, wl = self.rk, self.wl
        J, cap = wl.n_jobs, wl.cluster.G
        assign, placed, off, status = rk.new_assign(J), rk.new_assign(J), self.i32(J + 1), self.i32(J)
        entries = rk.new_place_entries(cap)
        if self.kind == "round":
            rk.rk_schedule_round(ctx, self.jobs, self.bounds, self.grid, self.env, self.cluster, assign, self.total)
        elif self.kind == "sla":
            draws = workloads.sla_draws(wl, seed=3, quota_share=0.5)
            zero = np.zeros(J, np.uint32)
            sla = rk.Sla(draws.guaranteed, draws.tenant, draws.quota_g, draws.quota_c, zero + 2, zero, zero,
                         torch.full((J,), 1e-3, device="cuda:0"), device="cuda:0")
            rk.rk_schedule_round_sla(ctx, self.jobs, self.bounds, self.grid, self.env, self.cluster, sla, assign, self.total)
        elif self.kind == "nodes":
            rk.rk_schedule_round_nodes(ctx, self.jobs, self.bounds, self.grid, self.env, self.nodes, self.i32(J) - 1, self.i32(J), assign,
                                       placed, off, entries, cap, self.total)
        elif self.kind == "enumerate":
            self.rk.enumerate_to_table(ctx, self.jobs, self.bounds, "cuda:0")
        elif self.kind == "rounds":                         # two rounds of half the jobs each
            rk.rk_schedule_rounds(ctx, self.jobs, self.bounds, self.grid, self.env, np.array([0, J // 2, J], np.uint32),
                                  [self.cluster, self.cluster], assign, self.total)
        else:                                               # reads the table's triples once more for the splits
            rk.rk_schedule_round_placed(ctx, self.jobs, self.bounds, self.grid, self.env, self.nodes, None, assign, placed, off, entries,
                                        cap, status, self.total, want_result=False)
        rk.rk_sync(ctx)
        return [x.cpu().numpy().tobytes() for x in (assign, placed, off, status, entries, self.total)]


@pytest.mark.parametrize("jobs,kind,per_gpu,tiers", [
    (3, "round", False, (64.0,)),                            # one launch behind the evaluation, four wavefronts per job
    (300, "round", True, (0.0, 64.0, 1024.0)),
    (300, "rounds", True, (64.0,)),
    (257, "placed", True, (64.0, 1024.0)),
    (2500, "round", True, (64.0,)),                          # equal jobs share their search
    (4200, "round", True, (0.0, 64.0)),                      # a wavefront per job
    (4200, "placed", True, (64.0,)),
])
def test_rounds_evaluated_before_their_size_is_known(jobs, kind, per_gpu, tiers):
    import torch
    import paper_2408_08586_amd as rk
    from gpu_harness import ways
    assert torch.cuda.is_available(), "these tests need the GPU"
    kinds = [(64, 1), (64, 1), (64, 1), (64, 1), (200, 7), (200, 7), (64, 1), (200, 7), (200, 7), (200, 7)]
    ctx = rk.rk_create(0)
    for i, (g_max, mu_mask) in enumerate(kinds):
        call = Call(_workload(20 + i, jobs, g_max, mu_mask, per_gpu, tiers), kind)
        got = call(ctx)
        fresh = rk.rk_create(0)
        want = call(fresh)
        rk.rk_destroy(fresh)
        assert got == want, (i, g_max, mu_mask)
    whole = ways(ctx)
    ahead, taken = (np.array(eval_ways(ctx)) + (whole["ahead"], whole["ahead_taken"])).tolist()
    assert taken >= 2 and ahead > taken                     # guesses that were right, and one at least that was refused
    rk.rk_destroy(ctx)


# Sequences on one context whose calls ask for different room: (entry point, CPU levels, g_max) each, all of the same jobs.  The
# second number is how many of them are evaluated ahead without being sent, and rightly so.
SEQUENCES = {
    # the first two size the curves' buffers by the GPU counts there are (10.7 of at most 12 a job), a plain round by 16 a job
    "placed, then plain": ([("placed", 5, 64)] * 4 + [("round", 5, 64)] * 4, 2),
    "levels of service, then plain": ([("sla", 5, 64)] * 4 + [("round", 5, 64)] * 4, 2),
    "over nodes, then plain": ([("nodes", 5, 64)] * 4 + [("round", 5, 64)] * 4, 2),
    "batches, then plain": ([("rounds", 5, 64)] * 4 + [("round", 5, 64)] * 4, 2),
    "enumerations, then plain": ([("enumerate", 5, 64)] * 3 + [("round", 5, 64)] * 4, 0),
    # room for eight levels is room for the GPU counts there are at twelve, and not for 16 a job
    "more levels": ([("round", 8, 64)] * 3 + [("round", 12, 64)] * 2 + [("round", 14, 64)] * 3 + [("round", 8, 64)] * 2, 0),
    "a grid that grows under batches": ([("rounds", 4, 64)] * 3 + [("rounds", 5, 64)] * 2 + [("rounds", 16, 64)] * 3, None),
    # a guess for wide tables that a narrow one, of a kind that takes one launch, comes under
    "wide, then narrow": ([("placed", 5, 512)] * 3 + [("round", 5, 64)] * 3 + [("placed", 5, 512)] + [("round", 5, 64)] * 2, None),
    "every entry point in turn": ([(k, 5, 64) for k in ("placed", "round", "sla", "rounds", "nodes", "round", "round", "placed", "rounds")], None),
}


@pytest.mark.parametrize("jobs", [64, 60])
@pytest.mark.parametrize("name", list(SEQUENCES))
def test_calls_of_several_kinds_on_one_context(name, jobs):
    """What an evaluation ahead has written is what the allocation reads: no buffer grows between the two, whatever the room that
    the calls before left.  Bit for bit what a fresh context finds."""
    import torch
    import paper_2408_08586_amd as rk
    assert torch.cuda.is_available(), "these tests need the GPU"
    calls, right = SEQUENCES[name]
    coef, ints = workloads.draw_jobs(5, 11, 0, np.arange(jobs), param_buckets=[(0.4, 0.1e9, 1.3e9), (0.4, 1.3e9, 13e9), (0.2, 13e9, 70e9)],
                                     layer_choices=(12, 24, 32, 40))
    ctx = rk.rk_create(0)
    want = {}
    for i, kind in enumerate(calls):
        entry, levels, g_max = kind
        wl = workloads.Workload("several", coef, ints, workloads.Bounds(g_max=g_max),
                                workloads.Grid(np.arange(1, levels + 1, dtype=np.uint32), 1, np.array([64.0], np.float32), 0),
                                workloads.Env(), workloads.Cluster(64, 16 * 64, 256.0 * 64))
        call = Call(wl, entry)
        got = call(ctx)
        if kind not in want:
            fresh = rk.rk_create(0)
            want[kind] = call(fresh)
            rk.rk_destroy(fresh)
        assert got == want[kind], (i, kind)
        assert entry == "enumerate" or any(got[0]), (i, kind)
    sent, taken = eval_ways(ctx)
    assert taken <= sent and (right is None or taken == right), (sent, taken)
    rk.rk_destroy(ctx)
