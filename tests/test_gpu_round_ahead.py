"""Rounds whose evaluation goes out before the host knows the plan table's size: from the third call of a kind on, the
evaluation makes the table's content itself from what the search left.  The same records, bit for bit, as a context that has
seen nothing before finds them, also after a guess that was wrong."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


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
        rk, wl = self.rk, self.wl
        J, cap = wl.n_jobs, wl.cluster.G
        assign, placed, off, status = rk.new_assign(J), rk.new_assign(J), self.i32(J + 1), self.i32(J)
        entries = rk.new_place_entries(cap)
        if self.kind == "round":
            rk.rk_schedule_round(ctx, self.jobs, self.bounds, self.grid, self.env, self.cluster, assign, self.total)
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
    rk.rk_destroy(ctx)
