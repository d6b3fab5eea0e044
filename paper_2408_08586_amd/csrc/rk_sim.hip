// Discrete-time simulation of a job trace through the greedy allocation with
// the reconfiguration-penalty gate (paper Sec. 5.2 "Incorporating
// reconfiguration penalty", Sec. 7.4).  The curves are computed once by the
// caller; a tick is
//   the allocation kernels from the floors of the tick
//   k_sim_step    (one workgroup) closes the tick: reconfiguration count and
//                 cost, progress, completion, what every job holds; then opens
//                 the next one: per-job state (inactive, frozen or free to
//                 move), floors of the frozen jobs, capacity left.
// A round is a function of what it starts from.  Where the next tick starts
// from exactly what the last round started from (nobody arrived, left or
// thawed, and for the loops nobody moved: 185 to 251 of the 720 ticks of the
// 406-job trace), its result is the one at hand, and k_sim_step closes that
// tick as well instead of handing it to the round's kernels (720 ticks: 35.9 ->
// 27.1 ms under the greedy, 73.0 -> 46.3 ms over the nodes, of which one kernel
// launch less per tick is about 2 ms).
// Under the greedy a round for few jobs needs none of this: k_sim_few runs
// whole ticks in one workgroup (rk_allocate.hip).  A simulation of few jobs has
// only such rounds.  One of up to 1,024 jobs has them most of the time: the host
// looks at the counter, and k_sim_few and the launches take turns as the rounds
// get smaller and larger.  Over nodes up to about 1,300 jobs need none of it
// either: k_sim_nodes has nodes and jobs in LDS from tick to tick (rk_nodes.hip).
// The tick counter lives on the device, so every tick is the same sequence of
// launches with the same arguments: the first tick runs eagerly (it also sizes
// the scratch memory), the sequence is then captured once as a HIP graph on a
// stream of the simulation's own and replayed until the counter, which
// k_sim_step also writes to pinned host memory, has reached the last tick.
#include "rk_sim.h"

namespace {

constexpr int SIM_THREADS = 1024;
constexpr uint32_t SIM_BATCH = 4;              // replays between two looks at the tick counter
constexpr uint32_t SIM_FEW_LAUNCHES = 4;       // launches of k_sim_few between two looks (those behind a round for many jobs return at once)
constexpr uint32_t SIM_WAIT_LEAST = 32, SIM_WAIT_MOST = 256;   // ticks as launches after one whose walks were long (the look costs such a tick)
constexpr int H_TICK = 62;                     // word of the context's pinned memory that holds it, and how many jobs the open tick is for

__global__ __launch_bounds__(SIM_THREADS) void k_sim_init(SimArgs A) {
    const uint32_t j = blockIdx.x * SIM_THREADS + threadIdx.x;
    if (j >= A.n_jobs) return;
    A.S.g[j] = 0; A.S.c[j] = 0; A.S.plan[j] = RK_NO_PLAN; A.S.seg[j] = -1; A.S.lvl[j] = 0;
    A.S.owed[j] = 0.0; A.S.done[j] = 0;
    A.held[j] = 0.0; A.progress[j] = 0.0; A.finish[j] = -1.0; A.n_reconf[j] = 0;
    if (j == 0) *A.tick = 0u;
    if (A.at_off) { A.at_off[j] = 0u; if (j == 0) A.at_off[A.n_jobs] = 0u; }   // nobody is anywhere yet
}

// One workgroup, a thread per job (and every SIM_THREADS-th after it): what a thread writes of its jobs only it reads.
// first: there is no tick to close yet.  Bound by the round trips to memory of the per-job words; at 406 jobs it takes
// the place of two kernels, and a tick that needs no round costs one turn of its loop.
__global__ __launch_bounds__(SIM_THREADS) void k_sim_step(SimArgs A, uint32_t first) {
    const uint32_t tid = threadIdx.x;
    uint32_t tick = *A.tick;
    if (tick >= A.n_ticks) return;                            // replays past the last tick have nothing to close
    bool round_needed = first != 0u;                          // the same in all threads
    if (!first && A.at_off) round_needed = sim_placed<SIM_THREADS>(A);
    uint32_t part = 0;
    (void)sim_ticks<SIM_THREADS, true>(A, tick, first != 0u, round_needed, &part);
    if (tid == 0) {
        *A.tick = tick;
        __hip_atomic_store(A.h_tick + 1, part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(A.h_tick, tick, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// A tick's launches as a graph, which has to outlive its replays.
struct TickGraph {
    hipStream_t s;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    explicit TickGraph(hipStream_t stream) : s(stream) {}
    ~TickGraph() {
        if (exec) { (void)hipStreamSynchronize(s); (void)hipGraphExecDestroy(exec); }
        if (graph) (void)hipGraphDestroy(graph);
    }
    TickGraph(const TickGraph &) = delete;
    TickGraph &operator=(const TickGraph &) = delete;
};

}  // namespace

extern "C" int32_t rk_simulate(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                               const rk_alloc_grid *grid, const rk_cluster *cluster, const float *best_thr,
                               const uint32_t *best_plan, const float *curve_thr, const rk_trace *trace,
                               const rk_sim_options *options, const rk_sim_result *result) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if (!table) return rk_fail(ctx, RK_ERR_INVALID_ARG, "table is null");
    if ((rc = rk_check_table(ctx, table, 0, table->n_jobs))) return rc;
    if ((rc = rk_check_grid(ctx, grid))) return rc;
    if (!cluster || !trace || !options || !result) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    const uint32_t J = table->n_jobs;
    if (J == 0 || options->n_ticks == 0) return RK_OK;
    if (!ref_thr || !best_thr || !best_plan || !curve_thr || !trace->arrival || !trace->work || !trace->delta)
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (!(options->dt > 0.0)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "dt must be positive");
    if (options->gate != options->gate) return rk_fail(ctx, RK_ERR_INVALID_ARG, "gate is NaN");
    if (options->policy > 2u)
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "policy must be 0 (greedy round), 1 (Schedule loop) or 2 (Schedule loop over nodes)");
    const rk_nodes *nodes = options->policy == 2u ? options->nodes : nullptr;
    uint64_t cap_parts = 0;
    if (options->policy == 2u) {
        if (!nodes) return rk_fail(ctx, RK_ERR_INVALID_ARG, "policy 2 needs the nodes");
        if (nodes->n_nodes == 0 || nodes->n_nodes > RK_MAX_NODES || nodes->gpus_per_node == 0 ||
            nodes->gpus_per_node > 65535u || nodes->cpus_per_node > 65535u || !(nodes->mem_per_node_gb >= 0.f))
            return rk_fail(ctx, RK_ERR_INVALID_ARG, "nodes: 1..%u nodes of 1..65535 GPUs, at most 65535 CPUs, memory >= 0", RK_MAX_NODES);
        if (grid->cpu_mode != 1u)
            return rk_fail(ctx, RK_ERR_UNSUPPORTED, "the search over nodes needs CPU levels per GPU (cpu_mode 1)");
        cap_parts = (uint64_t)nodes->n_nodes * nodes->gpus_per_node;
        if (cap_parts > (1u << 20)) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 2^20 GPUs on the nodes");
    }
    if (!(cluster->host_mem_gb >= 0.f)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "host_mem_gb negative or NaN");
    if (J > RK_MAX_JOBS_PER_ROUND)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u jobs, the allocation kernels take up to %u", J, RK_MAX_JOBS_PER_ROUND);
    if (table->max_segs_per_job > 32767u) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 32767 segments per job");
    RK_HIP(ctx, hipSetDevice(ctx->device));

    // per-job state in one scratch block, carved by alignment
    const size_t n8 = ((size_t)J * 8 + 255) & ~(size_t)255, n4 = ((size_t)J * 4 + 255) & ~(size_t)255;
    const size_t n1 = ((size_t)J + 255) & ~(size_t)255;
    char *blk;
    if ((rc = rk_scratch(ctx, SL_SIM_STATE, 5 * n8 + 8 * n4 + 2 * n1 + 256, (void **)&blk))) return rc;
    rk_assign *assign;
    if ((rc = rk_scratch(ctx, SL_SIM_ASSIGN, (size_t)J * sizeof(rk_assign) + 16, (void **)&assign))) return rc;
    auto take = [&](size_t bytes) { char *p = blk; blk += bytes; return p; };
    SimArgs A;
    A.tb = table_dev(table); A.grid = grid_dev(grid); A.cl = *cluster; A.n_jobs = J;
    A.arrival = trace->arrival; A.work = trace->work; A.delta = trace->delta;
    A.dt = options->dt; A.gate = options->gate; A.n_ticks = options->n_ticks; A.loop = options->policy != 0u;
    A.h_tick = nullptr;
    A.S.owed = (double *)take(n8);
    double *s_held = (double *)take(n8), *s_prog = (double *)take(n8), *s_fin = (double *)take(n8);
    A.F.cap0 = (unsigned long long *)take(256);
    A.S.g = (uint32_t *)take(n4); A.S.c = (uint32_t *)take(n4); A.S.plan = (uint32_t *)take(n4);
    A.S.seg = (int32_t *)take(n4); A.S.lvl = (uint32_t *)take(n4);
    A.F.gi = (int32_t *)take(n4); A.F.ci = (uint32_t *)take(n4);
    uint32_t *s_nrec = (uint32_t *)take(n4);
    A.S.done = (uint8_t *)take(n1); A.F.state = (uint8_t *)take(n1);
    A.out = *result;
    A.held = result->held ? result->held : s_held;
    A.progress = result->progress ? result->progress : s_prog;
    A.finish = result->finish ? result->finish : s_fin;
    A.n_reconf = result->n_reconf ? result->n_reconf : s_nrec;
    A.assign = assign;

    A.at_off = A.now_off = nullptr; A.at_ent = A.now_ent = nullptr;
    if (nodes) {                                               // two placements: where the jobs are, where they go
        char *pl;
        const size_t off_bytes = (((size_t)J + 1) * 4 + 255) & ~(size_t)255;
        const size_t ent_bytes = ((size_t)cap_parts * sizeof(rk_place_entry) + 255) & ~(size_t)255;
        if ((rc = rk_scratch(ctx, SL_SIM_PLACES, 2 * (off_bytes + ent_bytes), (void **)&pl))) return rc;
        A.at_off = (uint32_t *)pl; A.now_off = (uint32_t *)(pl + off_bytes);
        A.at_ent = (rk_place_entry *)(pl + 2 * off_bytes); A.now_ent = (rk_place_entry *)(pl + 2 * off_bytes + ent_bytes);
    }
    A.tick = reinterpret_cast<uint32_t *>(A.F.cap0 + 4);       // inside the 256-byte capacity block
    A.tick_total = reinterpret_cast<float *>(A.F.cap0 + 5);

    // a simulation that ended in an error may have left work on its way
    if (ctx->sim_failed && ctx->sim_stream) RK_HIP(ctx, hipStreamSynchronize(ctx->sim_stream));
    uint32_t most = 0;                                         // jobs of a round for k_sim_few
    const SimFew few = options->policy == 0u ? rk_sim_few(J, table->max_segs_per_job, grid, cluster, &most) : SIM_NOT_FEW;
    auto launch_few = [&](uint32_t n_launches, bool begin) {
        return rk_launch_sim_few(ctx, A, ref_thr, grid, table->max_segs_per_job, best_thr, best_plan, curve_thr, assign, n_launches, begin,
                                 few == SIM_OFTEN_FEW, most);
    };
    const uint32_t n = options->n_ticks;
    if (few == SIM_ALWAYS_FEW) {                               // whole ticks in one kernel
        ctx->ways[WAY_SIM_FEW]++;
        if ((rc = launch_few((n - 1u) / SIM_FEW_TICKS + 1u, true))) return rc;
        if (n > 1) RK_HIP(ctx, hipStreamSynchronize(ctx->stream));
        return RK_OK;
    }
    void *h_tick;
    RK_HIP(ctx, hipHostGetDevicePointer(&h_tick, ctx->h_pinned + H_TICK, 0));
    A.h_tick = static_cast<uint32_t *>(h_tick);
    if (nodes && rk_sim_nodes_fit(J, nodes)) {                 // the nodes and jobs fit a workgroup's LDS: ticks without launches between them
        ctx->ways[WAY_SIM_NODES]++;
        __atomic_store_n(ctx->h_pinned + H_TICK, 0u, __ATOMIC_RELEASE);    // (not what an earlier simulation ended with)
        k_sim_init<<<(J + SIM_THREADS - 1) / SIM_THREADS, SIM_THREADS, 0, ctx->stream>>>(A);
        RK_CHECK_LAUNCH(ctx, "k_sim_init");
        k_sim_step<<<1, SIM_THREADS, 0, ctx->stream>>>(A, 1u);
        RK_CHECK_LAUNCH(ctx, "k_sim_step");
        if ((rc = rk_launch_sim_nodes(ctx, A, ref_thr, table, grid, nodes, best_thr, best_plan, curve_thr, cap_parts, assign))) return rc;
        if (options->n_ticks > 1) {
            RK_HIP(ctx, hipStreamSynchronize(ctx->stream));
            const uint32_t closed = __atomic_load_n(ctx->h_pinned + H_TICK, __ATOMIC_ACQUIRE);
            if (closed != options->n_ticks) return rk_fail(ctx, RK_ERR_DEVICE, "the simulation ended after %u of %u ticks", closed, options->n_ticks);
        }
        return RK_OK;
    }
    // (of earlier simulations one of a single tick may still run: it can put 1 there, which ends no loop below)
    ctx->sim_failed = true;                                    // until this one has come to its end
    __atomic_store_n(ctx->h_pinned + H_TICK, 0u, __ATOMIC_RELEASE);

    // the simulation's own stream, ordered after what the context's stream holds
    if (!ctx->sim_stream) {
        RK_HIP(ctx, hipStreamCreateWithFlags(&ctx->sim_stream, hipStreamNonBlocking));
        for (hipEvent_t &ev : ctx->sim_ev) RK_HIP(ctx, hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    }
    hipStream_t user = ctx->stream, s = ctx->sim_stream;
    RK_HIP(ctx, hipEventRecord(ctx->sim_ev[0], user));
    RK_HIP(ctx, hipStreamWaitEvent(s, ctx->sim_ev[0], 0));

    auto tick_body = [&]() -> int32_t {
        ctx->stream = s;                                       // the allocation enqueues on the context's stream
        int32_t r;
        if (options->policy == 2u) {                           // ... searching node by node, from where the jobs are
            const rk_job_state held = {A.F.state, A.S.seg, A.S.lvl, nullptr, nullptr};
            r = rk_launch_reschedule_nodes(ctx, ref_thr, table, grid, nodes, best_thr, best_plan, curve_thr, &held, A.at_off,
                                           A.at_ent, cap_parts, assign, A.now_off, A.now_ent, A.tick_total, nullptr);
        } else if (options->policy == 1u) {                    // Algorithm 1's loop from what the jobs hold
            const rk_job_state held = {A.F.state, A.S.seg, A.S.lvl, nullptr, nullptr};
            r = rk_launch_reschedule(ctx, ref_thr, table, grid, cluster, best_thr, best_plan, curve_thr, &held, assign,
                                     A.tick_total, nullptr);
        } else {
            r = rk_launch_allocate(ctx, ref_thr, A.tb, grid, 1, nullptr, nullptr, cluster, 0, J, J,
                                   table->max_segs_per_job, best_thr, best_plan, curve_thr, nullptr, &A.F,
                                   nullptr, assign, A.tick_total);
        }
        ctx->stream = user;
        if (r) return r;
        k_sim_step<<<1, SIM_THREADS, 0, s>>>(A, 0u);
        RK_CHECK_LAUNCH(ctx, "k_sim_step");
        return RK_OK;
    };

    // Ticks as launches, from the open one until there are no more, or (n > 1) k_sim_few can take over: the first one ever
    // eagerly, the others as replays.  closed: ticks closed so far.
    TickGraph ticks(s);
    uint32_t closed = 0, wait = SIM_WAIT_LEAST, wait_for = 0;  // after long walks: launches for so many ticks, until that tick
    auto told = [&](int word) { return __atomic_load_n(ctx->h_pinned + H_TICK + word, __ATOMIC_ACQUIRE); };
    auto few_again = [&]() {                                   // (not back and forth)
        return few == SIM_OFTEN_FEW && closed < n && closed >= wait_for && told(1) <= most - most / 8u;
    };
    auto as_launches = [&]() -> int32_t {
        // Replays go out in batches, one batch ahead of the counter that is read back, never more of them than ticks
        // are left.  A replay past the last tick repeats the last round and changes nothing.
        uint32_t sent = 0, run = 0;                            // rounds enqueued, rounds known to have run
        uint32_t sent_by[2] = {0u, 0u};                        // rounds enqueued when an event was recorded
        int32_t r;
        if (!ticks.exec) {
            if ((r = tick_body())) return r;
            sent = 1;
            if (n == 1) return RK_OK;
            RK_HIP(ctx, hipStreamBeginCapture(s, hipStreamCaptureModeRelaxed));
            r = tick_body();
            const hipError_t e_end = hipStreamEndCapture(s, &ticks.graph);
            if (r) return r;
            if (e_end != hipSuccess) return rk_fail(ctx, RK_ERR_DEVICE, "hipStreamEndCapture: %s", hipGetErrorString(e_end));
            const hipError_t e = hipGraphInstantiate(&ticks.exec, ticks.graph, nullptr, nullptr, 0);
            if (e != hipSuccess) { ticks.exec = nullptr; return rk_fail(ctx, RK_ERR_DEVICE, "simulation graph: %s", hipGetErrorString(e)); }
        }
        const uint32_t from = closed;
        hipError_t e = hipSuccess;
        for (uint32_t b = 0; e == hipSuccess && closed < n && (closed == from || !few_again()); b ^= 1u) {
            const uint32_t before = sent;
            for (uint32_t k = 0; e == hipSuccess && k < SIM_BATCH && sent - run < n - closed; ++k, ++sent) e = hipGraphLaunch(ticks.exec, s);
            if (e == hipSuccess) e = hipEventRecord(ctx->sim_ev[2 + b], s);
            sent_by[b] = sent;
            const uint32_t w = sent > before ? b ^ 1u : b;     // the batch before this one; this one where nothing could be sent
            if (e == hipSuccess) e = hipEventSynchronize(ctx->sim_ev[2 + w]);
            run = sent_by[w] > run ? sent_by[w] : run;
            closed = told(0);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return rk_fail(ctx, RK_ERR_DEVICE, "simulation graph: %s", hipGetErrorString(e));
        closed = told(0);
        return RK_OK;
    };

    bool turn_few = few == SIM_OFTEN_FEW && n > 1;
    if (!turn_few) {
        k_sim_init<<<(J + SIM_THREADS - 1) / SIM_THREADS, SIM_THREADS, 0, s>>>(A);
        RK_CHECK_LAUNCH(ctx, "k_sim_init");
        k_sim_step<<<1, SIM_THREADS, 0, s>>>(A, 1u);
        RK_CHECK_LAUNCH(ctx, "k_sim_step");
    }
    for (bool begin = true; closed < n; begin = false) {
        if (turn_few) {
            const uint32_t from = closed;
            ctx->ways[WAY_SIM_FEW]++;
            ctx->stream = s;
            rc = launch_few(SIM_FEW_LAUNCHES, begin);
            ctx->stream = user;
            if (rc) return rc;
            RK_HIP(ctx, hipStreamSynchronize(s));
            closed = told(0);
            turn_few = closed - from == SIM_FEW_LAUNCHES * SIM_FEW_TICKS;     // nothing came in the way
            if (closed - from > wait) wait = SIM_WAIT_LEAST;
            if (told(1) == SIM_LONG_WALK) { wait_for = closed + wait; wait = wait < SIM_WAIT_MOST ? 2u * wait : wait; turn_few = false; }
            if (closed < n && !turn_few) {
                k_sim_step<<<1, SIM_THREADS, 0, s>>>(A, 1u);   // opens the tick for the launches
                RK_CHECK_LAUNCH(ctx, "k_sim_step");
            }
        } else {
            ctx->ways[WAY_SIM_LAUNCHES]++;
            if ((rc = as_launches())) return rc;
            if (n == 1) break;
            turn_few = few_again();
        }
    }
    RK_HIP(ctx, hipEventRecord(ctx->sim_ev[1], s));
    RK_HIP(ctx, hipStreamWaitEvent(user, ctx->sim_ev[1], 0));
    ctx->sim_failed = false;
    return RK_OK;
}
