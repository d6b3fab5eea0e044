// The state of a simulation and what a tick does to a job, shared by the kernel that closes and opens ticks around the
// rounds of any policy (k_sim_step) and the one that runs whole ticks of the greedy (k_sim_few).
#pragma once
#include "rk_internal.h"
#include "rk_model.h"

constexpr uint32_t SIM_FEW_TICKS = 128;        // ticks of a launch of k_sim_few, at most
constexpr uint32_t SIM_LONG_WALK = 0xFFFFFFFFu;

struct SimState {               // per job, between the ticks
    uint32_t *g, *c, *plan;     // what the job holds (g = 0: nothing)
    int32_t *seg;               // ... as segment index
    uint32_t *lvl;              // ... and CPU level
    double *owed;               // checkpoint-resume seconds still to pay
    uint8_t *done;
};

struct SimArgs {
    TableDev tb;
    GridDev grid;
    rk_cluster cl;
    uint32_t n_jobs, n_ticks;
    uint32_t loop;              // the round starts from what every job holds (policies 1 and 2), not the frozen ones only
    const double *arrival, *work, *delta;
    double dt, gate;
    SimState S;
    FloorsDev F;
    const rk_assign *assign;
    uint32_t *tick;             // device counter: the tick whose round comes next; behind it: a launch of k_sim_few was stopped
    uint32_t *h_tick;           // its copy in pinned host memory (may be null); behind it: how many jobs that round is for, or
                                // (k_sim_few) SIM_LONG_WALK when the last round walked long over the CPU levels
    float *tick_total;          // the allocation's total of the current tick
    rk_sim_result out;
    double *held;               // result arrays or scratch when the caller passes none
    double *progress, *finish;
    uint32_t *n_reconf;
    // the search over nodes only: where the jobs are (left by the last tick) and where this tick puts them
    uint32_t *at_off, *now_off;
    rk_place_entry *at_ent, *now_ent;
};

// What a tick needs of a job and leaves of it.
struct SimJob {
    uint32_t g, c, plan, n_reconf;
    double owed, held, progress, finish;
    bool done;
};

// Closes a tick at t for a job with the record a; true when it holds other amounts than before (nothing: g = 0).
__device__ __forceinline__ bool sim_close(SimJob &s, const rk_assign &a, double t, double dt, double delta, double work) {
    const uint32_t g_prev = s.g;
    uint32_t g = a.g;
    const bool same_amounts = g == g_prev && a.c == s.c;
    if (g_prev > 0 && g > 0 && (!same_amounts || a.plan != s.plan)) {
        s.n_reconf += 1;
        s.owed = s.owed + delta;
    }
    if (g > 0) {
        s.held = s.held + dt;
        const double paid = s.owed < dt ? s.owed : dt;
        s.owed = s.owed - paid;
        const double train = dt - paid;
        const double thr = (double)a.thr;
        const double gain = thr * train;
        if (s.progress + gain >= work) {
            s.finish = t + paid + (work - s.progress) / thr;
            s.progress = work;
            s.done = true;
            g = 0;
        } else {
            s.progress = s.progress + gain;
        }
    }
    s.g = g;
    s.c = g ? a.c : 0u;
    s.plan = g ? a.plan : RK_NO_PLAN;
    return g == 0 ? g_prev != 0 : !same_amounts;
}

// What an active job does in a round that begins now: free to move, or frozen.
__device__ __forceinline__ bool sim_frozen(uint32_t g, double held, uint32_t n_reconf, double delta, double gate) {
    if (g == 0) return false;
    const bool may_move = held - ((double)n_reconf + 1.0) * delta > gate * held;
    return !may_move;
}

// Closes a tick for job j; true when the job holds other amounts than before it.
__device__ __forceinline__ bool commit_job(const SimArgs &A, uint32_t j, double t, uint32_t &g_used) {
    const rk_assign a = A.assign[j];
    g_used += a.g;
    SimJob s = {A.S.g[j], A.S.c[j], A.S.plan[j], A.n_reconf[j], A.S.owed[j], A.held[j], A.progress[j], 0.0, false};
    const uint32_t n_reconf = s.n_reconf;
    const bool moved = sim_close(s, a, t, A.dt, A.delta[j], A.work[j]);
    if (s.n_reconf != n_reconf) A.n_reconf[j] = s.n_reconf;
    if (a.g > 0) {
        A.S.owed[j] = s.owed; A.held[j] = s.held; A.progress[j] = s.progress;
        if (s.done) { A.finish[j] = s.finish; A.S.done[j] = 1; }
    }
    if (s.g > 0) A.S.plan[j] = s.plan;
    if (!moved) return false;
    uint32_t seg = 0xFFFFFFFFu, lvl = 0;
    if (s.g > 0) {
        // segment index of g (the job's counts ascend) and the CPU level that costs a.c
        const uint32_t s0 = A.tb.seg_off[j], ns = A.tb.seg_off[j + 1] - s0;
        uint32_t hi = ns;
        seg = 0;
        while (seg < hi) {
            const uint32_t mid = (seg + hi) >> 1;
            if (A.tb.seg_g[s0 + mid] < s.g) seg = mid + 1; else hi = mid;
        }
        for (uint32_t i = 0; i < A.grid.n_cpu; ++i)
            if (cpus_of(A.grid, i, s.g) == s.c) { lvl = i; break; }
    }
    A.S.g[j] = s.g; A.S.c[j] = s.c; A.S.plan[j] = s.plan; A.S.seg[j] = (int32_t)seg; A.S.lvl[j] = lvl;
    return true;
}

// The placement a tick made becomes where the jobs are when the next tick begins; true: they were somewhere else before.
static_assert(sizeof(rk_place_entry) == sizeof(uint4), "a part is compared and copied as one piece");
template <int THREADS>
__device__ __forceinline__ bool sim_placed(const SimArgs &A) {
    const uint32_t tid = threadIdx.x;
    bool other = false;
    for (uint32_t i = tid; i <= A.n_jobs; i += THREADS) {
        const uint32_t now = A.now_off[i];
        other |= A.at_off[i] != now;
        A.at_off[i] = now;
    }
    const uint32_t n = A.now_off[A.n_jobs];
    const uint4 *now_ent = reinterpret_cast<const uint4 *>(A.now_ent);
    uint4 *at_ent = reinterpret_cast<uint4 *>(A.at_ent);
    for (uint32_t i = tid; i < n; i += THREADS) {
        const uint4 now = now_ent[i], at = at_ent[i];         // (a slot never written compares as it may: at worst a round more)
        other |= at.x != now.x || at.y != now.y || at.z != now.z || at.w != now.w;
        at_ent[i] = now;
    }
    return __syncthreads_or(other) != 0;
}

// A workgroup closes tick `tick`, whose round has run (first: there is none yet), and opens the next one; ticks that start
// from exactly what the last round started from are closed at once.  True: the tick `tick` is open and needs a round
// (round_needed: it does in any case); false: there are no more ticks.  What a thread writes of its jobs only it reads.
// COUNT: thread 0 finds in part how many jobs the round is for, those that are frozen not among them.
template <int THREADS, bool COUNT = false>
__device__ __forceinline__ bool sim_ticks(const SimArgs &A, uint32_t &tick, bool first, bool round_needed, uint32_t *part = nullptr) {
    __shared__ unsigned long long sum_g, sum_c;
    __shared__ uint32_t sum_f, sum_used, moved, sum_p;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    for (;;) {
        if (tid == 0) { sum_g = 0ull; sum_c = 0ull; sum_f = 0u; sum_used = 0u; moved = 0u; if (COUNT) sum_p = 0u; }
        __syncthreads();
        if (!first) {
            const double t = (double)tick * A.dt;
            uint32_t g_used = 0;
            bool other = false;
            for (uint32_t j = tid; j < A.n_jobs; j += THREADS)
                if (A.F.state[j] != RK_JOB_OUT) other |= commit_job(A, j, t, g_used);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) g_used += __shfl_xor(g_used, off, 64);
            if (lane == 0 && g_used) atomicAdd(&sum_used, g_used);
            if (A.loop && __ballot(other) && lane == 0) moved = 1u;
            __syncthreads();
            if (tid == 0) {
                if (A.out.gpus_in_use) A.out.gpus_in_use[tick] = sum_used;
                if (A.out.totals) A.out.totals[tick] = *A.tick_total;
            }
            if (moved) round_needed = true;
            if (++tick == A.n_ticks) return false;
        }
        const double t = (double)tick * A.dt;
        unsigned long long held_g = 0, held_c = 0;
        uint32_t n_frozen = 0, n_part = 0;
        bool other = false;
        for (uint32_t j = tid; j < A.n_jobs; j += THREADS) {
            const bool active = A.arrival[j] <= t && !A.S.done[j];
            const uint32_t g = A.S.g[j];
            uint8_t state = RK_JOB_OUT;
            int32_t gi = -1;
            uint32_t ci = 0;
            if (active) {
                state = RK_JOB_NORMAL;
                if (sim_frozen(g, A.held[j], A.n_reconf[j], A.delta[j], A.gate)) {
                    state = RK_JOB_FROZEN;
                    gi = A.S.seg[j];
                    ci = A.S.lvl[j];
                    held_g += g;
                    held_c += A.grid.cpu_mode ? (unsigned long long)A.grid.cpu_levels[ci] * g
                                              : (unsigned long long)A.grid.cpu_levels[ci];
                    ++n_frozen;
                }
            }
            if (first || A.F.state[j] != state || A.F.gi[j] != gi || A.F.ci[j] != ci) {
                A.F.state[j] = state;
                A.F.gi[j] = gi;
                A.F.ci[j] = ci;
                other = true;
            }
            if (COUNT) n_part += (uint32_t)__popcll(__ballot(state == RK_JOB_NORMAL));    // (lane 0 has every turn of its wavefront)
        }
        if (COUNT && lane == 0 && n_part) atomicAdd(&sum_p, n_part);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            held_g += __shfl_xor(held_g, off, 64);
            held_c += __shfl_xor(held_c, off, 64);
            n_frozen += __shfl_xor(n_frozen, off, 64);
        }
        if (lane == 0 && n_frozen) { atomicAdd(&sum_g, held_g); atomicAdd(&sum_c, held_c); atomicAdd(&sum_f, n_frozen); }
        if (__syncthreads_or(other)) round_needed = true;
        if (tid == 0) {
            const unsigned long long hg = sum_g, hc = sum_c;
            A.F.cap0[0] = hg < A.cl.G ? A.cl.G - hg : 0ull;   // frozen jobs are charged first
            A.F.cap0[1] = hc < A.cl.C ? A.cl.C - hc : 0ull;
            if (A.out.frozen) A.out.frozen[tick] = sum_f;
            if (COUNT) *part = sum_p;
        }
        if (round_needed) return true;
        __syncthreads();                                      // the sums are read before they are cleared
    }
}

// Ticks of a simulation under the greedy in one workgroup, on the context's stream: SIM_NOT_FEW: none; SIM_ALWAYS_FEW: all of
// them; SIM_OFTEN_FEW: those whose rounds are for at most `most` jobs that do not walk long over the CPU levels.
enum SimFew { SIM_NOT_FEW, SIM_OFTEN_FEW, SIM_ALWAYS_FEW };
SimFew rk_sim_few(uint32_t n_jobs, uint32_t max_segs_per_job, const rk_alloc_grid *grid, const rk_cluster *cluster, uint32_t *most);
// n_launches of SIM_FEW_TICKS ticks each from the one that *A.tick says (begin: from the first one).  A tick whose round is for
// more than `most` jobs ends them, and stays open; one whose walks were long ends them when it is closed.
int32_t rk_launch_sim_few(rk_ctx *ctx, const SimArgs &A, const float *ref_thr, const rk_alloc_grid *grid, uint32_t max_segs_per_job,
                          const float *best_thr, const uint32_t *best_plan, const float *curve_thr, rk_assign *assign,
                          uint32_t n_launches, bool begin, bool often, uint32_t most);

// Whether a simulation over these nodes has its ticks in one workgroup's LDS, and all its ticks (rk_nodes.hip).
bool rk_sim_nodes_fit(uint32_t n_jobs, const rk_nodes *nodes);
int32_t rk_launch_sim_nodes(rk_ctx *ctx, const SimArgs &S, const float *ref_thr, const rk_plan_table *table, const rk_alloc_grid *grid,
                            const rk_nodes *nodes, const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                            uint64_t cap_parts, rk_assign *assign);
