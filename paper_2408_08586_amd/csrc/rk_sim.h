// The state of a simulation and what a tick does to a job, shared by the kernel that closes and opens ticks around the
// rounds of any policy (k_sim_step) and the one that runs whole ticks of the greedy (k_sim_few).
#pragma once
#include "rk_internal.h"
#include "rk_model.h"

constexpr uint32_t SIM_FEW_TICKS = 128;        // ticks of a launch of k_sim_few

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
    uint32_t *tick;             // device counter: the tick whose round comes next
    uint32_t *h_tick;           // its copy in pinned host memory
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

// Ticks [t0, t1) of a simulation under the greedy, on the context's stream; false in *taken: not a simulation for it.
int32_t rk_launch_sim_few(rk_ctx *ctx, const SimArgs &A, const float *ref_thr, const rk_alloc_grid *grid, uint32_t max_segs_per_job,
                          const float *best_thr, const uint32_t *best_plan, const float *curve_thr, rk_assign *assign, bool *taken);
