// Greedy marginal-gain allocation over the resource sensitivity curves
// (paper Sec. 5.2: prefer the jobs that gain the most per unit of resource,
// GPU slopes before CPU slopes; memory is granted last from the chosen plan's
// estimate).
//
// The rule is sequential: repeatedly take the (job, larger amount) with the
// highest float32 slope ((v1 - v0) / ref_thr) / delta among the steps that
// still fit; ties go to the smaller amount, then to the lower job index.
// It is evaluated without running every step in sequence.  Per pass (GPUs,
// then CPUs):
//
//  k_hull   Each job's steps, were capacity never short, form a fixed walk
//           over the upper hull of its curve (one wavefront per job; two or
//           four jobs per wavefront when none has more than 32 or 16 amounts:
//           k_hull_groups).  With
//           each slope replaced by the running minimum of the walk, the
//           sequential order is the descending order of these keys (then job,
//           then position in the walk).
//  k_hist   Any key threshold whose whole set of steps {key > threshold} fits
//           the capacity selects a prefix of the sequential order.  Two
//           histogram levels over the top 12 + 12 key bits (cost per bin) find
//           the largest such threshold at 24-bit resolution.
//  k_apply  applies that prefix to every job at once and caches each job's
//           next step (the walk's next step if it still fits, otherwise a fresh
//           search within the capacity that is left).
//  k_tail   the plain step-by-step loop on the little capacity that is left:
//           one workgroup per round, whose first wavefront takes steps from a
//           list of the best cached ones, which all wavefronts keep and find;
//           in smaller rounds a few steps are taken one by one instead.
//  When no job's CPU walk has a step, the CPU pass's k_hist, k_apply and k_tail
//  return at once (a per-round flag raised by its k_hull).
//
// Memory (k_mem_wish / k_mem_finish): when the tiers every job would like fit
// with margin, all are granted in parallel; otherwise one wavefront takes the
// decisions in job order.
//
// Service-level floors (k_floors, optional): before the passes, guaranteed
// jobs are granted their minimum demand in job order while their tenant's
// quota and the free capacity last; the passes then start from these floors
// and leave out the guaranteed jobs that have to wait.
#include <type_traits>

#include "rk_internal.h"
#include "rk_model.h"
#include "rk_loop.h"
#include "rk_sim.h"

namespace {

constexpr int TAIL_THREADS = 1024;
constexpr int HULL_THREADS = 256;
constexpr int JOB_THREADS = 256;           // kernels with one thread per job
constexpr uint32_t BINS = 4096;            // 12 key bits per histogram level
// Where bin b is kept: the T threads of find_cut take BINS / T neighbouring bins each, and laid out like this their
// i-th bins are neighbours (from plain order every load met a 16- to 32-way bank conflict in LDS, or as many cache lines
// as lanes in memory).
template <int T>
__device__ __forceinline__ uint32_t bin_at(uint32_t b) { return (b % (BINS / T)) * T + b / (BINS / T); }

struct HullBuf {             // walk steps, entry (k, job) at k*stride + job (job relative to the call's first job)
    uint32_t *key;           // float bits of the running-minimum slope; 0 from the end of the walk on
    float *raw;              // the step's own slope
    uint16_t *tgt;           // target: segment index (GPU pass) or CPU level (CPU pass)
    uint32_t *dg;            // GPUs the step adds
    unsigned long long *dc;  // CPUs the step adds
    uint32_t stride, width;
};

// Highest bin of a histogram whose steps, added to everything above it, no longer fit.
// bin = -1: all bins fit.  base*: cost of the bins above `bin`.
struct Cut { int32_t bin; unsigned long long baseG, baseC; };

struct Hist {                // per round, pass and level: cost of the steps per key bin, and per group of bins
    uint32_t *g;             // [n_rounds][2 passes][2 levels][HIST_WORDS]
    unsigned long long *c;
    Cut *cut;                // per round: where level 0 of the pass under way was cut
};

struct JobState {            // per job of the call, between the kernels
    int32_t *gi;             // granted segment index, -1 = no GPUs
    uint32_t *g;             // granted GPUs
    uint32_t *ci;            // granted CPU level
    float *step_slope;       // cached best next step: slope (0 = none), target, GPUs it adds
    uint16_t *step_tgt, *step_dg;
    unsigned long long *free_g, *free_c;   // per round: capacity left (after apply; after the tail)
    uint32_t *cpu_steps;     // per round: non-zero when some job's CPU walk has a step (else the CPU pass has nothing to do)
    double *partial;         // per round and block of k_mem_wish: {sum of wish GiB, sum of thr/ref}
    uint32_t blocks_per_round;
    // floors, all null without them: the state a job starts from (segment index
    // or -1, CPU level), whether it takes part (RK_JOB_NORMAL), sits the round
    // out (RK_JOB_OUT) or keeps exactly its floor (RK_JOB_FROZEN), and per round
    // the capacity left after the floors ([free G | free C])
    int32_t *fl_gi;
    uint32_t *fl_ci;
    uint8_t *waits;
    unsigned long long *cap0;
};

struct Floor { int32_t gi; uint32_t ci; uint32_t state; };

__device__ __forceinline__ Floor floor_of(const JobState &st, uint32_t jrel) {
    Floor f = {-1, 0u, RK_JOB_NORMAL};
    if (st.fl_gi) { f.gi = st.fl_gi[jrel]; f.ci = st.fl_ci[jrel]; f.state = st.waits[jrel]; }
    return f;
}

// Rounds: job ranges and cluster capacities, either device arrays or, for a
// single round, values carried in the kernel arguments.
struct RoundArgs {
    const uint32_t *round_off;
    const rk_cluster *clusters;
    uint32_t n_rounds, inline_one;
    uint32_t off0, off1;
    rk_cluster cl;
};

struct Ctx {                 // what every kernel of the allocation needs
    const float *ref_thr;
    TableDev tb;
    GridDev grid;
    RoundArgs R;
    uint32_t jb;             // first job of the call (origin of the segment-layout arrays)
    const uint32_t *jmap;    // optional: the job whose curves slot j of the call uses (rounds that share jobs)
    const float *best_thr;
    const uint32_t *best_plan;
    const float *curve_thr;
};

// The job whose plan table, curves and reference throughput slot j uses.
__device__ __forceinline__ uint32_t job_of(const Ctx &X, uint32_t j) { return X.jmap ? X.jmap[j] : j; }

__device__ __forceinline__ void round_of(const RoundArgs &R, uint32_t r, uint32_t &j0, uint32_t &j1, rk_cluster &cl) {
    if (R.inline_one) { j0 = R.off0; j1 = R.off1; cl = R.cl; }
    else { j0 = R.round_off[r]; j1 = R.round_off[r + 1]; cl = R.clusters[r]; }
}

__device__ __forceinline__ uint32_t round_index_of(const RoundArgs &R, uint32_t j) {
    uint32_t lo = 0, hi = R.n_rounds;                     // last r with round_off[r] <= j
    while (!R.inline_one && hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (R.round_off[mid] <= j) lo = mid; else hi = mid;
    }
    return lo;
}


// A histogram in memory: its bins, then the sums of every GROUP_BINS neighbouring ones.
constexpr uint32_t GROUP_BINS = 64, GROUPS = BINS / GROUP_BINS, HIST_WORDS = BINS + GROUPS;
static_assert(GROUPS == 64 && GROUP_BINS == 64, "a wavefront looks at the groups, then at the bins of one");
__device__ __forceinline__ size_t hist_at(uint32_t rnd, int pass, int level) {
    return (((size_t)rnd * 2 + pass) * 2 + level) * HIST_WORDS;
}

// capacities a pass starts from
template <int PASS>
__device__ __forceinline__ void pass_caps(const RoundArgs &R, const rk_cluster &cl, const JobState &st, uint32_t rnd,
                                          unsigned long long &capG, unsigned long long &capC) {
    if (PASS == 0) {
        if (st.cap0) { capG = st.cap0[rnd]; capC = st.cap0[R.n_rounds + rnd]; }
        else { capG = cl.G; capC = cl.C; }
    } else { capG = 0; capC = st.free_c[rnd]; }
}

// ------------------------------------------------------------------ hull walks
// One wavefront per job; lanes hold the candidate amounts.  PASS 0: GPU counts
// of the job (CPU level of its floor, the lowest without one; highest memory
// tier; values from the curves); PASS 1: CPU levels at the granted GPU count
// (values from the per-segment maxima).  Amounts that the whole round could
// never afford are left out.
template <int PASS>
__global__ __launch_bounds__(HULL_THREADS) void k_hull(Ctx X, JobState st, HullBuf H, Hist zero, size_t zero_bins) {
    // the histograms of the kernels that follow start at zero (zero_bins = 0: nothing to clear)
    for (size_t i = (size_t)blockIdx.x * HULL_THREADS + threadIdx.x; i < zero_bins; i += (size_t)gridDim.x * HULL_THREADS) {
        zero.g[i] = 0u;
        zero.c[i] = 0ull;
        if (i < X.R.n_rounds) st.cpu_steps[i] = 0u;       // (there are more bins than rounds)
    }
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t jrel = blockIdx.x * (HULL_THREADS / 64) + (threadIdx.x >> 6);
    if (jrel >= H.stride) return;                         // whole wavefront
    const uint32_t j = X.jb + jrel;
    const uint32_t rnd = round_index_of(X.R, j);
    uint32_t rj0, rj1;
    rk_cluster cl;
    round_of(X.R, rnd, rj0, rj1, cl);
    const GridDev &grid = X.grid;
    const float *__restrict__ vals = PASS == 0 ? X.curve_thr : X.best_thr;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem;
    const uint32_t ju = job_of(X, j);
    const uint32_t s0 = X.tb.seg_off[ju], ns = X.tb.seg_off[ju + 1] - s0;
    const uint64_t jbase = (uint64_t)n_rows * (s0 - X.tb.seg_off[X.jb]);
    const float ref = X.ref_thr[ju];

    uint32_t npts, g_fixed = 0, c_fixed = 0;
    int32_t cur_i;
    unsigned long long cost_cur, cap_c, cap_g = 0;
    float cur;
    int32_t gi = -1;
    if (PASS == 0) {
        const Floor fl = floor_of(st, jrel);
        unsigned long long startG, startC;
        pass_caps<0>(X.R, cl, st, rnd, startG, startC);
        c_fixed = fl.ci;
        npts = fl.state != RK_JOB_NORMAL ? 0u : ns;
        cur_i = fl.gi;
        cost_cur = fl.gi < 0 ? 0ull : (unsigned long long)X.tb.seg_g[s0 + fl.gi];
        cur = fl.gi < 0 ? 0.f : vals[jbase + (uint64_t)(c_fixed * n_mem + n_mem - 1) * ns + fl.gi];
        cap_g = startG + cost_cur;                       // the floor is already paid for
        cap_c = startC + (fl.gi < 0 ? 0ull : cpu_cost(grid, c_fixed, (uint32_t)cost_cur));
    } else {
        gi = st.gi[jrel];
        npts = (gi < 0 || (st.waits && st.waits[jrel] != RK_JOB_NORMAL)) ? 0u : grid.n_cpu;
        g_fixed = gi < 0 ? 0u : st.g[jrel];
        cur_i = (int32_t)st.ci[jrel];
        cost_cur = cpu_cost(grid, (uint32_t)cur_i, g_fixed);
        cap_c = st.free_c[rnd] + cost_cur;               // the level held is already paid for
        cur = gi < 0 ? 0.f : vals[jbase + (uint64_t)((uint32_t)cur_i * n_mem + n_mem - 1) * ns + gi];
    }
    // amount s: its cost in the pass's resource and its value
    auto cost_of = [&](uint32_t s) -> unsigned long long {
        return PASS == 0 ? (unsigned long long)X.tb.seg_g[s0 + s] : cpu_cost(grid, s, g_fixed);
    };
    auto value_of = [&](uint32_t s) -> float {
        return PASS == 0 ? vals[jbase + (uint64_t)(c_fixed * n_mem + n_mem - 1) * ns + s]
                         : vals[jbase + (uint64_t)(s * n_mem + n_mem - 1) * ns + gi];
    };
    auto affordable = [&](unsigned long long cost) -> bool {
        if (PASS == 0) return cost <= cap_g && cpu_cost(grid, c_fixed, (uint32_t)cost) <= cap_c;
        return cost <= cap_c;
    };

    // the first 64 amounts stay in registers over the whole walk (most jobs have no more)
    unsigned long long cost0 = 0;
    float val0 = 0.f;
    if (lane < npts) { cost0 = cost_of(lane); val0 = value_of(lane); }

    uint32_t k = 0;
    float prev = __uint_as_float(0x7F800000u);
    while (k < H.width) {
        unsigned long long best = 0;
        for (uint32_t base = 0; base < npts; base += 64) {
            const uint32_t s = base + lane;
            if (s < npts && (int32_t)s > cur_i) {
                const unsigned long long cost = base == 0 ? cost0 : cost_of(s);
                if (affordable(cost)) {
                    const float v = base == 0 ? val0 : value_of(s);
                    if (v > cur) {
                        float sl = (v - cur) / ref;
                        sl = sl / (float)(cost - cost_cur);
                        const unsigned long long c = ((unsigned long long)__float_as_uint(sl) << 32) | (0xFFFFFFFFu - s);
                        best = c > best ? c : best;
                    }
                }
            }
        }
        best = wave_max_u64_rows(best);                   // all lanes are here: the loops above run the same number of times
        if (!(best >> 32)) break;
        const float top = __uint_as_float((uint32_t)(best >> 32));
        const uint32_t top_s = 0xFFFFFFFFu - (uint32_t)best;
        // cost and value of the chosen amount: from its lane's registers when it is among the first 64
        unsigned long long top_cost;
        float top_val;
        if (top_s < 64u) {
            const int src = __builtin_amdgcn_readfirstlane((int)top_s);
            top_cost = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(cost0 >> 32), src) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)cost0, src);
            top_val = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(val0), src));
        } else {
            top_cost = cost_of(top_s);
            top_val = value_of(top_s);
        }
        prev = top < prev ? top : prev;
        if (lane == 0) {
            const size_t e = (size_t)k * H.stride + jrel;
            H.key[e] = __float_as_uint(prev);
            H.raw[e] = top;
            H.tgt[e] = (uint16_t)top_s;
            if (PASS == 0) {
                H.dg[e] = (uint32_t)(top_cost - cost_cur);
                H.dc[e] = cpu_cost(grid, c_fixed, (uint32_t)top_cost) - (cost_cur ? cpu_cost(grid, c_fixed, (uint32_t)cost_cur) : 0ull);
            } else {
                H.dg[e] = 0u;
                H.dc[e] = top_cost - cost_cur;
            }
        }
        cur = top_val;
        cur_i = (int32_t)top_s;
        cost_cur = top_cost;
        ++k;
    }
    for (uint32_t kk = k + lane; kk < H.width; kk += 64) H.key[(size_t)kk * H.stride + jrel] = 0u;   // unused positions
    if (PASS == 1 && k > 0 && lane == 0) st.cpu_steps[rnd] = 1u;
}

// The same walks with several jobs per wavefront, for calls in which no job has
// more than LANES amounts (LANES = 16 or 32): a job takes LANES neighbouring
// lanes, the wavefront loops until the last of its jobs has finished, and a
// job's maximum is taken over its own lanes only.  Bound by instructions: the
// maximum is of one word, the amount that reaches it comes from a ballot, and
// a step stays in the lane of its number until the walk is over (pairs of
// words and five stores per step: 123 us for 128,000 jobs with up to 32
// amounts, now 90).
template <int LANES>
__device__ __forceinline__ uint32_t group_max_u32(uint32_t v, uint32_t lane) {
    v = rs_max_u32(v, rs_dpp_u32<0xB1, 0xF>(0u, v));               // quad_perm [1,0,3,2]
    v = rs_max_u32(v, rs_dpp_u32<0x4E, 0xF>(0u, v));               // quad_perm [2,3,0,1]
    v = rs_max_u32(v, rs_dpp_u32<0x141, 0xF>(0u, v));              // row_half_mirror
    v = rs_max_u32(v, rs_dpp_u32<0x140, 0xF>(0u, v));              // row_mirror: every row of 16 lanes holds its maximum
    if (LANES == 16) return v;
    const uint32_t lo = rs_max_u32((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16));
    const uint32_t hi = rs_max_u32((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48));
    return lane < 32 ? lo : hi;
}

template <int PASS, int LANES>
__global__ __launch_bounds__(HULL_THREADS) void k_hull_groups(Ctx X, JobState st, HullBuf H, Hist zero, size_t zero_bins) {
    for (size_t i = (size_t)blockIdx.x * HULL_THREADS + threadIdx.x; i < zero_bins; i += (size_t)gridDim.x * HULL_THREADS) {
        zero.g[i] = 0u;
        zero.c[i] = 0ull;
        if (i < X.R.n_rounds) st.cpu_steps[i] = 0u;
    }
    constexpr uint32_t PER_WAVE = 64 / LANES;
    const uint32_t lane = threadIdx.x & 63u, sub = lane % LANES, group_base = lane - sub;
    const uint32_t slot = (blockIdx.x * (HULL_THREADS / 64) + (threadIdx.x >> 6)) * PER_WAVE + lane / LANES;
    const bool valid = slot < H.stride;                    // lanes of a slot past the end stay for the shuffles
    const uint32_t jrel = valid ? slot : H.stride - 1;
    const uint32_t j = X.jb + jrel;
    const uint32_t rnd = round_index_of(X.R, j);
    uint32_t rj0, rj1;
    rk_cluster cl;
    round_of(X.R, rnd, rj0, rj1, cl);
    const GridDev &grid = X.grid;
    const float *__restrict__ vals = PASS == 0 ? X.curve_thr : X.best_thr;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem;
    const uint32_t ju = job_of(X, j);
    const uint32_t s0 = X.tb.seg_off[ju], ns = X.tb.seg_off[ju + 1] - s0;
    const uint64_t jbase = (uint64_t)n_rows * (s0 - X.tb.seg_off[X.jb]);
    const float ref = X.ref_thr[ju];

    uint32_t npts, g_fixed = 0, c_fixed = 0;
    int32_t cur_i;
    unsigned long long cost_held, cap_c, cap_g = 0;
    float cur;
    int32_t gi = -1;
    if (PASS == 0) {
        const Floor fl = floor_of(st, jrel);
        unsigned long long startG, startC;
        pass_caps<0>(X.R, cl, st, rnd, startG, startC);
        c_fixed = fl.ci;
        npts = fl.state != RK_JOB_NORMAL ? 0u : ns;
        cur_i = fl.gi;
        cost_held = fl.gi < 0 ? 0ull : (unsigned long long)X.tb.seg_g[s0 + fl.gi];
        cur = fl.gi < 0 ? 0.f : vals[jbase + (uint64_t)(c_fixed * n_mem + n_mem - 1) * ns + fl.gi];
        cap_g = startG + cost_held;                      // the floor is already paid for
        cap_c = startC + (fl.gi < 0 ? 0ull : cpu_cost(grid, c_fixed, (uint32_t)cost_held));
    } else {
        gi = st.gi[jrel];
        npts = (gi < 0 || (st.waits && st.waits[jrel] != RK_JOB_NORMAL)) ? 0u : grid.n_cpu;
        g_fixed = gi < 0 ? 0u : st.g[jrel];
        cur_i = (int32_t)st.ci[jrel];
        cost_held = cpu_cost(grid, (uint32_t)cur_i, g_fixed);
        cap_c = st.free_c[rnd] + cost_held;              // the level held is already paid for
        cur = gi < 0 ? 0.f : vals[jbase + (uint64_t)((uint32_t)cur_i * n_mem + n_mem - 1) * ns + gi];
    }
    if (!valid) npts = 0;
    // the lane's amount: cost in the pass's resource, value, and whether the round could ever afford it
    // (of the costs the walk takes the low words: a step that the round can afford fits one)
    uint32_t cost0 = 0;
    float val0 = 0.f;
    bool can = false;
    if (sub < npts) {
        const unsigned long long cost = PASS == 0 ? (unsigned long long)X.tb.seg_g[s0 + sub] : cpu_cost(grid, sub, g_fixed);
        val0 = PASS == 0 ? vals[jbase + (uint64_t)(c_fixed * n_mem + n_mem - 1) * ns + sub]
                         : vals[jbase + (uint64_t)(sub * n_mem + n_mem - 1) * ns + gi];
        can = PASS == 0 ? (cost <= cap_g && cpu_cost(grid, c_fixed, (uint32_t)cost) <= cap_c) : cost <= cap_c;
        cost0 = (uint32_t)cost;
    }

    uint32_t k = 0;
    float prev = __uint_as_float(0x7F800000u);
    // the lane's step of the walk: step number = lane number within the job
    uint32_t my_key = 0, my_raw = 0, my_tgt = 0;
    uint32_t my_from = 0, my_to = 0;                       // its costs before and after
    uint32_t cost_cur = (uint32_t)cost_held;
    bool walking = npts > 0;                               // the same in all lanes of a job (H.width is at least 1)
    while (__ballot(walking)) {                            // until the wavefront's last job has finished
        uint32_t best = 0;
        if (walking && can && (int32_t)sub > cur_i && val0 > cur) {
            float sl = (val0 - cur) / ref;
            sl = sl / (float)(cost0 - cost_cur);
            best = __float_as_uint(sl);
        }
        const uint32_t top = group_max_u32<LANES>(best, lane);
        walking = walking && top != 0u;
        // the smallest amount that reaches it, and what the lane that holds it knows
        const uint32_t reach = (uint32_t)(__ballot(best == top) >> group_base) & (LANES == 16 ? 0xFFFFu : 0xFFFFFFFFu);
        const uint32_t top_s = reach ? (uint32_t)__ffs((int)reach) - 1u : 0u;
        const int src = (int)(group_base + top_s);
        const uint32_t top_cost = (uint32_t)__shfl((int)cost0, src, 64);
        const float top_val = __shfl(val0, src, 64);
        if (walking) {
            prev = __uint_as_float(top) < prev ? __uint_as_float(top) : prev;
            if (sub == k) { my_key = __float_as_uint(prev); my_raw = top; my_tgt = top_s; my_from = cost_cur; my_to = top_cost; }
            cur = top_val;
            cur_i = (int32_t)top_s;
            cost_cur = top_cost;
            ++k;
            walking = k < H.width;
        }
    }
    if (valid) {
        if (sub < k) {                                     // (a walk has no more steps than the job has lanes)
            const size_t e = (size_t)sub * H.stride + jrel;
            H.raw[e] = __uint_as_float(my_raw);
            H.tgt[e] = (uint16_t)my_tgt;
            if (PASS == 0) {
                H.dg[e] = my_to - my_from;
                H.dc[e] = cpu_cost(grid, c_fixed, my_to) - (my_from ? cpu_cost(grid, c_fixed, my_from) : 0ull);
            } else {
                H.dg[e] = 0u;
                H.dc[e] = my_to - my_from;
            }
        }
        for (uint32_t kk = sub; kk < H.width; kk += LANES) H.key[(size_t)kk * H.stride + jrel] = kk < k ? my_key : 0u;
        if (PASS == 1 && k > 0 && sub == 0) st.cpu_steps[rnd] = 1u;
    }
}

// ------------------------------------------------------------------ threshold search
struct CutScratch {
    uint32_t wave_g[16];                     // totals of the wavefronts
    unsigned long long wave_c[16];
    int32_t first[16];                       // their first thread with a failing bin (-1: none), and what lies above its bins
    unsigned long long firstG[16], firstC[16];
};

// Inclusive sums along the rows of 16 lanes, and over the whole wavefront (all 64 lanes active).
template <int CTRL, int ROWS>
__device__ __forceinline__ void scan_add(uint32_t &g, unsigned long long &c) {
    const uint32_t lo = rs_dpp_u32<CTRL, ROWS>(0u, (uint32_t)c), hi = rs_dpp_u32<CTRL, ROWS>(0u, (uint32_t)(c >> 32));
    g += rs_dpp_u32<CTRL, ROWS>(0u, g);
    c += ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ void row_scan(uint32_t &g, unsigned long long &c) {
    scan_add<0x111, 0xF>(g, c); scan_add<0x112, 0xF>(g, c); scan_add<0x114, 0xF>(g, c); scan_add<0x118, 0xF>(g, c);
}
__device__ __forceinline__ void wave_scan(uint32_t &g, unsigned long long &c) {
    row_scan(g, c);
    scan_add<0x142, 0xA>(g, c);              // row_bcast:15 into rows 1 and 3
    scan_add<0x143, 0xC>(g, c);              // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ unsigned long long wave_lane_u64(unsigned long long x, uint32_t s) {
    return ((unsigned long long)wave_lane_u32((uint32_t)(x >> 32), s) << 32) | wave_lane_u32((uint32_t)x, s);
}

// Workgroup-wide, T threads: thread t owns the BINS / T bins from BINS-1-t*BINS/T downwards; every thread must call it
// (two barriers; the histogram may be written again after one more) and gets the result.  A chain on the way of every
// pass: sums by data-parallel-primitive moves, and the bins of the one thread where the sum goes beyond the capacity
// looked at by sixteen lanes of every wavefront (shuffled pairs, sixteen bins per thread one after the other and three
// barriers took 3.3 to 4.2 us, this takes 1.4).  GPU costs of a round fit 32 bits (jobs * RK_MAX_G).
template <int T>
__device__ Cut find_cut(const uint32_t *__restrict__ hG, const unsigned long long *__restrict__ hC,
                        unsigned long long baseG, unsigned long long baseC, unsigned long long capG,
                        unsigned long long capC, CutScratch &S) {
    constexpr uint32_t PER = BINS / T, NW = T / 64;
    static_assert(PER <= 16 && NW <= 16 && (unsigned long long)RK_MAX_JOBS_PER_ROUND * RK_MAX_G < (1ull << 32), "one row of lanes; 32-bit sums");
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t top = BINS - 1 - tid * PER;
    uint32_t sg = 0;
    unsigned long long sc = 0;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) { sg += hG[bin_at<T>(top - i)]; sc += hC[bin_at<T>(top - i)]; }
    uint32_t ig = sg;
    unsigned long long ic = sc;
    wave_scan(ig, ic);
    if (lane == 63u) { S.wave_g[wave] = ig; S.wave_c[wave] = ic; }
    __syncthreads();
    uint32_t wg = (lane & 15u) < NW ? S.wave_g[lane & 15u] : 0u;
    unsigned long long wc = (lane & 15u) < NW ? S.wave_c[lane & 15u] : 0ull;
    row_scan(wg, wc);
    const uint32_t allG = wave_lane_u32(wg, 15u);
    const unsigned long long allC = wave_lane_u64(wc, 15u);
    const uint32_t w1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)wave);
    const unsigned long long aboveG = baseG + (w1 ? wave_lane_u32(wg, w1 - 1u) : 0u) + (ig - sg);    // everything above this thread's bins
    const unsigned long long aboveC = baseC + (w1 ? wave_lane_u64(wc, w1 - 1u) : 0ull) + (ic - sc);
    const unsigned long long over = __ballot(aboveG + sg > capG || aboveC + sc > capC);
    if (over ? lane == (uint32_t)__ffsll((long long)over) - 1u : lane == 0u) {
        S.first[wave] = over ? (int32_t)tid : -1;
        S.firstG[wave] = aboveG; S.firstC[wave] = aboveC;
    }
    __syncthreads();
    Cut out = {-1, baseG + allG, baseC + allC};
    const unsigned long long with = __ballot(lane < NW && S.first[lane < NW ? lane : 0u] >= 0);
    if (!with) return out;                                 // all bins fit
    const uint32_t w0 = (uint32_t)__ffsll((long long)with) - 1u;
    const int32_t first = S.first[w0];
    const unsigned long long g0 = S.firstG[w0], c0 = S.firstC[w0];
    const uint32_t at = BINS - 1u - (uint32_t)first * PER - (lane < PER ? lane : 0u);
    const uint32_t vg = lane < PER ? hG[bin_at<T>(at)] : 0u;
    const unsigned long long vc = lane < PER ? hC[bin_at<T>(at)] : 0ull;
    ig = vg; ic = vc;
    row_scan(ig, ic);
    const uint32_t i0 = (uint32_t)__ffsll((long long)__ballot(lane < PER && (g0 + ig > capG || c0 + ic > capC))) - 1u;
    out.bin = (int32_t)(BINS - 1u - (uint32_t)first * PER - i0);
    out.baseG = g0 + wave_lane_u32(ig - vg, i0);
    out.baseC = c0 + wave_lane_u64(ic - vc, i0);
    return out;
}

// The same from a histogram in memory, by every wavefront for itself: the first failing group of the 64, from the highest
// down, then the first failing bin of that group; a lane per group and bin, two rounds of loads and 1.5 KB where all bins
// are 48 KB (4 us in each kernel that has to find one).
struct GroupSums { uint32_t g; unsigned long long c; };
__device__ __forceinline__ GroupSums load_groups(const uint32_t *__restrict__ hG, const unsigned long long *__restrict__ hC) {
    const uint32_t at = BINS + GROUPS - 1u - (threadIdx.x & 63u);
    return GroupSums{hG[at], hC[at]};
}
__device__ __forceinline__ Cut find_cut_groups(const uint32_t *__restrict__ hG, const unsigned long long *__restrict__ hC, GroupSums sum,
                                               unsigned long long baseG, unsigned long long baseC, unsigned long long capG,
                                               unsigned long long capC) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t ig = sum.g;
    unsigned long long ic = sum.c;
    wave_scan(ig, ic);
    const unsigned long long over = __ballot(baseG + ig > capG || baseC + ic > capC);
    if (!over) return Cut{-1, baseG + wave_lane_u32(ig, 63u), baseC + wave_lane_u64(ic, 63u)};      // all bins fit
    const uint32_t group = (uint32_t)__ffsll((long long)over) - 1u;                                 // (counted from the highest)
    baseG += wave_lane_u32(ig - sum.g, group); baseC += wave_lane_u64(ic - sum.c, group);
    const uint32_t top = BINS - 1u - group * GROUP_BINS;
    const uint32_t vg = hG[top - lane];
    const unsigned long long vc = hC[top - lane];
    ig = vg; ic = vc;
    wave_scan(ig, ic);
    const uint32_t i0 = (uint32_t)__ffsll((long long)__ballot(baseG + ig > capG || baseC + ic > capC)) - 1u;
    return Cut{(int32_t)(top - i0), baseG + wave_lane_u32(ig - vg, i0), baseC + wave_lane_u64(ic - vc, i0)};
}

template <int PASS>
__device__ __forceinline__ uint32_t walk_width(const Ctx &X, const HullBuf &H) {
    return PASS == 0 ? H.width : (X.grid.n_cpu - 1 < H.width ? X.grid.n_cpu - 1 : H.width);
}

// The first steps of a job's walk, in the registers of its thread: the selection in one workgroup goes over them three
// times (two histograms and the application), each time a round or two of loads from memory that other chiplets wrote.
// Rounds of 300 and 700 jobs 74.4 -> 70.2 and 87.3 -> 85.2 us with a job per thread; through a pointer, in scratch memory,
// 76.7 and 93.0.
constexpr uint32_t AHEAD = 8;
struct WalkAhead { uint32_t key[AHEAD], dg[AHEAD], tgt[AHEAD]; float raw[AHEAD]; unsigned long long dc[AHEAD]; };
template <int PASS>
__device__ __forceinline__ void walk_ahead(const Ctx &X, const HullBuf &H, bool have, uint32_t jrel, WalkAhead &W) {
    const uint32_t width = walk_width<PASS>(X, H);
#pragma unroll
    for (uint32_t u = 0; u < AHEAD; ++u) {
        const bool in = have && u < width;
        const size_t e = in ? (size_t)u * H.stride + jrel : 0;
        W.key[u] = in ? H.key[e] : 0u;
        W.raw[u] = in ? H.raw[e] : 0.f; W.tgt[u] = in ? H.tgt[e] : 0u;
        W.dg[u] = in && PASS == 0 ? H.dg[e] : 0u; W.dc[u] = in ? H.dc[e] : 0ull;
    }
}

// Adds a step to a histogram in LDS; false: the walk has no further step that counts.
template <int LEVEL, int T>
__device__ __forceinline__ bool hist_step(uint32_t key, uint32_t dg, unsigned long long dc, int32_t want_top, uint32_t *lg, unsigned long long *lc) {
    if (!key) return false;
    uint32_t bin;
    if (LEVEL == 0) bin = key >> 20;
    else {
        if ((int32_t)(key >> 20) > want_top) return true;
        if ((int32_t)(key >> 20) < want_top) return false;        // keys only decrease along a walk
        bin = (key >> 8) & (BINS - 1);
    }
    if (dg) atomicAdd(&lg[bin_at<T>(bin)], dg);
    if (dc) atomicAdd(&lc[bin_at<T>(bin)], dc);
    return true;
}

// Adds the steps of one job's walk to a histogram in LDS.  The walk is read
// four steps at a time (all twelve loads go out together; positions past the
// walk's end are inside the buffers and ignored).
template <int PASS, int LEVEL, int T>
__device__ __forceinline__ void hist_add(const Ctx &X, const HullBuf &H, uint32_t jrel, int32_t want_top, uint32_t *lg,
                                         unsigned long long *lc, uint32_t from = 0) {
    const uint32_t width = walk_width<PASS>(X, H);
    for (uint32_t k0 = from; k0 < width; k0 += 4) {
        uint32_t key[4], dg[4];
        unsigned long long dc[4];
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t k = k0 + u < width ? k0 + u : width - 1;
            const size_t e = (size_t)k * H.stride + jrel;
            key[u] = H.key[e];
            dg[u] = PASS == 0 ? H.dg[e] : 0u;
            dc[u] = H.dc[e];
        }
#pragma unroll
        for (uint32_t u = 0; u < 4; ++u)
            if (k0 + u >= width || !hist_step<LEVEL, T>(key[u], dg[u], dc[u], want_top, lg, lc)) return;
    }
}
// ... of which the first are in registers
template <int PASS, int LEVEL, int T>
__device__ __forceinline__ void hist_add(const Ctx &X, const HullBuf &H, const WalkAhead &W, uint32_t jrel, int32_t want_top, uint32_t *lg,
                                         unsigned long long *lc) {
    bool on = true;
#pragma unroll
    for (uint32_t u = 0; u < AHEAD; ++u) on = on && hist_step<LEVEL, T>(W.key[u], W.dg[u], W.dc[u], want_top, lg, lc);
    if (on) hist_add<PASS, LEVEL, T>(X, H, jrel, want_top, lg, lc, AHEAD);
}

// Cost histogram of one level.  Level 0: bin = key bits 31..20 of every step.
// Level 1: key bits 19..8 of the steps inside the bin where level 0 was cut,
// which the round's first workgroup leaves in hist.cut for the kernel that
// applies the selection.
template <int PASS, int LEVEL>
__global__ __launch_bounds__(JOB_THREADS) void k_hist(Ctx X, JobState st, HullBuf H, Hist hist) {
    __shared__ uint32_t lg[BINS];
    __shared__ unsigned long long lc[BINS];
    const uint32_t rnd = blockIdx.y, tid = threadIdx.x;
    if (PASS == 1 && st.cpu_steps[rnd] == 0u) return;       // no job can use more CPUs: the whole pass is empty
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    int32_t want_top = 0;
    if (LEVEL == 1) {
        unsigned long long capG, capC;
        pass_caps<PASS>(X.R, cl, st, rnd, capG, capC);
        const size_t h0 = hist_at(rnd, PASS, 0);
        const Cut c0 = find_cut_groups(hist.g + h0, hist.c + h0, load_groups(hist.g + h0, hist.c + h0), 0, 0, capG, capC);
        if (blockIdx.x == 0 && tid == 0) hist.cut[rnd] = c0;
        if (c0.bin < 0) return;                           // everything fits: no second level needed
        want_top = c0.bin;
    }
    for (uint32_t i = tid; i < BINS; i += JOB_THREADS) { lg[i] = 0; lc[i] = 0; }
    __syncthreads();
    const uint32_t jl = blockIdx.x * JOB_THREADS + tid;
    if (J0 + jl < J1) hist_add<PASS, LEVEL, 1>(X, H, J0 + jl - X.jb, want_top, lg, lc);
    __syncthreads();
    const size_t h = hist_at(rnd, PASS, LEVEL);
    for (uint32_t i = tid; i < BINS; i += JOB_THREADS) {    // (neighbouring bins by neighbouring lanes: a line at a time)
        if (lg[i]) atomicAdd(&hist.g[h + i], lg[i]);
        if (lc[i]) atomicAdd(&hist.c[h + i], lc[i]);
    }
    // the groups' sums: sixteen neighbouring bins a thread, in an order that spreads the LDS banks
    constexpr uint32_t PER = BINS / JOB_THREADS;
    static_assert(PER * 4u == GROUP_BINS, "four threads per group");
    uint32_t sg = 0;
    unsigned long long sc = 0;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) {
        const uint32_t b = tid * PER + ((i + tid) & (PER - 1u));
        sg += lg[b]; sc += lc[b];
    }
    sg += __shfl_xor(sg, 1, 64); sg += __shfl_xor(sg, 2, 64);
    sc += __shfl_xor(sc, 1, 64); sc += __shfl_xor(sc, 2, 64);
    if ((tid & 3u) == 0u) {
        if (sg) atomicAdd(&hist.g[h + BINS + (tid >> 2)], sg);
        if (sc) atomicAdd(&hist.c[h + BINS + (tid >> 2)], sc);
    }
}

// ------------------------------------------------------------------ best step from scratch
struct Step { float slope; uint32_t tgt, dg; };

// Best step of job j from its current state under the free capacity.  The
// candidates are read four at a time, so that their loads (and those of the
// current state) are in flight together; positions past the end repeat the
// last one and are ignored.
template <int PASS>
__device__ __forceinline__ Step best_step(const Ctx &X, uint32_t j, int32_t gi, uint32_t g_held, uint32_t ci,
                                          unsigned long long freeG, unsigned long long freeC) {
    const GridDev &grid = X.grid;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem, m_top = n_mem - 1;
    const uint32_t ju = job_of(X, j);
    const uint32_t s0 = X.tb.seg_off[ju], ns = X.tb.seg_off[ju + 1] - s0;
    const uint64_t jbase = (uint64_t)n_rows * (s0 - X.tb.seg_off[X.jb]);
    const float ref = X.ref_thr[ju];
    Step out = {0.f, 0u, 0u};
    if (PASS == 0) {
        const uint64_t row = jbase + (uint64_t)(ci * n_mem + m_top) * ns;      // the CPU level the job holds
        const uint32_t g_cur = gi < 0 ? 0u : X.tb.seg_g[s0 + gi];
        const float cur = gi < 0 ? 0.f : X.curve_thr[row + gi];
        const unsigned long long c_cur = gi < 0 ? 0ull : cpu_cost(grid, ci, g_cur);
        for (uint32_t b = (uint32_t)(gi + 1); b < ns; b += 4) {
            uint32_t gs[4];
            float vs[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t s = b + u < ns ? b + u : ns - 1;
                gs[u] = X.tb.seg_g[s0 + s];
                vs[u] = X.curve_thr[row + s];
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t s = b + u;
                if (s >= ns) return out;
                const uint32_t dg = gs[u] - g_cur;
                if (dg > freeG) return out;                    // amounts ascend: nothing further on fits
                const float v = vs[u];
                if (!(v > cur)) continue;
                if (cpu_cost(grid, ci, g_cur + dg) - c_cur > freeC) continue;
                float sl = (v - cur) / ref;
                sl = sl / (float)dg;
                if (sl > out.slope) { out.slope = sl; out.tgt = s; out.dg = dg; }
            }
        }
    } else if (gi >= 0) {
        const float cur = X.best_thr[jbase + (uint64_t)(ci * n_mem + m_top) * ns + gi];
        const unsigned long long have = cpu_cost(grid, ci, g_held);
        for (uint32_t b = ci + 1; b < grid.n_cpu; b += 4) {
            float vs[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t c = b + u < grid.n_cpu ? b + u : grid.n_cpu - 1;
                vs[u] = X.best_thr[jbase + (uint64_t)(c * n_mem + m_top) * ns + gi];
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t c = b + u;
                if (c >= grid.n_cpu) return out;
                const unsigned long long dc = cpu_cost(grid, c, g_held) - have;
                if (dc > freeC) return out;                    // levels ascend
                const float v = vs[u];
                if (!(v > cur)) continue;
                float sl = (v - cur) / ref;
                sl = sl / (float)dc;
                if (sl > out.slope) { out.slope = sl; out.tgt = c; }
            }
        }
    }
    return out;
}

// ------------------------------------------------------------------ apply the selected prefix
// The threshold from the two histogram levels: steps with (key >> 8) > thr24
// are applied; freeG / freeC = what is left after them.
struct Selection { long long thr24; unsigned long long freeG, freeC; };

// Applies the selected prefix (steps with key >> 8 above thr24) to job j and
// caches its best next step under what is left.
template <int PASS, bool NEAR = false>
__device__ __forceinline__ void apply_job(const Ctx &X, const JobState &st, const HullBuf &H, uint32_t j, long long thr24,
                                          unsigned long long freeG, unsigned long long freeC, const WalkAhead &W = {}) {
    {
        const uint32_t jrel = j - X.jb;
        const uint32_t width = walk_width<PASS>(X, H);
        const Floor fl = PASS == 0 ? floor_of(st, jrel) : Floor{-1, 0u, RK_JOB_NORMAL};
        const uint32_t s0 = PASS == 0 ? X.tb.seg_off[job_of(X, j)] : 0u;         // (on its way while the walk is read)
        int32_t gi = PASS == 0 ? fl.gi : st.gi[jrel];
        uint32_t g_held = PASS == 0 ? 0u : st.g[jrel];
        uint32_t ci = PASS == 0 ? fl.ci : st.ci[jrel];
        uint32_t k = 0, key = 0;
        size_t e = 0;
        bool open_end = true;                                      // no step left out so far
        Step next = {0.f, 0u, 0u};                                 // the first step left out, when it is among those in registers
        unsigned long long next_dc = 0;
        bool near = false;
        if constexpr (NEAR) {
#pragma unroll
            for (uint32_t u = 0; u < AHEAD; ++u) {
                if (!open_end || u >= width) continue;
                k = u;
                key = W.key[u];
                if (!key || (long long)(key >> 8) <= thr24) {
                    open_end = false;
                    near = true;
                    next = Step{W.raw[u], W.tgt[u], W.dg[u]};
                    next_dc = W.dc[u];
                    continue;
                }
                if (PASS == 0) gi = (int32_t)W.tgt[u]; else ci = W.tgt[u];
                k = u + 1;
            }
        }
        for (uint32_t k0 = NEAR ? AHEAD : 0u; k0 < width && open_end; k0 += 4) {   // four steps per round of loads
            uint32_t keys[4], tgts[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                const uint32_t kk = k0 + u < width ? k0 + u : width - 1;
                keys[u] = H.key[(size_t)kk * H.stride + jrel];
                tgts[u] = H.tgt[(size_t)kk * H.stride + jrel];
            }
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                if (!open_end || k0 + u >= width) continue;
                k = k0 + u;
                e = (size_t)k * H.stride + jrel;
                key = keys[u];
                if (!key || (long long)(key >> 8) <= thr24) { open_end = false; continue; }
                if (PASS == 0) gi = (int32_t)tgts[u]; else ci = tgts[u];
                k = k0 + u + 1;
            }
        }
        if (k == width) key = 0;
        if (PASS == 0) {
            g_held = gi < 0 ? 0u : X.tb.seg_g[s0 + gi];
            st.gi[jrel] = gi;
            st.g[jrel] = g_held;
        }
        st.ci[jrel] = ci;
        // the job's best next step: the walk's next step if it still fits, else a fresh search
        Step nx = {0.f, 0u, 0u};
        if (key) {
            if (!near) { next = Step{H.raw[e], H.tgt[e], H.dg[e]}; next_dc = H.dc[e]; }
            if (next.dg <= freeG && next_dc <= freeC) nx = next;
            else nx = best_step<PASS>(X, j, gi, g_held, ci, freeG, freeC);
        }
        st.step_slope[jrel] = nx.slope;
        st.step_tgt[jrel] = (uint16_t)nx.tgt;
        st.step_dg[jrel] = (uint16_t)nx.dg;
    }
}

// One thread per job.  Every wavefront derives the threshold from the cut of
// level 0, which k_hist<1> left, and the histogram of level 1 (same inputs,
// same result in all of them).  10,000 jobs: 18.1 -> 10.5 us, while every
// workgroup read both histograms whole.
template <int PASS>
__global__ __launch_bounds__(JOB_THREADS) void k_apply(Ctx X, JobState st, HullBuf H, Hist hist) {
    const uint32_t rnd = blockIdx.y, tid = threadIdx.x;
    if (PASS == 1 && st.cpu_steps[rnd] == 0u) return;       // empty pass: every job keeps the CPU level it has
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    unsigned long long capG, capC;
    pass_caps<PASS>(X.R, cl, st, rnd, capG, capC);
    const size_t h1 = hist_at(rnd, PASS, 1);
    const GroupSums sums = load_groups(hist.g + h1, hist.c + h1);            // (all zero where level 0 has no cut)
    const Cut c0 = hist.cut[rnd];
    Selection sel;
    sel.thr24 = -1;
    unsigned long long usedG = c0.baseG, usedC = c0.baseC;
    if (c0.bin >= 0) {
        const Cut c1 = find_cut_groups(hist.g + h1, hist.c + h1, sums, c0.baseG, c0.baseC, capG, capC);
        sel.thr24 = ((long long)c0.bin << 12) + (long long)c1.bin;           // c1.bin = -1: the whole of c0.bin fits as well
        usedG = c1.baseG; usedC = c1.baseC;
    }
    sel.freeG = capG - usedG;
    sel.freeC = capC - usedC;

    const uint32_t jl = blockIdx.x * JOB_THREADS + tid;
    if (J0 + jl < J1) apply_job<PASS>(X, st, H, J0 + jl, sel.thr24, sel.freeG, sel.freeC);
    // the capacity left goes to the tail through a second pair of words: the
    // pass's starting capacity (free_c) is still being read by other workgroups
    if (blockIdx.x == 0 && tid == 0) { st.free_g[rnd] = sel.freeG; st.free_g[X.R.n_rounds + rnd] = sel.freeC; }
}

// ------------------------------------------------------------------ step by step on what is left
// The same search as best_step, by a whole wavefront: every lane passes the
// same arguments and gets the same result.  Lanes take one candidate target
// each, so the loads of a job's amounts and values go out together instead of
// one after the other.
template <int PASS>
__device__ __forceinline__ Step best_step_wave(const Ctx &X, uint32_t j, int32_t gi, uint32_t g_held, uint32_t ci,
                                               unsigned long long freeG, unsigned long long freeC) {
    const GridDev &grid = X.grid;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem, m_top = n_mem - 1;
    const uint32_t ju = job_of(X, j);
    const uint32_t s0 = X.tb.seg_off[ju], ns = X.tb.seg_off[ju + 1] - s0;
    const uint64_t jbase = (uint64_t)n_rows * (s0 - X.tb.seg_off[X.jb]);
    const float ref = X.ref_thr[ju];
    unsigned long long mine = 0;                                // (slope bits, inverted target): lowest target wins ties
    uint32_t mine_dg = 0;
    if (PASS == 0) {
        const uint32_t g_cur = gi < 0 ? 0u : X.tb.seg_g[s0 + gi];
        const uint64_t row = jbase + (uint64_t)(ci * n_mem + m_top) * ns;
        const float cur = gi < 0 ? 0.f : X.curve_thr[row + gi];
        const unsigned long long c_cur = gi < 0 ? 0ull : cpu_cost(grid, ci, g_cur);
        for (uint32_t b = (uint32_t)(gi + 1); b < ns; b += 64) {
            const uint32_t s = b + lane;
            const bool in = s < ns;
            uint32_t dg = 0;
            float v = 0.f;
            if (in) { dg = X.tb.seg_g[s0 + s] - g_cur; v = X.curve_thr[row + s]; }
            const bool fits = in && dg <= freeG;
            if (fits && v > cur && cpu_cost(grid, ci, g_cur + dg) - c_cur <= freeC) {
                float sl = (v - cur) / ref;
                sl = sl / (float)dg;
                const unsigned long long key = ((unsigned long long)__float_as_uint(sl) << 32) | (0xFFFFFFFFu - s);
                if (key > mine) { mine = key; mine_dg = dg; }
            }
            if (__ballot(in && !fits)) break;                   // amounts ascend: nothing further on fits
        }
    } else if (gi >= 0) {
        const float cur = X.best_thr[jbase + (uint64_t)(ci * n_mem + m_top) * ns + gi];
        const unsigned long long have = cpu_cost(grid, ci, g_held);
        for (uint32_t b = ci + 1; b < grid.n_cpu; b += 64) {
            const uint32_t c = b + lane;
            const bool in = c < grid.n_cpu;
            unsigned long long dc = 0;
            float v = 0.f;
            if (in) {
                dc = cpu_cost(grid, c, g_held) - have;
                v = X.best_thr[jbase + (uint64_t)(c * n_mem + m_top) * ns + gi];
            }
            const bool fits = in && dc <= freeC;
            if (fits && v > cur) {
                float sl = (v - cur) / ref;
                sl = sl / (float)dc;
                const unsigned long long key = ((unsigned long long)__float_as_uint(sl) << 32) | (0xFFFFFFFFu - c);
                if (key > mine) mine = key;
            }
            if (__ballot(in && !fits)) break;                   // levels ascend
        }
    }
    const uint32_t mine_sl = (uint32_t)(mine >> 32), mine_s = 0xFFFFFFFFu - (uint32_t)mine;
    const uint32_t best = wave_max_u32_rows(mine_sl);
    Step out = {0.f, 0u, 0u};
    if (best) {                                                 // a positive slope; the lowest target that has it
        out.slope = __uint_as_float(best);
        out.tgt = wave_min_u32_rows(mine_sl == best ? mine_s : 0xFFFFFFFFu);
        if (PASS == 0) {
            const unsigned long long holder = __ballot(mine_sl == best && mine_s == out.tgt);   // one lane
            out.dg = (uint32_t)__builtin_amdgcn_readlane((int)mine_dg, __builtin_amdgcn_readfirstlane((int)__ffsll((long long)holder) - 1));
        }
    }
    return out;
}

// The same search over amounts that lie in LDS, a lane each: v, g = the lane's amount's value and GPUs, `at` = the amount the
// job is at (-1: it holds nothing).
template <int PASS>
__device__ __forceinline__ Step best_step_listed(const GridDev &grid, const uint32_t *lvl, float v, uint32_t g, float ref, int32_t at, uint32_t ns,
                                                 uint32_t g_held, uint32_t ci, uint32_t roomG, uint32_t roomC) {
    const uint32_t lane = threadIdx.x & 63u;
    const float cur = at < 0 ? 0.f : __uint_as_float(wave_lane_u32(__float_as_uint(v), (uint32_t)at));
    uint32_t mine = 0, dg = 0;
    if (PASS == 0) {
        dg = g - (at < 0 ? 0u : wave_lane_u32(g, (uint32_t)at));
        const unsigned long long dc = (unsigned long long)lvl[ci] * (grid.cpu_mode ? dg : (at < 0 ? 1u : 0u));
        if ((int32_t)lane > at && lane < ns && v > cur && dg <= roomG && dc <= roomC) {
            float sl = (v - cur) / ref;
            sl = sl / (float)dg;
            mine = __float_as_uint(sl);
        }
    } else if ((int32_t)lane > at && lane < ns && v > cur) {
        const unsigned long long times = grid.cpu_mode ? g_held : 1u;
        const unsigned long long dc = (unsigned long long)lvl[lane] * times - (unsigned long long)lvl[at] * times;
        if (dc <= roomC) {
            float sl = (v - cur) / ref;
            sl = sl / (float)(uint32_t)dc;
            mine = __float_as_uint(sl);
        }
    }
    const uint32_t best = wave_max_u32_rows(mine);
    Step out = {0.f, 0u, 0u};
    if (best) {
        out.slope = __uint_as_float(best);
        out.tgt = (uint32_t)__ffsll((long long)__ballot(mine == best)) - 1u;       // the lowest lane is the smallest amount
        out.dg = PASS == 0 ? wave_lane_u32(dg, out.tgt) : 0u;
    }
    return out;
}

// A barrier that orders LDS only: loads from memory that are on their way stay there.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The list that the first wavefront works on, a job per lane: the jobs, their cached steps, the steps behind those (next_tgt
// TAIL_NONE: not known), how many amounts they have, and per wavefront the best step that is not in the list; and what the
// first wavefront leaves for the others.  Where steps are taken one by one: what every wavefront offers, its best exact step with its
// costs and its best bound, in two copies used in turn.
struct TailOffer { uint32_t slope, job, dg, dc, bound, bound_job; };
constexpr uint32_t TAIL_LIST = 64, TAIL_PER = 4, TAIL_NONE = 0xFFFFFFFFu;
// Steps taken one by one, at most.  Room for so many halves of a step, like all there are or, behind the first, like those
// offered, goes to lists (more CPUs of a step do not count: the sums stay words).
constexpr uint32_t TAIL_SINGLY = 5, TAIL_MANY_STEPS = 7, TAIL_MANY_OFFERED = 4, TAIL_MOST_CPUS = 1u << 20;
struct TailShared {
    unsigned long long free_g, free_c, best, moved;
    float slope[TAIL_LIST], next_slope[TAIL_LIST], ref[TAIL_LIST];
    uint32_t job[TAIL_LIST], dg[TAIL_LIST], dc[TAIL_LIST], next_tgt[TAIL_LIST], next_dg[TAIL_LIST], next_dc[TAIL_LIST], ns[TAIL_LIST];
    uint32_t rest[TAIL_THREADS / 64], rest_job[TAIL_THREADS / 64], lvl[RK_MAX_CPU_LEVELS], what;
    TailOffer offers[2][TAIL_THREADS / 64];
    uint32_t steps[TAIL_THREADS / 64], steps_g[TAIL_THREADS / 64], steps_c[TAIL_THREADS / 64];   // of a wavefront: exact steps, their GPUs and CPUs
};
enum { TAIL_END = 0, TAIL_LOOK = 1, TAIL_SEARCH = 2 };
// dynamic LDS of tail_run: 8 bytes per job, then values and GPUs of the list's amounts
__host__ __device__ constexpr size_t tail_scratch_bytes(uint32_t max_jobs) { return ((size_t)max_jobs * 8 + 15) & ~(size_t)15; }
__host__ __device__ constexpr size_t tail_lds_bytes(uint32_t max_jobs) { return tail_scratch_bytes(max_jobs) + TAIL_LIST * 64 * 8; }

// Workgroup of T threads; lds = tail_lds_bytes(max_jobs) of scratch; at most KMAX * T jobs.  Starts from the state k_apply /
// apply_job left in st.  A thread owns every T-th job, whose cached steps stay in its registers.
//
// A step is a chain that nothing else hides, so what counts is its length.  The wavefronts find the jobs with the best steps
// together, TAIL_PER each, the steps behind those, and lay the jobs' amounts into LDS; the first wavefront then takes steps from
// this list by itself, a job per lane, without barriers, for as long as the best of the list comes before everything that is
// not in it.  Which steps are in the list does not change the result: a step that is not among the best of its wavefront ends
// the list's turn before it could have been taken.  28 steps of 3,333 jobs 70 -> 28 us, 10 steps and 5 bounds of 10,000
// jobs 39 -> 18 us.
// A list costs about 3 us, a step of its own 1.3 in a round of up to 2,048 jobs (2.3 with 12 jobs per thread): all wavefronts
// offer their best, find the best offer behind one barrier, and the winner finds its next step from what was on its way
// meanwhile.  So those rounds take steps one by one where there will be few.  How many is foretold by what is free divided by what
// the steps of all jobs need on average, and again, when the first is known, from what is free behind it and from the steps
// that the wavefronts offer.  The lines lie at 3.5 steps and at two more: of 99 rounds of drawn sizes, those below both took one to
// six steps, with few exceptions, and up to 5.7 us less one by one, those above either four to 35 and up to 27 us less from
// lists.  The sixth step goes to a list in any case, and where a list has many bounds to search it is given up and the steps
// are few again.  All steps from lists, all one by one, and this way: 300 jobs, one step 41.1, 38.4 and 38.5 us a round's allocation;
// 500 jobs on coarse curves, one step 40.7, 38.2 and 37.9, four groups of bounds 70.6, 57.0 and 60.0; 2,000 jobs, three groups 91.3, 73.9 and 81.9; 800
// jobs, 24 steps 59.0, 75.4 and 59.0; 1,000 alike, 250 steps 144, 362 and 144; the 56 drawn rounds of up to 512 jobs 2.45,
// 2.57 and 2.43 ms together, the 29 of up to 1,024 1.58, 1.68 and 1.56, the 25 of more 1.65, 1.77 and 1.66.
// Neighbours of jobs that are all alike come first one after the other: in rounds of up to 2,048 jobs, where the loads are few,
// a wavefront has only TAIL_PER neighbours each, and all of them are in one list (250 steps of 1,000 such jobs 141 us instead of
// 415; 364 before); 10,000 jobs read that way take 6 us more.
template <int PASS, int KMAX, int T>
__device__ __forceinline__ void tail_run(const Ctx &X, const JobState &st, uint32_t rnd, uint32_t J0, uint32_t J1,
                                         unsigned long long freeG, unsigned long long freeC, uint32_t max_jobs,
                                         void *lds, TailShared &S) {
    constexpr uint32_t WAVES = T / 64, PER = TAIL_PER, NONE = TAIL_NONE;
    constexpr uint32_t MANY = 8;                                   // bounds that lists make exact one by one
    static_assert(WAVES <= 16 && PER * WAVES <= TAIL_LIST, "lists of whole wavefronts");
    uint16_t *tgt = static_cast<uint16_t *>(lds);                  // target of the cached step (segment index or CPU level)
    int16_t *gi = reinterpret_cast<int16_t *>(tgt + max_jobs);     // granted segment index, -1 = none
    uint16_t *ci = reinterpret_cast<uint16_t *>(gi + max_jobs);    // granted CPU level
    uint16_t *gh = ci + max_jobs;                                  // GPUs held (CPU pass)
    float *const amount_v = reinterpret_cast<float *>(static_cast<unsigned char *>(lds) + tail_scratch_bytes(max_jobs));
    uint32_t *const amount_g = reinterpret_cast<uint32_t *>(amount_v + TAIL_LIST * 64);
    uint32_t *const lvl = S.lvl;                                   // CPU levels, for indexing by lane

    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t nj = J1 - J0, jrel0 = J0 - X.jb;
    // the thread's first job: jobs of a wavefront are PER neighbours each where that costs no more loads to speak of
    const uint32_t own = KMAX <= 2 ? (lane / PER * WAVES + wave) * PER + lane % PER : tid;
    const GridDev &grid = X.grid;

    // CPUs a step costs (saturated to 32 bits: the free CPUs fit in 32)
    auto need_cpus = [&](int32_t g_i, uint32_t c_i, uint32_t target, uint32_t gpus) -> uint32_t {
        unsigned long long c;
        if (PASS == 0) {
            const unsigned long long times = grid.cpu_mode ? gpus : (g_i < 0 ? 1u : 0u);
            c = (unsigned long long)lvl[c_i] * times;
        } else {
            const unsigned long long times = grid.cpu_mode ? gpus : 1u;
            c = (unsigned long long)lvl[target] * times - (unsigned long long)lvl[c_i] * times;
        }
        return c > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)c;
    };

    if (nj == 0) {                                                 // the same in all threads
        if (PASS == 0 && tid == 0) st.free_c[rnd] = freeC;
        return;
    }
    if (tid < RK_MAX_CPU_LEVELS) lvl[tid] = grid.cpu_levels[tid];
    float slope[KMAX];                                             // cached best step of the thread's jobs:
    uint32_t dg[KMAX], dc[KMAX];                                   // > 0 exact, < 0 an upper bound, 0 none; its GPUs, CPUs
    constexpr bool SMALL = KMAX <= 2;
    uint32_t seg_lo[SMALL ? KMAX : 1], seg_hi[SMALL ? KMAX : 1];   // where the jobs' amounts are
    float ref_thr[SMALL ? KMAX : 1];
    auto find_amounts = [&]() {                                    // (not waited for before a wavefront knows its best step)
#pragma unroll
        for (int k = 0; k < (SMALL ? KMAX : 0); ++k) {
            const uint32_t jl = own + (uint32_t)k * T, slot = job_of(X, J0 + (jl < nj ? jl : nj - 1u));
            seg_lo[k] = X.tb.seg_off[slot];
            seg_hi[k] = X.tb.seg_off[slot + 1];
            ref_thr[k] = X.ref_thr[slot];
        }
    };
    {
        int32_t g_i[KMAX];
        uint32_t c_i[KMAX], target[KMAX], gpus[KMAX];
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {                           // all loads go out before the first is used
            const uint32_t jl = own + (uint32_t)k * T;
            const uint32_t at = jrel0 + (jl < nj ? jl : nj - 1u);
            g_i[k] = st.gi[at];
            c_i[k] = st.ci[at];
            target[k] = st.step_tgt[at];
            gpus[k] = PASS == 0 ? st.step_dg[at] : st.g[at];
            slope[k] = st.step_slope[at];
        }
        if constexpr (KMAX == 1) find_amounts();                   // (with two jobs per thread only where steps are taken one by one: lists would wait for it)
        __syncthreads();                                           // the levels are in LDS
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const uint32_t jl = own + (uint32_t)k * T;
            const bool have = jl < nj;
            const uint32_t need = need_cpus(g_i[k], c_i[k], target[k], gpus[k]);
            slope[k] = have ? slope[k] : 0.f;
            dg[k] = PASS == 0 && have ? gpus[k] : 0u;
            dc[k] = have ? need : 0u;
            if (have) {
                tgt[jl] = (uint16_t)target[k];
                gi[jl] = (int16_t)g_i[k];
                ci[jl] = (uint16_t)c_i[k];
                if (PASS == 1) gh[jl] = (uint16_t)gpus[k];
            }
        }
    }

    // A cached step that stops fitting is not searched anew at once: it is
    // kept, negated, as an upper bound of whatever the job can still do (the
    // job's state is unchanged and the capacity only shrank).  A step is
    // taken when it comes before every other step and every such bound under
    // the tie rule (lower job index first); a bound that comes first is made
    // exact.
    auto key_of = [](float v, uint32_t jl) -> unsigned long long {
        return ((unsigned long long)__float_as_uint(v) << 32) | (0xFFFFFFFFu - jl);
    };
    auto one = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    auto room = [&](unsigned long long x) { return one(x > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)x); };
    uint32_t asked = 0;                                         // (the first wavefront's) bounds made exact one by one
    uint32_t moved = 0;                                         // bit k = the thread's k-th job took a step here
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem, first_seg = X.tb.seg_off[X.jb];
    // their threads make the bounds that could win exact: those whose key comes before that of the best exact step
    auto search = [&](unsigned long long best) {
        uint32_t todo = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const float v = slope[k];
            if (v < 0.f && key_of(-v, own + (uint32_t)k * T) > best) todo |= 1u << k;
        }
        for (; todo; todo &= todo - 1u) {                       // (the register arrays are only ever indexed by constants)
            const uint32_t at = (uint32_t)__ffs((int)todo) - 1u, jl = own + at * T;
            const uint32_t held = PASS == 0 ? 0u : gh[jl];
            const Step nx = best_step<PASS>(X, J0 + jl, gi[jl], held, ci[jl], freeG, freeC);
            const uint32_t need = need_cpus(gi[jl], ci[jl], nx.tgt, PASS == 0 ? nx.dg : held);
            tgt[jl] = (uint16_t)nx.tgt;
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if ((uint32_t)k == at) { slope[k] = nx.slope; dg[k] = PASS == 0 ? nx.dg : 0u; dc[k] = need; }
        }
    };
    // What the wavefront has read of the job with its best step: a lane per amount (GPU pass: its GPUs too).
    uint32_t kept_job = NONE, kept_g = 0, kept_n = 0, turn = 0, singly = 0;
    float kept_v = 0.f, kept_ref = 1.f;
    bool one_by_one = false;
    // is there room for so many halves of a step, if steps are like these?
    auto room_for = [&](uint32_t halves, uint32_t n, uint32_t sum_g, uint32_t sum_c, uint32_t roomG, uint32_t roomC) {
        return 2ull * roomG * n >= (unsigned long long)sum_g * halves && 2ull * roomC * n >= (unsigned long long)sum_c * halves;
    };
    bool none = false;                                          // (no job has a step, as in most CPU passes of small rounds)
    if constexpr (SMALL) {
        uint32_t n = 0, sum_g = 0, sum_c = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const bool step = slope[k] > 0.f;
            n += (uint32_t)__popcll(__ballot(step));
            sum_g += step ? dg[k] : 0u;
            sum_c += step ? (dc[k] < TAIL_MOST_CPUS ? dc[k] : TAIL_MOST_CPUS) : 0u;
        }
        if (n) { if (PASS == 0) sum_g = wave_sum_u32(sum_g); sum_c = wave_sum_u32(sum_c); }
        if (lane == 0) { S.steps[wave] = n; S.steps_g[wave] = sum_g; S.steps_c[wave] = sum_c; }
        lds_barrier();
        const bool in = (lane & 15u) < WAVES;                   // (sums over a row of lanes: a wavefront's in each)
        n = one(row_sum_u32(in ? S.steps[lane & (WAVES - 1u)] : 0u));
        none = n == 0u;
        if (!none) {
            sum_g = PASS == 0 ? one(row_sum_u32(in ? S.steps_g[lane & (WAVES - 1u)] : 0u)) : 0u;
            sum_c = one(row_sum_u32(in ? S.steps_c[lane & (WAVES - 1u)] : 0u));
            one_by_one = !room_for(TAIL_MANY_STEPS, n, sum_g, sum_c, room(freeG), room(freeC));
            if (KMAX > 1 && one_by_one) find_amounts();
        }
    }
    while (!none) {
        if (PASS == 0 ? freeG == 0 : freeC == 0) break;         // nothing can fit any more
        const uint32_t roomG = room(freeG), roomC = room(freeC);
        if constexpr (SMALL) {
            if (one_by_one) {
                // ---- one step, by all wavefronts: the thread's best exact step and best bound, then the wavefront's
                float vf = 0.f, vs = 0.f;
                uint32_t kf = 0, ks = 0;
#pragma unroll
                for (int k = 0; k < KMAX; ++k) {
                    float v = slope[k];
                    v = v > 0.f && ((PASS == 0 && dg[k] > roomG) || dc[k] > roomC) ? -v : v;
                    slope[k] = v;
                    if (v > vf) { vf = v; kf = (uint32_t)k; }
                    if (-v > vs) { vs = -v; ks = (uint32_t)k; }
                }
                const bool second = KMAX > 1 && kf != 0u;
                const uint32_t jf = own + kf * T, js = own + ks * T, bf = __float_as_uint(vf), bs = __float_as_uint(vs);
                const uint32_t mf = wave_max_u32_rows(bf), ms = wave_max_u32_rows(bs);
                uint32_t jm = NONE, jb = NONE, dgm = 0, dcm = 0;
                if (mf) {
                    jm = wave_min_u32_rows(bf == mf ? jf : NONE);
                    const uint32_t at = (uint32_t)__ffsll((long long)__ballot(bf == mf && jf == jm)) - 1u;
                    dgm = wave_lane_u32(second ? dg[KMAX - 1] : dg[0], at);
                    dcm = wave_lane_u32(second ? dc[KMAX - 1] : dc[0], at);
                    if (jm != kept_job) {                       // what its next step needs is on its way before it wins
                        const uint32_t s0 = wave_lane_u32(second ? seg_lo[KMAX - 1] : seg_lo[0], at), n = wave_lane_u32(second ? seg_hi[KMAX - 1] : seg_hi[0], at) - s0;
                        kept_ref = __uint_as_float(wave_lane_u32(__float_as_uint(second ? ref_thr[KMAX - 1] : ref_thr[0]), at));
                        kept_job = jm;
                        kept_n = n;
                        const uint64_t base = (uint64_t)n_rows * (s0 - first_seg);
                        if (PASS == 0) {
                            const uint32_t i = lane < n ? lane : n - 1u;
                            kept_g = X.tb.seg_g[s0 + i];
                            kept_v = X.curve_thr[base + (uint64_t)(one(ci[jm]) * n_mem + n_mem - 1u) * n + i];
                        } else {
                            const uint32_t c = lane < grid.n_cpu ? lane : grid.n_cpu - 1u;
                            kept_v = X.best_thr[base + (uint64_t)(c * n_mem + n_mem - 1u) * n + one((uint32_t)(int32_t)gi[jm])];
                        }
                    }
                }
                if (ms) jb = wave_min_u32_rows(bs == ms ? js : NONE);
                turn ^= 1u;
                if (lane == 0) S.offers[turn][wave] = TailOffer{mf, jm, dgm, dcm, ms, jb};
                lds_barrier();
                const TailOffer o = S.offers[turn][lane & (WAVES - 1u)];          // every row of 16 lanes has all of them
                const uint32_t top = one(row_max_u32(o.slope)), jw = one(row_min_u32(o.slope == top ? o.job : NONE));
                const uint32_t bound = one(row_max_u32(o.bound)), jbound = one(row_min_u32(o.bound == bound ? o.bound_job : NONE));
                if (bound && (bound > top || (bound == top && jbound < jw))) {    // a bound could win: make those exact
                    search(top ? key_of(__uint_as_float(top), jw) : 0ull);
                    continue;
                }
                if (!top) break;
                const uint32_t won = (uint32_t)__ffsll((long long)__ballot(o.slope == top && o.job == jw)) - 1u;       // (below WAVES)
                const uint32_t dg_won = wave_lane_u32(o.dg, won), dc_won = wave_lane_u32(o.dc, won);                   // (CPU pass: no GPUs)
                if (singly == 0u)                               // behind the best step, of those that are offered
                    one_by_one = !room_for(TAIL_MANY_OFFERED, (uint32_t)__popcll(__ballot(o.slope != 0u) & 0xFFFFull), one(row_sum_u32(o.slope ? o.dg : 0u)),
                                           one(row_sum_u32(o.slope ? (o.dc < TAIL_MOST_CPUS ? o.dc : TAIL_MOST_CPUS) : 0u)), roomG - dg_won, roomC - dc_won);
                if (one_by_one) {
                    freeG -= dg_won;
                    freeC -= dc_won;
                    if (wave == won) {
                        const bool owner = jf == jw && bf == top;
                        int32_t g_i = gi[jw];
                        uint32_t c_i = ci[jw];
                        if (PASS == 0) g_i = (int32_t)tgt[jw]; else c_i = tgt[jw];
                        const uint32_t held = PASS == 0 ? 0u : gh[jw];
                        Step nx = {0.f, 0u, 0u};
                        if (PASS == 0 ? freeG != 0 : freeC != 0)
                            nx = PASS == 1 || kept_n <= 64u
                                     ? best_step_listed<PASS>(grid, lvl, kept_v, kept_g, kept_ref, PASS == 0 ? (int32_t)one((uint32_t)g_i) : (int32_t)one(c_i),
                                                              PASS == 0 ? kept_n : grid.n_cpu, one(held), one(c_i), room(freeG), room(freeC))
                                     : best_step_wave<PASS>(X, J0 + jw, g_i, held, c_i, freeG, freeC);
                        if (owner) {
                            if (PASS == 0) gi[jw] = (int16_t)g_i; else ci[jw] = (uint16_t)c_i;
                            moved |= 1u << kf;
                            tgt[jw] = (uint16_t)nx.tgt;
                            const uint32_t need = need_cpus(g_i, c_i, nx.tgt, PASS == 0 ? nx.dg : held);
#pragma unroll
                            for (int k = 0; k < KMAX; ++k)
                                if ((uint32_t)k == kf) { slope[k] = nx.slope; dg[k] = PASS == 0 ? nx.dg : 0u; dc[k] = need; }
                        }
                    }
                    one_by_one = ++singly < TAIL_SINGLY;
                    continue;
                }
            }
        }
        // ---- the thread's best step or bound and its second (a thread's jobs come in rising order, so the first of equal
        // slopes is the lower job)
        float a1 = 0.f, a2 = 0.f;
        uint32_t k1 = 0, k2 = 0;
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            const float v = slope[k], a = fabsf(v);
            if (v > 0.f && ((PASS == 0 && dg[k] > roomG) || dc[k] > roomC)) slope[k] = -v;
            if (a > a1) { a2 = a1; k2 = k1; a1 = a; k1 = (uint32_t)k; }
            else if (a > a2) { a2 = a; k2 = (uint32_t)k; }
        }
        // ---- the wavefront's best, word by word: the highest slope, then the lowest job among those that have it
        const uint32_t j1 = own + k1 * T;
        uint32_t mine = NONE, job = NONE;                       // the thread's place in the list; lane p: the job of place p
        uint32_t left = __float_as_uint(a1);
#pragma unroll
        for (uint32_t p = 0; p < PER; ++p) {
            const uint32_t top = wave_max_u32_rows(left);
            if (!top) break;
            const uint32_t jm = wave_min_u32_rows(left == top ? j1 : NONE);
            if (left == top && j1 == jm) { mine = wave * PER + p; left = 0u; }
            if (lane == p) job = jm;
        }
        {
            const uint32_t r = mine == NONE ? left : __float_as_uint(a2), rj = own + (mine == NONE ? k1 : k2) * T;
            const uint32_t top = wave_max_u32_rows(r);
            const uint32_t jm = top ? wave_min_u32_rows(r == top ? rj : NONE) : NONE;
            if (lane == 0) { S.rest[wave] = top; S.rest_job[wave] = jm; }
        }
        if (mine != NONE) {
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if ((uint32_t)k == k1) { S.slope[mine] = slope[k]; S.dg[mine] = dg[k]; S.dc[mine] = dc[k]; }
        }
        // ---- their amounts go into LDS
        rs_wave_order();
        uint32_t s0 = 0, ns = 0, row = 0, to = 0, held = 0, step_g = 0, step_c = 0;
        float ref = 1.f, step = 0.f;
        if (job != NONE) {
            const uint32_t slot = job_of(X, J0 + job);
            ref = X.ref_thr[slot];
            s0 = X.tb.seg_off[slot];
            ns = X.tb.seg_off[slot + 1] - s0;
            row = PASS == 0 ? (uint32_t)ci[job] : (uint32_t)(int32_t)gi[job];
            S.ref[wave * PER + lane] = ref;
            to = tgt[job];
            held = PASS == 1 ? gh[job] : 0u;
            step = S.slope[wave * PER + lane]; step_g = S.dg[wave * PER + lane]; step_c = S.dc[wave * PER + lane];
        }
        if (lane < PER) { S.job[wave * PER + lane] = job; S.ns[wave * PER + lane] = ns; }
        {
            float v[PER];
            uint32_t g[PER];
#pragma unroll
            for (uint32_t p = 0; p < PER; ++p) {
                const uint32_t n = wave_lane_u32(ns, p), s = wave_lane_u32(s0, p), r = wave_lane_u32(row, p);
                v[p] = 0.f; g[p] = 0u;
                if (n == 0u) continue;
                const uint64_t base = (uint64_t)n_rows * (s - first_seg);
                if (PASS == 0) {
                    const uint32_t i = lane < n ? lane : n - 1u;
                    g[p] = X.tb.seg_g[s + i];
                    v[p] = X.curve_thr[base + (uint64_t)(r * n_mem + n_mem - 1u) * n + i];
                } else {
                    const uint32_t c = lane < grid.n_cpu ? lane : grid.n_cpu - 1u;
                    v[p] = X.best_thr[base + (uint64_t)(c * n_mem + n_mem - 1u) * n + r];
                }
            }
#pragma unroll
            for (uint32_t p = 0; p < PER; ++p) {
                amount_v[(wave * PER + p) * 64u + lane] = v[p];
                if (PASS == 0) amount_g[(wave * PER + p) * 64u + lane] = g[p];
            }
            // The step behind a job's step, as if it were the next one taken: a step that others' leave no room for is a bound
            // like any other (one that still fits then is the best that fits).
            float next = 0.f;
            uint32_t next_tgt = NONE, next_g = 0, next_c = 0;
#pragma unroll
            for (uint32_t p = 0; p < PER; ++p) {
                const uint32_t n = wave_lane_u32(ns, p), dg_p = wave_lane_u32(step_g, p), dc_p = wave_lane_u32(step_c, p);
                if (!((int32_t)wave_lane_u32(__float_as_uint(step), p) > 0) || dg_p > roomG || dc_p > roomC || (PASS == 0 && n > 64u)) continue;
                const uint32_t to_p = wave_lane_u32(to, p), held_p = wave_lane_u32(held, p);
                const uint32_t level = PASS == 0 ? wave_lane_u32(row, p) : to_p;
                const Step nx = best_step_listed<PASS>(grid, lvl, v[p], g[p], __uint_as_float(wave_lane_u32(__float_as_uint(ref), p)), (int32_t)to_p,
                                                       PASS == 0 ? n : grid.n_cpu, held_p, level, roomG - dg_p, roomC - dc_p);
                if (lane == p) {
                    next = nx.slope > 0.f ? nx.slope : 0.f; next_tgt = nx.tgt; next_g = nx.dg;     // (not a number: none)
                    next_c = need_cpus((int32_t)to_p, level, nx.tgt, PASS == 0 ? nx.dg : held_p);
                }
            }
            if (lane < PER) {
                const uint32_t e = wave * PER + lane;
                S.next_slope[e] = next; S.next_tgt[e] = next_tgt; S.next_dg[e] = next_g; S.next_dc[e] = next_c;
            }
        }
        lds_barrier();
        // ---- the first wavefront takes steps from the list
        if (wave == 0) {
            const uint32_t jl = lane < PER * WAVES ? S.job[lane] : NONE, n_l = S.ns[lane];
            const bool have = jl != NONE;
            float v = have ? S.slope[lane] : 0.f;
            const float ref_l = have ? S.ref[lane] : 1.f, next_v = S.next_slope[lane];
            uint32_t d = have ? S.dg[lane] : 0u, c = have ? S.dc[lane] : 0u, t = have ? tgt[jl] : 0u, c_l = have ? ci[jl] : 0u;
            const uint32_t held_l = PASS == 1 && have ? gh[jl] : 0u, next_d = S.next_dg[lane], next_c = S.next_dc[lane];
            uint32_t next_t = S.next_tgt[lane];
            int32_t g_l = have ? gi[jl] : -1;
            const uint32_t r = lane < WAVES ? S.rest[lane] : 0u, rest = wave_max_u32_rows(r);
            const uint32_t rest_job = wave_min_u32_rows(lane < WAVES && r == rest ? S.rest_job[lane] : NONE);
            uint32_t what = TAIL_END, fg = roomG, fc = roomC;     // (what is free fits in 32 bits)
            bool took = false;
            for (;;) {
                if (PASS == 0 ? fg == 0u : fc == 0u) break;
                if (v > 0.f && ((PASS == 0 && d > fg) || c > fc)) v = -v;
                const uint32_t bits = __float_as_uint(fabsf(v)), top = wave_max_u32_rows(bits);
                if (!top) { what = rest ? TAIL_LOOK : TAIL_END; break; }
                const unsigned long long tops = __ballot(bits == top);
                uint32_t w = (uint32_t)__ffsll((long long)tops) - 1u, jw = wave_lane_u32(jl, w);
                if (tops & (tops - 1ull)) {                      // several have it: the lowest job
                    jw = wave_min_u32_rows(bits == top ? jl : NONE);
                    w = (uint32_t)__ffsll((long long)__ballot(bits == top && jl == jw)) - 1u;
                }
                if (top < rest || (top == rest && rest_job < jw)) { what = TAIL_LOOK; break; }
                const bool exact = (int32_t)wave_lane_u32(__float_as_uint(v), w) > 0;
                if (exact) {
                    if (PASS == 0) fg -= wave_lane_u32(d, w);
                    fc -= wave_lane_u32(c, w);
                    const bool known = wave_lane_u32(next_t, w) != NONE;
                    if (lane == w) {
                        took = true;
                        if (PASS == 0) g_l = (int32_t)t; else c_l = t;
                        v = next_v; t = next_t; d = next_d; c = next_c;
                        next_t = NONE;
                    }
                    if (known) continue;
                } else {                                         // a bound: are there others before the best exact step?
                    const uint32_t best = wave_max_u32_rows(v > 0.f ? bits : 0u);
                    if (__popcll(__ballot(v < 0.f && bits > best)) > 2 || ++asked > MANY) {
                        what = TAIL_SEARCH;
                        asked = 0;
                        break;
                    }
                }
                const int32_t g_w = (int32_t)wave_lane_u32((uint32_t)g_l, w);
                const uint32_t c_w = wave_lane_u32(c_l, w), held_w = PASS == 1 ? wave_lane_u32(held_l, w) : 0u, n = wave_lane_u32(n_l, w);
                Step nx;
                if (PASS == 1 || n <= 64u)
                    nx = best_step_listed<PASS>(grid, lvl, amount_v[w * 64u + lane], PASS == 0 ? amount_g[w * 64u + lane] : 0u,
                                                __uint_as_float(wave_lane_u32(__float_as_uint(ref_l), w)), PASS == 0 ? g_w : (int32_t)c_w,
                                                PASS == 0 ? n : grid.n_cpu, held_w, c_w, fg, fc);
                else
                    nx = best_step_wave<PASS>(X, J0 + jw, g_w, held_w, c_w, fg, fc);
                if (lane == w) {
                    t = nx.tgt;
                    v = nx.slope > 0.f ? nx.slope : 0.f; d = nx.dg;             // (not a number: none)
                    c = need_cpus(g_w, c_w, nx.tgt, PASS == 0 ? nx.dg : held_w);
                    next_t = NONE;                               // (what is behind the step that it was listed with is not behind this one)
                }
            }
            freeG = PASS == 0 ? fg : freeG; freeC = fc;
            if (have) {
                S.slope[lane] = v; S.dg[lane] = d; S.dc[lane] = c;
                tgt[jl] = (uint16_t)t; gi[jl] = (int16_t)g_l; ci[jl] = (uint16_t)c_l;
            }
            unsigned long long best = 0;
            if (what == TAIL_SEARCH) {                           // the list's best exact step
                const uint32_t bits = v > 0.f ? __float_as_uint(v) : 0u, top = wave_max_u32_rows(bits);
                if (top) best = key_of(__uint_as_float(top), wave_min_u32_rows(bits == top ? jl : NONE));
            }
            const unsigned long long m = __ballot(took);
            if (lane == 0) { S.free_g = freeG; S.free_c = freeC; S.best = best; S.moved = m; S.what = what; }
        }
        lds_barrier();
        freeG = S.free_g; freeC = S.free_c;
        const uint32_t what = S.what;
        if (mine != NONE) {
            if ((S.moved >> mine) & 1ull) moved |= 1u << k1;
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if ((uint32_t)k == k1) { slope[k] = S.slope[mine]; dg[k] = S.dg[mine]; dc[k] = S.dc[mine]; }
        }
        if (what == TAIL_END) break;
        if (what == TAIL_SEARCH) {                               // many bounds could win
            search(S.best);
            one_by_one = SMALL;
            singly = 0;
            if constexpr (SMALL && KMAX > 1) find_amounts();
        }
    }
    for (; moved; moved &= moved - 1u) {                        // only the jobs that took a step here changed since k_apply
        const uint32_t jl = own + ((uint32_t)__ffs((int)moved) - 1u) * T;
        if (PASS == 0) {
            const int32_t s_i = gi[jl];
            uint32_t s0;
            if constexpr (KMAX == 1) s0 = seg_lo[0]; else s0 = X.tb.seg_off[job_of(X, J0 + jl)];
            st.gi[jrel0 + jl] = s_i;
            st.g[jrel0 + jl] = s_i < 0 ? 0u : X.tb.seg_g[s0 + s_i];
        } else {
            st.ci[jrel0 + jl] = ci[jl];
        }
    }
    if (PASS == 0 && tid == 0) st.free_c[rnd] = freeC;          // what the CPU pass starts from
}

constexpr int TAIL_KMAX = (RK_MAX_JOBS_PER_ROUND + TAIL_THREADS - 1) / TAIL_THREADS;

template <int PASS>
__global__ __launch_bounds__(TAIL_THREADS) void k_tail(Ctx X, uint32_t max_jobs, JobState st) {
    extern __shared__ uint4 lds_dyn[];
    __shared__ TailShared shared;
    const uint32_t rnd = blockIdx.x;
    if (PASS == 1 && st.cpu_steps[rnd] == 0u) return;       // empty pass
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    tail_run<PASS, TAIL_KMAX, TAIL_THREADS>(X, st, rnd, J0, J1, st.free_g[rnd], st.free_g[X.R.n_rounds + rnd], max_jobs, lds_dyn, shared);
}

// ------------------------------------------------------------------ selection of a pass in one workgroup
// For rounds of at most SMALL_ROUND_JOBS jobs the histograms, the threshold,
// the application and the step-by-step tail of a pass run in one workgroup per
// round, with the histograms in LDS: one launch instead of six (a job per thread
// of 512 or 1,024, above 1,024 jobs two: KMAX).  The workgroup of the CPU pass
// also takes the memory step that ends the round.  Larger rounds use the same kernel for their CPU pass
// (KMAX = TAIL_KMAX, without the memory step) as long as all CPU walks together
// are short, which the host can tell from the grid:
// (CPU levels - 1) * jobs <= CPU_ONE_WG_STEPS.
// The histogram (48 KiB) and the tail's scratch share the
// dynamic LDS: the tail starts when the threshold is known.
constexpr uint32_t SMALL_ROUND_JOBS = 2048;
constexpr uint64_t CPU_ONE_WG_STEPS = 65536;
constexpr size_t SELECT_HIST_BYTES = (size_t)BINS * 12;

__device__ __forceinline__ void mem_wish_job(const Ctx &X, const JobState &st, uint32_t j, rk_assign *__restrict__ assign,
                                             double &cost_d, double &val_d);
__device__ bool mem_close_round(const Ctx &X, const int32_t *gi_of, const uint32_t *g_of, const uint32_t *ci_of, uint32_t rnd,
                                double wish, double val, rk_assign *__restrict__ assign, float *__restrict__ totals);

template <int PASS, int KMAX, int T>
__global__ __launch_bounds__(T) void k_select_small(Ctx X, uint32_t max_jobs, JobState st, HullBuf H,
                                                              rk_assign *__restrict__ assign, float *__restrict__ totals) {
    extern __shared__ unsigned long long lds_sel[];             // the histogram, then the tail's scratch
    unsigned long long *hc = lds_sel;                           // one histogram, used for level 0 and then level 1
    uint32_t *hg = reinterpret_cast<uint32_t *>(hc + BINS);
    __shared__ CutScratch cs;
    __shared__ TailShared shared;
    __shared__ double sums[2 * (T / 64)];
    const uint32_t rnd = blockIdx.x, tid = threadIdx.x;
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    const uint32_t nj = J1 - J0;
    // whether any job's CPU walk has a step at all (same in all threads): a large round knows it
    bool empty_pass = false;
    if (PASS == 1) {
        if (KMAX == TAIL_KMAX) empty_pass = st.cpu_steps[rnd] == 0u;
        else {
            bool any = false;
            for (uint32_t jl = tid; jl < nj; jl += T) any |= H.key[J0 + jl - X.jb] != 0u;
            empty_pass = __syncthreads_or(any) == 0;
        }
    }
    if (!empty_pass) {
        unsigned long long capG, capC;
        pass_caps<PASS>(X.R, cl, st, rnd, capG, capC);
        WalkAhead W;                                            // (a job per thread)
        if constexpr (KMAX == 1) walk_ahead<PASS>(X, H, tid < nj, J0 + tid - X.jb, W);
        for (uint32_t i = tid; i < BINS; i += T) { hg[i] = 0; hc[i] = 0; }
        __syncthreads();
        auto add = [&](auto level, int32_t want_top) {
            constexpr int LEVEL = decltype(level)::value;
            if constexpr (KMAX == 1) {
                if (tid < nj) hist_add<PASS, LEVEL, T>(X, H, W, J0 + tid - X.jb, want_top, hg, hc);
            } else {
                for (uint32_t jl = tid; jl < nj; jl += T) hist_add<PASS, LEVEL, T>(X, H, J0 + jl - X.jb, want_top, hg, hc);
            }
        };
        add(std::integral_constant<int, 0>{}, 0);
        __syncthreads();
        const Cut c0 = find_cut<T>(hg, hc, 0, 0, capG, capC, cs);
        Selection sel;
        sel.thr24 = -1;
        unsigned long long usedG = c0.baseG, usedC = c0.baseC;
        if (c0.bin >= 0) {                                      // uniform over the workgroup
            __syncthreads();                                    // the last look at level 0
            for (uint32_t i = tid; i < BINS; i += T) { hg[i] = 0; hc[i] = 0; }
            __syncthreads();
            add(std::integral_constant<int, 1>{}, c0.bin);
            __syncthreads();
            const Cut c1 = find_cut<T>(hg, hc, c0.baseG, c0.baseC, capG, capC, cs);
            sel.thr24 = ((long long)c0.bin << 12) + (long long)c1.bin;
            usedG = c1.baseG; usedC = c1.baseC;
        }
        sel.freeG = capG - usedG;
        sel.freeC = capC - usedC;
        if constexpr (KMAX == 1) {
            if (tid < nj) apply_job<PASS, true>(X, st, H, J0 + tid, sel.thr24, sel.freeG, sel.freeC, W);
        } else {
            for (uint32_t jl = tid; jl < nj; jl += T) apply_job<PASS>(X, st, H, J0 + jl, sel.thr24, sel.freeG, sel.freeC);
        }
        __syncthreads();                                        // the state in st is read back by the whole workgroup; the
                                                                // histogram's LDS passes to the tail
        tail_run<PASS, KMAX, T>(X, st, rnd, J0, J1, sel.freeG, sel.freeC, max_jobs, lds_sel, shared);
    }
    if (PASS == 0 || KMAX == TAIL_KMAX) return;                 // (large rounds: a thread per job does it faster, k_mem_wish)
    // memory: every thread writes the wishes of its jobs, the first wavefront closes the round
    __syncthreads();                                            // the granted amounts are in st
    double cost_d = 0.0, val_d = 0.0;
    for (uint32_t jl = tid; jl < nj; jl += T) mem_wish_job(X, st, J0 + jl, assign, cost_d, val_d);
    cost_d = wave_sum_f64(cost_d);
    val_d = wave_sum_f64(val_d);
    if ((tid & 63u) == 0) { sums[tid >> 6] = cost_d; sums[T / 64 + (tid >> 6)] = val_d; }
    __syncthreads();                                            // also: the wishes are stored before anything replaces them
    if (tid < 64u) {
        const bool has = tid < T / 64;
        const double wish = wave_sum_f64(has ? sums[tid] : 0.0), val = wave_sum_f64(has ? sums[T / 64 + tid] : 0.0);
        const uint32_t jrel0 = J0 - X.jb;
        mem_close_round(X, st.gi + jrel0, st.g + jrel0, st.ci + jrel0, rnd, wish, val, assign + jrel0, totals);
    }
}

// ------------------------------------------------------------------ memory
// Wish of a job: the smallest tier that reaches its best throughput over all
// tiers.  The wishes are written as the result; they are kept when all of them
// together stay 1 % below the round's host memory (then every job finds its
// wish still free when its turn comes: the float32 running remainder of the
// in-order rule drifts by far less), otherwise the round is redone in job order.
// Large rounds: k_mem_wish (a thread per job) and k_mem_finish (a wavefront per
// round); small rounds: the workgroup of the CPU pass's selection does both.

// the wish of a job that holds segment gi (-1: nothing) with g GPUs at CPU level c_lvl of level_cpus CPUs; s0, ns: its
// segments; adds its cost and its normalised throughput to the two sums
__device__ __forceinline__ rk_assign mem_wish(const Ctx &X, int32_t gi, uint32_t g, uint32_t c_lvl, uint32_t level_cpus, uint32_t s0,
                                              uint32_t ns, uint32_t first_seg, float ref, double &cost_d, double &val_d) {
    const GridDev &grid = X.grid;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem;
    rk_assign out = {0u, 0u, 0.f, RK_NO_PLAN, 0.f};
    if (gi < 0) return out;
    const uint64_t base = (uint64_t)n_rows * (s0 - first_seg) + (uint64_t)(c_lvl * n_mem) * ns + (uint32_t)gi;
    float bv = 0.f, cost = 0.f;
    uint32_t bm = 0;
    for (uint32_t m = 0; m < n_mem; ++m) {
        const float v = X.best_thr[base + (uint64_t)m * ns];
        if (v > bv) { bv = v; bm = m; cost = grid.mem_levels_gb[m]; }
    }
    if (bv > 0.f) {
        if (grid.mem_mode) cost = cost * (float)g;
        out.g = g;
        out.c = grid.cpu_mode ? level_cpus * g : level_cpus;
        out.mem_gb = cost;
        out.plan = X.best_plan[base + (uint64_t)bm * ns];
        out.thr = bv;
        cost_d += (double)cost;
        val_d += (double)bv / (double)ref;
    }
    return out;
}

// ... of job j, written to its record
__device__ __forceinline__ void mem_wish_job(const Ctx &X, const JobState &st, uint32_t j, rk_assign *__restrict__ assign,
                                             double &cost_d, double &val_d) {
    const uint32_t jrel = j - X.jb;
    rk_assign out = {0u, 0u, 0.f, RK_NO_PLAN, 0.f};
    const int32_t gi = st.gi[jrel];
    if (gi >= 0) {
        const uint32_t ju = job_of(X, j);
        const uint32_t s0 = X.tb.seg_off[ju], ns = X.tb.seg_off[ju + 1] - s0;
        const uint32_t c_lvl = st.ci[jrel];
        out = mem_wish(X, gi, st.g[jrel], c_lvl, X.grid.cpu_levels[c_lvl], s0, ns, X.tb.seg_off[X.jb], X.ref_thr[ju], cost_d, val_d);
    }
    assign[jrel] = out;
}

__global__ __launch_bounds__(JOB_THREADS) void k_mem_wish(Ctx X, JobState st, rk_assign *__restrict__ assign) {
    __shared__ double red[2][JOB_THREADS / 64];
    const uint32_t rnd = blockIdx.y, tid = threadIdx.x;
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    const uint32_t jl = blockIdx.x * JOB_THREADS + tid;
    double cost_d = 0.0, val_d = 0.0;
    if (J0 + jl < J1) mem_wish_job(X, st, J0 + jl, assign, cost_d, val_d);
    cost_d = wave_sum_f64(cost_d);
    val_d = wave_sum_f64(val_d);
    if ((tid & 63u) == 0) { red[0][tid >> 6] = cost_d; red[1][tid >> 6] = val_d; }
    __syncthreads();
    if (tid == 0) {
        double a = 0.0, b = 0.0;
        for (int w = 0; w < JOB_THREADS / 64; ++w) { a += red[0][w]; b += red[1][w]; }
        st.partial[((size_t)rnd * st.blocks_per_round + blockIdx.x) * 2 + 0] = a;
        st.partial[((size_t)rnd * st.blocks_per_round + blockIdx.x) * 2 + 1] = b;
    }
}

// One wavefront (threadIdx.x = lane) closes a round whose wishes sum to `wish` GiB and `val` normalised throughput.
// gi_of, g_of, ci_of: what the round's jobs hold, assign: their records, from its first job on.  True: the records were
// decided in job order and replace the wishes.
__device__ bool mem_close_round(const Ctx &X, const int32_t *gi_of, const uint32_t *g_of, const uint32_t *ci_of, uint32_t rnd,
                                double wish, double val, rk_assign *__restrict__ assign, float *__restrict__ totals) {
    const uint32_t tid = threadIdx.x;
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    const GridDev &grid = X.grid;
    const uint32_t nj = J1 - J0;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem;
    if (wish <= 0.99 * (double)cl.host_mem_gb) {
        if (tid == 0) totals[rnd] = (float)val;
        return false;
    }
    // In job order: lanes load a batch of 64 jobs, then the jobs that hold something are decided one after the other by all
    // lanes alike, and every lane writes its record afterwards.  (512 of 1,000 jobs: 79 us when a lane at a time made its
    // record between the decisions, also for jobs that hold nothing; 21.)
    float freeM = cl.host_mem_gb, level_gb[RK_MAX_MEM_LEVELS];
#pragma unroll
    for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) level_gb[m] = m < n_mem ? grid.mem_levels_gb[m] : 0.f;
    double sum = 0.0;
    for (uint32_t base = 0; base < nj; base += 64) {
        const uint32_t jl = base + tid;
        const bool have = jl < nj && gi_of[jl] >= 0;
        uint32_t g = 0, c_lvl = 0, ns = 0;
        uint64_t at0 = 0;
        unsigned long long choice = 0;      // 4 bits per prefix length: best tier among tiers 0..k
        uint32_t valid = 0;                 // bit k: that best throughput is positive
        float thr_m[RK_MAX_MEM_LEVELS];
#pragma unroll
        for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) thr_m[m] = 0.f;
        if (have) {
            const uint32_t j = J0 + jl;
            g = g_of[jl]; c_lvl = ci_of[jl];
            const uint32_t ju = job_of(X, j);
            const uint32_t s0 = X.tb.seg_off[ju];
            ns = X.tb.seg_off[ju + 1] - s0;
            at0 = (uint64_t)n_rows * (s0 - X.tb.seg_off[X.jb]) + (uint64_t)(c_lvl * n_mem) * ns + (uint32_t)gi_of[jl];
            float bv = 0.f;
            uint32_t bm = 0;
#pragma unroll
            for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) {
                if (m < n_mem) {
                    const float v = X.best_thr[at0 + (uint64_t)m * ns];
                    thr_m[m] = v;
                    if (v > bv) { bv = v; bm = m; }
                    choice |= (unsigned long long)bm << (4 * m);
                    if (bv > 0.f) valid |= 1u << m;
                }
            }
        }
        uint32_t tier = 0xFFFFFFFFu;        // the lane's job's, none: it is left out
        for (unsigned long long todo = __ballot(have); todo;) {
            const uint32_t turn = (uint32_t)__ffsll((long long)todo) - 1u;
            todo &= todo - 1ull;
            const float g_turn = (float)wave_lane_u32(g, turn);
            const unsigned long long choice_turn = wave_lane_u64(choice, turn);
            const uint32_t valid_turn = wave_lane_u32(valid, turn);
            auto cost_of = [&](uint32_t m) { return grid.mem_mode ? level_gb[m] * g_turn : level_gb[m]; };
            int32_t k = -1;                                 // last tier that still fits (tiers ascend)
#pragma unroll
            for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) if (m < n_mem && cost_of(m) <= freeM) k = (int32_t)m;
            if (k < 0 || !((valid_turn >> k) & 1u)) continue;
            const uint32_t bm = (uint32_t)(choice_turn >> (4 * k)) & 15u;
            float spent = 0.f;
#pragma unroll
            for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) if (m == bm) spent = cost_of(m);
            freeM = freeM - spent;
            if (tid == turn) tier = bm;
        }
        rk_assign out = {0u, 0u, 0.f, RK_NO_PLAN, 0.f};
        if (tier != 0xFFFFFFFFu) {
            float v = 0.f, cost = 0.f;
#pragma unroll
            for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) if (m == tier) { v = thr_m[m]; cost = grid.mem_mode ? level_gb[m] * (float)g : level_gb[m]; }
            out.g = g;
            out.c = (uint32_t)cpu_cost(grid, c_lvl, g);
            out.mem_gb = cost;
            out.plan = X.best_plan[at0 + (uint64_t)tier * ns];
            out.thr = v;
            sum += (double)v / (double)X.ref_thr[job_of(X, J0 + jl)];
        }
        if (jl < nj) assign[jl] = out;
    }
    sum = wave_sum_f64(sum);
    if (tid == 0) totals[rnd] = (float)sum;
    return true;
}

// One wavefront per round.
__global__ __launch_bounds__(64) void k_mem_finish(Ctx X, JobState st, rk_assign *__restrict__ assign,
                                                   float *__restrict__ totals) {
    const uint32_t rnd = blockIdx.x, tid = threadIdx.x;
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    const uint32_t used_blocks = (J1 - J0 + JOB_THREADS - 1) / JOB_THREADS;
    double wish = 0.0, val = 0.0;
    for (uint32_t b = tid; b < used_blocks; b += 64) {
        wish += st.partial[((size_t)rnd * st.blocks_per_round + b) * 2 + 0];
        val += st.partial[((size_t)rnd * st.blocks_per_round + b) * 2 + 1];
    }
    wish = wave_sum_f64(wish);
    val = wave_sum_f64(val);
    const uint32_t jrel0 = J0 - X.jb;
    mem_close_round(X, st.gi + jrel0, st.g + jrel0, st.ci + jrel0, rnd, wish, val, assign + jrel0, totals);
}

// ------------------------------------------------------------------ rounds of few jobs
// The whole allocation of a round whose walks take a few turns of one workgroup's wavefronts, in one launch: walks,
// histogram, threshold, application, the steps on what is left and the memory step of both passes.  Such a round is a
// chain of latencies, so everything a step of the chain hands to the next lies in LDS: a pass compacts the jobs that take
// part in it, a job takes 16, 32 or 64 neighbouring lanes (at least its amounts), and its amounts, values and walk stay
// where those lanes can read them.  The steps on what is left are taken by one wavefront without barriers; the others
// come in where cached steps that stopped fitting have to be made exact.
// The lines: a wavefront takes the GPU walks of 64 / lanes jobs in about 2.7 us, bound by its instructions, while a launch
// of its own over the whole chip takes 4 to 5 us for any number of jobs that comes into question.  Whole rounds on jobs
// with up to 16 GPU counts, four launches and one: 8 jobs 48 and 39 us, 64 jobs 56 and 44, 128 jobs 58 and 52, 192 jobs
// 64 and 62, 256 jobs 67 and 72.  Leaving the walks of larger rounds to a launch in front of this one brings nothing:
// their threads wait for memory in every step instead (500 jobs 68 and 74 us, 1,000 jobs 79 and 92).  The same line holds
// for many rounds in a call: 256 rounds of 64 jobs 132 and 103, 1,024 of 128 jobs 587 and 530, 4,096 of 8 jobs 572 and 555.
// Jobs with up to 32 and 64 counts, the allocation alone on walks as long as they can be: 64 jobs of 31 49 and 50, 32 of 53
// 52 and 37.
// CPU walks are too long for one workgroup where every one of many jobs holds GPUs and gains at every level, as curves
// handed in by the caller may say: the allocation alone 59 and 102 us for 128 jobs at 32 levels, 91 and 154 for 64 at 64; at
// FEW_CPU_LANES, 64 jobs at 32 levels and 128 at 16, 60 and 54, 48 and 48.  The curves of a round that evaluates the model
// itself do not: at FEW_CPU_LANES_MODEL, whole rounds of 128 jobs at 32 levels 60 and 48, where nothing but offload fits the
// GPUs 75 and 53, and 82 and 80 where only offload is allowed and every job that holds GPUs takes all CPUs.
// The pass over CPUs ends behind its walks where all their steps fit together: rounds of 8 and 64 jobs 1.6 and 1.3 us less.
constexpr int FEW_THREADS = 1024, FEW_WAVES = FEW_THREADS / 64;
constexpr uint32_t FEW_JOBS = FEW_THREADS;        // at most a job per thread (T: threads of the workgroup, 256, 512 or FEW_THREADS)
constexpr uint32_t FEW_GPU_LANES = 2048;          // of a round: jobs times lanes of a job, in the pass over GPUs
constexpr uint32_t FEW_CPU_LANES = 2048, FEW_CPU_LANES_MODEL = 4096;   // ... and over CPUs, on curves handed in and on the model's
constexpr uint32_t FEW_BINS = 1024, FEW_FINE = 128;
constexpr uint32_t FEW_TICK_LANES = 4096;         // of a tick of a simulation (k_sim_few): jobs that take part times lanes of a job
constexpr uint32_t FEW_TICK_LANES_16 = 5120;      // ... where no walk has more than 16 steps
constexpr uint32_t FEW_TICK_WALK = 64;            // ... steps over CPU levels that a wavefront walks, one job or group of jobs after the other
constexpr size_t FEW_SIM_LDS = 152 * 1024;
constexpr uint64_t FEW_WALK_BYTES = 32ull << 20;  // walks that are found before the first tick, at most
constexpr uint32_t FEW_WALKS_PER_TICK = 8192;     // ... that a tick pays for

struct FewMem {                  // per round, in LDS
    unsigned long long *hc;      // histogram of a pass: CPUs and GPUs of the steps per bin
    uint32_t *hg;
    uint32_t *lvl;               // CPU levels
    uint32_t *range;             // highest and lowest key of the pass's walks; steps that the first wavefront walked; CPUs of all steps
    // per job of the round: where its segments are, its reference throughput, what it holds
    uint32_t *s0, *ns;
    float *ref;
    int32_t *gi;
    uint32_t *g, *ci;
    // per job that takes part in the pass, in job order: the job, its cached next step (slope > 0 exact, < 0 an upper
    // bound, 0 none; target | GPUs << 16; CPUs)
    uint32_t *part, *to;
    float *slope;
    uint32_t *dc;
    uint32_t *cnt;               // FEW_WAVES words: the wavefronts' counts
    unsigned long long *box;     // what the first wavefront tells the others
};
// Per lane of a job that takes part: its value and amount (GPUs, GPU pass), and the walk's step of the lane's number:
// key (0: none), slope, target | GPUs << 16, CPUs.  In LDS, or in memory where a pass's do not fit there.
struct FewLanes {
    uint4 *step;
    float *val;
    uint32_t *amt;
};
constexpr size_t FEW_FIXED_BYTES = (size_t)FEW_BINS * 12 + (RK_MAX_CPU_LEVELS + FEW_WAVES + 4) * 4 + 4 * 8;
constexpr size_t FEW_JOB_BYTES = 10 * 4, FEW_LANE_BYTES = 16 + 2 * 4;

// The per-job words of `jobs` jobs (rounded up to four); *end: the LDS behind them.
__device__ __forceinline__ FewMem few_mem(unsigned long long *lds, uint32_t jobs, uint32_t **end) {
    FewMem M;
    M.hc = lds;
    M.box = M.hc + FEW_BINS;
    uint32_t *p = reinterpret_cast<uint32_t *>(M.box + 4);
    auto take = [&](uint32_t n) { uint32_t *q = p; p += n; return q; };
    M.hg = take(FEW_BINS); M.lvl = take(RK_MAX_CPU_LEVELS); M.cnt = take(FEW_WAVES); M.range = take(4);
    jobs = (jobs + 3u) & ~3u;
    M.s0 = take(jobs); M.ns = take(jobs); M.ref = reinterpret_cast<float *>(take(jobs));
    M.gi = reinterpret_cast<int32_t *>(take(jobs)); M.g = take(jobs); M.ci = take(jobs);
    M.part = take(jobs); M.to = take(jobs); M.slope = reinterpret_cast<float *>(take(jobs)); M.dc = take(jobs);
    *end = p;
    return M;
}
// (n a multiple of four)
__device__ __forceinline__ FewLanes few_lane_mem(uint32_t *p, uint32_t n) {
    return FewLanes{reinterpret_cast<uint4 *>(p), reinterpret_cast<float *>(p + 4 * (size_t)n), p + 5 * (size_t)n};
}

// Lanes a job takes: `amounts` <= 64.
inline uint32_t few_lanes(uint32_t amounts) { return amounts <= 16u ? 16u : amounts <= 32u ? 32u : 64u; }

// Maximum over the 16, 32 or 64 neighbouring lanes of a job; all 64 lanes must be active.
__device__ __forceinline__ uint32_t few_max(uint32_t v, uint32_t lanes, uint32_t lane) {
    v = row_max_u32(v);
    if (lanes == 16u) return v;
    const uint32_t lo = rs_max_u32(wave_lane_u32(v, 0u), wave_lane_u32(v, 16u));
    const uint32_t hi = rs_max_u32(wave_lane_u32(v, 32u), wave_lane_u32(v, 48u));
    return lanes == 64u ? rs_max_u32(lo, hi) : lane < 32u ? lo : hi;
}
__device__ __forceinline__ uint32_t few_bits(unsigned long long ballot, uint32_t base, uint32_t lanes) {   // first lane + 1, 0: none
    return (uint32_t)__ffsll((long long)((ballot >> base) & (~0ull >> (64u - lanes))));
}

// Best next step of the job whose lanes these are, from where it is (`at`), under what is free: best_step's search.
// v, amt: the lane's value (0 beyond the job's amounts) and GPU count.
template <int PASS>
__device__ __forceinline__ Step few_search(const GridDev &grid, const uint32_t *lvl, uint32_t lanes, float v, uint32_t amt, int32_t at,
                                           uint32_t g_held, uint32_t ci, float ref, unsigned long long freeG,
                                           unsigned long long freeC, uint32_t &dc_out) {
    const uint32_t lane = threadIdx.x & 63u, sub = lane & (lanes - 1u), base = lane - sub;
    const int from = (int)(base + (at < 0 ? 0u : (uint32_t)at));
    const float v_at = __shfl(v, from, 64);
    const float cur = at < 0 ? 0.f : v_at;
    uint32_t dg = 0;
    unsigned long long dc;
    if (PASS == 0) {
        const uint32_t g_at = (uint32_t)__shfl((int)amt, from, 64);
        dg = amt - (at < 0 ? 0u : g_at);
        dc = (unsigned long long)lvl[ci] * (grid.cpu_mode ? dg : (at < 0 ? 1u : 0u));
    } else {
        const unsigned long long times = grid.cpu_mode ? g_held : 1u;
        dc = (unsigned long long)lvl[sub] * times - (unsigned long long)lvl[at] * times;
    }
    uint32_t bits = 0;
    if ((int32_t)sub > at && v > cur && (PASS == 1 || dg <= freeG) && dc <= freeC) {
        float sl = (v - cur) / ref;
        sl = sl / (PASS == 0 ? (float)dg : (float)dc);
        bits = sl > 0.f ? __float_as_uint(sl) : 0u;
    }
    const uint32_t top = few_max(bits, lanes, lane);
    Step out = {0.f, 0u, 0u};
    const uint32_t holder = few_bits(__ballot(bits == top), base, lanes) - 1u;       // the lowest lane is the smallest amount
    const uint32_t dg_top = PASS == 0 ? (uint32_t)__shfl((int)dg, (int)(base + holder), 64) : 0u;
    dc_out = (uint32_t)__shfl((int)(uint32_t)dc, (int)(base + holder), 64);          // (what fits the free CPUs fits a word)
    if (top) { out.slope = __uint_as_float(top); out.tgt = holder; out.dg = dg_top; }
    return out;
}

// The jobs of the round with take(job) in job order; returns how many.  Two barriers.
template <int T, class F>
__device__ __forceinline__ uint32_t few_compact(const FewMem &M, uint32_t nj, F take) {
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const bool in = tid < nj && take(tid);
    const unsigned long long b = __ballot(in);
    if (lane == 0) M.cnt[wave] = (uint32_t)__popcll(b);
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (uint32_t w = 0; w < T / 64; ++w) { const uint32_t n = M.cnt[w]; before += w < wave ? n : 0u; all += n; }
    if (in) M.part[before + (uint32_t)__popcll(b & ((1ull << lane) - 1ull))] = tid;
    __syncthreads();
    return all;
}

// Where bin b is kept: lane l of few_cut takes the FEW_BINS / 64 bins from (FEW_BINS / 64) l on, one at a time.
__device__ __forceinline__ uint32_t few_bin_at(uint32_t b) { return (b % (FEW_BINS / 64u)) * 64u + b / (FEW_BINS / 64u); }

template <int T>
__device__ __forceinline__ void few_clear(const FewMem &M) {
    for (uint32_t i = threadIdx.x; i < FEW_BINS; i += T) { M.hg[i] = 0u; M.hc[i] = 0ull; }
    if (threadIdx.x == 0) { M.range[0] = 0u; M.range[1] = 0xFFFFFFFFu; M.range[2] = 0u; M.range[3] = 0u; }
}

// One wavefront: the first bin (bin 0 holds the highest keys) whose steps, with everything before it, no longer fit
// (FEW_BINS: all fit); usedG, usedC: the cost of the bins before it.
__device__ __forceinline__ uint32_t few_cut(const FewMem &M, unsigned long long capG, unsigned long long capC,
                                            unsigned long long &usedG, unsigned long long &usedC) {
    constexpr uint32_t PER = FEW_BINS / 64u;
    static_assert(PER <= 16u, "a row of lanes looks through one lane's bins");
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t sg = 0;
    unsigned long long sc = 0;
#pragma unroll
    for (uint32_t i = 0; i < PER; ++i) { sg += M.hg[i * 64u + lane]; sc += M.hc[i * 64u + lane]; }
    uint32_t ig = sg;
    unsigned long long ic = sc;
    wave_scan(ig, ic);
    const unsigned long long over = __ballot(ig > capG || ic > capC);
    if (!over) { usedG = wave_lane_u32(ig, 63u); usedC = wave_lane_u64(ic, 63u); return FEW_BINS; }
    const uint32_t l0 = (uint32_t)__ffsll((long long)over) - 1u;
    const unsigned long long g0 = wave_lane_u32(ig - sg, l0), c0 = wave_lane_u64(ic - sc, l0);
    const uint32_t vg = lane < PER ? M.hg[lane * 64u + l0] : 0u;
    const unsigned long long vc = lane < PER ? M.hc[lane * 64u + l0] : 0ull;
    ig = vg; ic = vc;
    row_scan(ig, ic);
    const uint32_t i0 = (uint32_t)__ffsll((long long)__ballot(lane < PER && (g0 + ig > capG || c0 + ic > capC))) - 1u;
    usedG = g0 + wave_lane_u32(ig - vg, i0);
    usedC = c0 + wave_lane_u64(ic - vc, i0);
    return l0 * PER + i0;
}

// The walk of the job whose lanes these are (k_hull_groups): from an amount (start, its value cur and cost cost_cur; -1: from
// nothing) always to the one with the highest slope, among the amounts whose lanes `can`.  v, cost: the lane's value and cost.
// Lane k ends with step k: its key (the lowest slope so far), slope, target, the amount before it and both costs; n: steps.
struct FewWalk { uint32_t n, key, raw, at, from, to; int32_t before, last; };
template <bool COUNT>
__device__ __forceinline__ FewWalk few_walk(uint32_t lanes, bool walking, bool can, float v, uint32_t cost, int32_t start, float cur,
                                            uint32_t cost_cur, float ref, uint32_t &walked) {
    const uint32_t lane = threadIdx.x & 63u, sub = lane & (lanes - 1u), base = lane - sub;
    FewWalk W = {0u, 0u, 0u, 0u, 0u, 0u, -1, start};
    float prev = __uint_as_float(0x7F800000u);
    while (__ballot(walking)) {
        if (COUNT) ++walked;
        uint32_t best = 0;
        if (walking && can && (int32_t)sub > W.last && v > cur) {
            float sl = (v - cur) / ref;
            sl = sl / (float)(cost - cost_cur);
            best = __float_as_uint(sl);
        }
        const uint32_t top = few_max(best, lanes, lane);
        walking = walking && top != 0u;
        const uint32_t holder = few_bits(__ballot(best == top), base, lanes);
        const int src = (int)(base + (holder ? holder - 1u : 0u));
        const uint32_t top_cost = (uint32_t)__shfl((int)cost, src, 64);
        const float top_val = __shfl(v, src, 64);
        if (walking) {
            prev = __uint_as_float(top) < prev ? __uint_as_float(top) : prev;
            if (sub == W.n) {
                W.key = __float_as_uint(prev); W.raw = top; W.at = (uint32_t)src - base;
                W.before = W.last; W.from = cost_cur; W.to = top_cost;
            }
            cur = top_val;
            W.last = src - (int)base;
            cost_cur = top_cost;
            ++W.n;
        }
    }
    return W;
}

// What a simulation's jobs do in rounds from nothing does not depend on the other jobs, and there are few answers per job: they
// are all found before the first tick (k_few_states).
struct FewStates {
    const uint4 *walk;           // per job, number of amounts that the capacity allows (`rows` of them) and lane: step (key, slope,
                                 // target | GPUs << 16) of the lane's number on the walk over GPUs; the lane's value
    const uint4 *cpu;            // per job and amount, after the walk over all CPU levels: throughput and plan of the best memory tier,
                                 // tier (FEW_NO_TIER: none) | level << 8, CPUs the walk costs
    const uint8_t *allowed;      // per GPUs (up to most_g) and job: how many of its amounts are not larger
    uint32_t rows, most_g;
};
constexpr uint32_t FEW_STEP_CPUS = 1u << 15;      // (a step that costs as many, or all of them together, counts as one that may not fit: sums stay words)
constexpr uint32_t FEW_NO_TIER = 0xFFu;
constexpr uint32_t FEW_MANY_CPUS = 1u << 20;      // (a walk that costs that many counts as one that does not fit)

// A workgroup per job; 406 jobs of up to 16 amounts: 6,900 walks.
__global__ __launch_bounds__(256) void k_few_states(Ctx X, uint32_t lanes0, uint32_t lanes1, FewStates T, uint4 *walk, uint4 *cpu, uint8_t *allowed) {
    const GridDev &grid = X.grid;
    const uint32_t j = blockIdx.x, tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t s0 = X.tb.seg_off[j], ns = X.tb.seg_off[j + 1] - s0, first_seg = X.tb.seg_off[0];
    const uint32_t n_mem = grid.n_mem, m_top = n_mem - 1u, n_cpu = grid.n_cpu;
    const uint64_t jbase = (uint64_t)n_cpu * n_mem * (s0 - first_seg);
    const float ref = X.ref_thr[j];
    uint32_t walked = 0;
    {
        const uint32_t sub = lane & (lanes0 - 1u), per = 64u / lanes0, mine = lane / lanes0;
        const uint32_t amt = sub < ns ? X.tb.seg_g[s0 + sub] : 0u;
        const float v = sub < ns ? X.curve_thr[jbase + (uint64_t)m_top * ns + sub] : 0.f;
        const uint32_t cost = amt;
        for (uint32_t a0 = wave * per; a0 <= ns; a0 += 4u * per) {
            const uint32_t a = a0 + mine;
            const FewWalk W = few_walk<false>(lanes0, a <= ns, sub < a, v, cost, -1, 0.f, 0u, ref, walked);
            if (a > ns) continue;
            const bool on = sub < W.n;
            walk[((size_t)j * T.rows + a) * lanes0 + sub] = make_uint4(on ? W.key : 0u, W.raw, W.at | (on ? W.to - W.from : 0u) << 16, __float_as_uint(v));
        }
    }
    {
        const uint32_t sub = lane & (lanes1 - 1u), per = 64u / lanes1, mine = lane / lanes1;
        for (uint32_t i0 = wave * per; i0 < ns; i0 += 4u * per) {
            const bool valid = i0 + mine < ns;
            const uint32_t gi = valid ? i0 + mine : ns - 1u, g = X.tb.seg_g[s0 + gi];
            const float v = sub < n_cpu ? X.best_thr[jbase + (uint64_t)(sub * n_mem + m_top) * ns + gi] : 0.f;
            const uint32_t cost = (sub < n_cpu ? grid.cpu_levels[sub] : 0u) * (grid.cpu_mode ? g : 1u);
            const uint32_t cost_at = (uint32_t)__shfl((int)cost, (int)(lane - sub), 64);
            const float v_at = __shfl(v, (int)(lane - sub), 64);
            const FewWalk W = few_walk<false>(lanes1, valid, sub < n_cpu, v, cost, 0, v_at, cost_at, ref, walked);
            const uint32_t level = (uint32_t)W.last;
            const unsigned long long end = cpu_cost(grid, level, g) - cpu_cost(grid, 0u, g);
            if (!valid || sub != 0) continue;
            uint4 out = {0u, RK_NO_PLAN, FEW_NO_TIER | level << 8, end < FEW_MANY_CPUS && cpu_cost(grid, n_cpu - 1u, g) <= 0xFFFFFFFFull ? (uint32_t)end : FEW_MANY_CPUS};
            float best = 0.f;
            for (uint32_t m = 0; m < n_mem; ++m) {
                const uint64_t at = jbase + (uint64_t)(level * n_mem + m) * ns + gi;
                const float x = X.best_thr[at];
                if (x > best) { best = x; out.x = __float_as_uint(x); out.y = X.best_plan[at]; out.z = m | level << 8; }
            }
            cpu[(size_t)j * (T.rows - 1u) + gi] = out;
        }
    }
    for (uint32_t g = tid; g <= T.most_g; g += 256u) {
        uint32_t lo = 0, hi = ns;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (X.tb.seg_g[s0 + mid] <= g) lo = mid + 1u; else hi = mid;
        }
        allowed[(size_t)g * gridDim.x + j] = (uint8_t)lo;
    }
}

// A pass over the P jobs in M.part.  On entry the histogram is clear; on return (behind a barrier) M.gi, M.g and M.ci
// hold what the pass leaves, freeG / freeC what is left.  COUNT: M.range[2] is how many steps the first wavefront walked (the
// others have as many jobs, or a turn less), as if there were FEW_THREADS.  KNOWN: the walks are in S, all from nothing.
template <int T, int PASS, bool COUNT = false, bool KNOWN = false>
__device__ __forceinline__ void few_pass(const Ctx &X, const FewMem &M, const FewLanes &L, uint32_t P, uint32_t lanes,
                                         uint32_t first_seg, unsigned long long &freeG, unsigned long long &freeC,
                                         const FewStates *S = nullptr) {
    constexpr uint32_t WAVES = T / 64;
    const GridDev &grid = X.grid;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t sub = lane & (lanes - 1u), base = lane - sub, per = 64u / lanes, mine = base / lanes;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem, m_top = n_mem - 1u;
    const unsigned long long capG = freeG, capC = freeC;
    const float *__restrict__ vals = PASS == 0 ? X.curve_thr : X.best_thr;
    // a job per thread: the jobs in turn over the wavefronts, so that few jobs are spread over all of them
    const uint32_t own = lane * WAVES + wave;

    // the walks.  Costs by their low words: a step within the capacity fits a word.
    uint32_t high = 0, low = 0xFFFFFFFFu, walked = 0, cpus_all = 0;
    if constexpr (KNOWN) {                                     // (a job's own row of the table: M.dc holds how many amounts are allowed)
        constexpr uint32_t UN = T <= 512 ? 4 : 2;              // turns whose loads are in flight (1,024 threads have the registers for two)
        for (uint32_t p0 = wave * per; p0 < P; p0 += UN * WAVES * per) {
            uint4 w[UN];
            uint32_t amt[UN];
#pragma unroll
            for (uint32_t u = 0; u < UN; ++u) {
                const uint32_t p = p0 + u * WAVES * per + mine, j = M.part[p < P ? p : P - 1u];
                w[u] = S->walk[((size_t)j * S->rows + M.dc[j]) * lanes + sub];
                amt[u] = sub < M.ns[j] ? X.tb.seg_g[M.s0[j] + sub] : 0u;
            }
#pragma unroll
            for (uint32_t u = 0; u < UN; ++u) {
                const uint32_t p = p0 + u * WAVES * per + mine, e = p * lanes + sub;
                if (p >= P) continue;
                const uint32_t dg = w[u].z >> 16;
                if (w[u].x) { high = w[u].x > high ? w[u].x : high; low = w[u].x < low ? w[u].x : low; }
                L.val[e] = __uint_as_float(w[u].w);
                L.amt[e] = amt[u];
                L.step[e] = make_uint4(w[u].x, w[u].y, w[u].z, w[u].x ? M.lvl[0] * (grid.cpu_mode ? dg : sub == 0 ? 1u : 0u) : 0u);
            }
        }
    } else
    for (uint32_t p0 = wave * per; p0 < P; p0 += WAVES * per) {
        const bool valid = p0 + mine < P;
        const uint32_t p = valid ? p0 + mine : P - 1u, j = M.part[p];
        const float ref = M.ref[j];
        const uint32_t ci = M.ci[j], g_held = PASS == 0 ? 0u : M.g[j];
        const uint32_t npts = PASS == 0 ? M.ns[j] : grid.n_cpu;
        const uint32_t s0 = M.s0[j], ns = M.ns[j];
        const uint64_t jbase = (uint64_t)n_rows * (s0 - first_seg);
        uint32_t amt = 0;
        float v = 0.f;
        if (sub < npts) {
            if (PASS == 0) amt = X.tb.seg_g[s0 + sub];
            v = PASS == 0 ? vals[jbase + (uint64_t)(ci * n_mem + m_top) * ns + sub]
                          : vals[jbase + (uint64_t)(sub * n_mem + m_top) * ns + (uint32_t)M.gi[j]];
        }
        const int32_t start = PASS == 0 ? M.gi[j] : (int32_t)ci;
        const int from = (int)(base + (start < 0 ? 0u : (uint32_t)start));
        const float v_at = __shfl(v, from, 64);
        const float cur = start < 0 ? 0.f : v_at;
        // the amount's cost in the pass's resource and in CPUs, and those of what the job holds (paid for already)
        const uint32_t level = M.lvl[PASS == 0 ? ci : sub];
        const uint32_t times = PASS == 0 ? (grid.cpu_mode ? amt : 1u) : (grid.cpu_mode ? g_held : 1u);
        const unsigned long long cpus = (unsigned long long)level * times;
        const uint32_t cost = PASS == 0 ? amt : (uint32_t)cpus;
        const uint32_t cost_at = (uint32_t)__shfl((int)cost, from, 64);
        const unsigned long long cpus_at = ((unsigned long long)(uint32_t)__shfl((int)(uint32_t)(cpus >> 32), from, 64) << 32) |
                                           (uint32_t)__shfl((int)(uint32_t)cpus, from, 64);
        const uint32_t cost_cur = start < 0 ? 0u : cost_at;
        const bool can = sub < npts && (PASS == 1 || amt <= capG + cost_cur) && cpus <= capC + (start < 0 ? 0ull : cpus_at);
        const FewWalk W = few_walk<COUNT>(lanes, valid, can, v, cost, start, cur, cost_cur, ref, walked);
        if (valid) {
            uint32_t dg = 0, dc = 0;
            if (sub < W.n) {
                if (PASS == 0) {
                    dg = W.to - W.from;
                    dc = M.lvl[ci] * (grid.cpu_mode ? dg : W.before < 0 ? 1u : 0u);
                } else {
                    dc = W.to - W.from;
                    cpus_all += dc < FEW_STEP_CPUS ? dc : FEW_STEP_CPUS;
                }
                high = W.key > high ? W.key : high;
                low = W.key < low ? W.key : low;
            }
            const uint32_t e = p * lanes + sub;
            L.val[e] = v;
            if (PASS == 0) L.amt[e] = amt;
            L.step[e] = make_uint4(sub < W.n ? W.key : 0u, W.raw, W.at | dg << 16, dc);
        }
    }
    high = wave_max_u32_rows(high);
    low = wave_min_u32_rows(low);
    if (high) {
        if (PASS == 1) cpus_all = wave_sum_u32(cpus_all);
        if (lane == 0) {
            atomicMax(&M.range[0], high); atomicMin(&M.range[1], low);
            if (PASS == 1) atomicAdd(&M.range[3], cpus_all);
        }
    }
    if (COUNT && tid == 0) M.range[2] = walked * T / FEW_THREADS;
    __syncthreads();
    if (PASS == 1) {
        // Where all walks fit together, every job goes to the end of its own and finds no step beyond it: mostly the curves
        // are flat over the CPU levels, and few jobs gain by any.
        const uint32_t all = M.range[3];
        if (all < FEW_STEP_CPUS && all <= freeC) {
            freeC -= all;
            if (all)
                for (uint32_t p0 = wave * per; p0 < P; p0 += WAVES * per) {
                    const bool valid = p0 + mine < P;
                    const uint32_t p = valid ? p0 + mine : P - 1u;
                    const uint4 s = L.step[p * lanes + sub];
                    const uint32_t n = (uint32_t)__popcll((__ballot(s.x != 0u) >> base) & (~0ull >> (64u - lanes)));
                    if (valid && n && sub == n - 1u) M.ci[M.part[p]] = s.z & 0xFFFFu;
                }
            __syncthreads();
            return;
        }
    }
    // The threshold: steps whose key lies less than `limit` below the highest one.  Any threshold whose whole set of steps
    // fits selects a prefix of the order: FEW_BINS bins over the keys that occur, and what is left of the bin where the
    // capacity ends is taken step by step.  With more than FEW_FINE jobs that bin is divided once more, which takes 1.2 us
    // and saves turns of 1 to 3 us (1,000 jobs: 10 turns without, 2 with).  (4,096 bins, scanned by all wavefronts: 3.7 us
    // for two levels, this 1.0 for one.)
    const uint32_t top_key = M.range[0];
    uint32_t shift = 0, from = 0;                              // bins are 2^shift wide and begin `from` below the highest key
    if (top_key) { const uint32_t span = top_key - M.range[1]; shift = span < FEW_BINS ? 0u : 22u - (uint32_t)__clz((int)span); }
    auto count = [&](const uint4 &s) {
        const uint32_t at = top_key - s.x - from;
        if (at >> shift >= FEW_BINS) return;
        const uint32_t bin = few_bin_at(at >> shift);
        if (PASS == 0 && s.z >> 16) atomicAdd(&M.hg[bin], s.z >> 16);
        if (s.w) atomicAdd(&M.hc[bin], (unsigned long long)s.w);
    };
    unsigned long long limit;
    for (uint32_t level = 0;; ++level) {
        for (uint32_t e = tid; e < P * lanes; e += T) {
            const uint4 s = L.step[e];
            if (s.x) count(s);
        }
        __syncthreads();
        if (wave == 0) {
            unsigned long long usedG, usedC;
            const uint32_t cut = few_cut(M, freeG, freeC, usedG, usedC);
            if (lane == 0) { M.box[0] = freeG - usedG; M.box[1] = freeC - usedC; M.box[2] = cut; }
        }
        __syncthreads();
        freeG = M.box[0];
        freeC = M.box[1];
        const uint32_t cut = (uint32_t)M.box[2];
        limit = ((unsigned long long)cut << shift) + from;
        if (level == 1u || cut == FEW_BINS || shift == 0u || P <= FEW_FINE) break;
        from = (uint32_t)limit;                                // the bin that did not fit, divided
        shift = shift > 10u ? shift - 10u : 0u;
        for (uint32_t i = tid; i < FEW_BINS; i += T) { M.hg[i] = 0u; M.hc[i] = 0ull; }
        __syncthreads();
    }
    // the prefix goes to every job at once; its next step: the walk's if it still fits, else a search (apply_job)
    const bool some = PASS == 0 ? freeG != 0 : freeC != 0;     // (every step costs something of the pass's resource)
    for (uint32_t p0 = wave * per; p0 < P; p0 += WAVES * per) {
        const bool valid = p0 + mine < P;
        const uint32_t p = valid ? p0 + mine : P - 1u, j = M.part[p], e0 = p * lanes;
        const uint4 s = L.step[e0 + sub];
        const uint32_t n = (uint32_t)__popcll((__ballot(s.x && top_key - s.x < limit) >> base) & (~0ull >> (64u - lanes)));
        int32_t at = PASS == 0 ? M.gi[j] : (int32_t)M.ci[j];
        const uint32_t g_held = PASS == 0 ? 0u : M.g[j], ci = M.ci[j];
        if (n) at = (int32_t)(L.step[e0 + n - 1u].z & 0xFFFFu);
        const uint4 next = n < lanes ? L.step[e0 + n] : make_uint4(0u, 0u, 0u, 0u);
        Step nx = {0.f, 0u, 0u};
        uint32_t dc = next.w;
        bool search = false;
        if (next.x && some) {
            nx = Step{__uint_as_float(next.y), next.z & 0xFFFFu, next.z >> 16};
            search = nx.dg > freeG || dc > freeC;
        }
        if (__ballot(search)) {
            uint32_t dc2;
            const Step found = few_search<PASS>(grid, M.lvl, lanes, L.val[e0 + sub], PASS == 0 ? L.amt[e0 + sub] : 0u, at, g_held, ci,
                                                M.ref[j], freeG, freeC, dc2);
            if (search) { nx = found; dc = dc2; }
        }
        if (valid && sub == 0) {
            if (n) {
                if (PASS == 0) { M.gi[j] = at; M.g[j] = L.amt[e0 + (uint32_t)at]; }
                else M.ci[j] = (uint32_t)at;
            }
            M.slope[p] = nx.slope;
            M.to[p] = nx.tgt | nx.dg << 16;
            M.dc[p] = dc;
        }
    }
    __syncthreads();
    if (!some) return;
    // Step by step on what is left, by the first wavefront: the highest slope, the lower job among equals.  A step that
    // no longer fits stays as an upper bound of what its job can still do; where a bound comes out highest, all
    // wavefronts make the bounds that could win exact (tail_run's rule).
    for (;;) {
        if (wave == 0) {
            uint32_t command = 0, exact = 0, exact_p = 0;
            while (PASS == 0 ? freeG != 0 : freeC != 0) {
                uint32_t best = 0, best_p = 0, sure = 0, sure_p = 0;
                for (uint32_t p0 = lane; p0 < P; p0 += 256u) {   // four of the lane's jobs per round of reads
                    float sl[4];
                    uint32_t to[4], dc[4];
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u) {
                        const uint32_t p = p0 + 64u * u < P ? p0 + 64u * u : p0;
                        sl[u] = M.slope[p]; to[u] = M.to[p]; dc[u] = M.dc[p];
                    }
#pragma unroll
                    for (uint32_t u = 0; u < 4; ++u) {
                        const uint32_t p = p0 + 64u * u;
                        if (p >= P) continue;
                        if (sl[u] > 0.f && ((to[u] >> 16) > freeG || dc[u] > freeC)) { sl[u] = -sl[u]; M.slope[p] = sl[u]; }
                        const uint32_t b = __float_as_uint(sl[u]) & 0x7FFFFFFFu;
                        if (b > best) { best = b; best_p = p; }
                        if (sl[u] > 0.f && b > sure) { sure = b; sure_p = p; }
                    }
                }
                const uint32_t top = wave_max_u32_rows(best);
                if (!top) break;
                const uint32_t p = wave_min_u32_rows(best == top ? best_p : 0xFFFFFFFFu);
                if (!(M.slope[p] > 0.f)) {                     // a bound
                    exact = wave_max_u32_rows(sure);
                    exact_p = wave_min_u32_rows(exact && sure == exact ? sure_p : 0xFFFFFFFFu);
                    command = 1;
                    break;
                }
                const uint32_t to = M.to[p], j = M.part[p], e = p * lanes + sub;
                freeG -= to >> 16;
                freeC -= M.dc[p];
                const int32_t at = (int32_t)(to & 0xFFFFu);
                const uint32_t ci = PASS == 0 ? M.ci[j] : 0u, g_held = PASS == 0 ? 0u : M.g[j];
                const uint32_t amt = PASS == 0 ? L.amt[e] : 0u;
                uint32_t dc;
                const Step nx = few_search<PASS>(grid, M.lvl, lanes, L.val[e], amt, at, g_held, ci, M.ref[j], freeG, freeC, dc);
                const uint32_t g_at = (uint32_t)__shfl((int)amt, (int)(base + (uint32_t)at), 64);
                if (lane == 0) {
                    if (PASS == 0) { M.gi[j] = at; M.g[j] = g_at; }
                    else M.ci[j] = (uint32_t)at;
                    M.slope[p] = nx.slope;
                    M.to[p] = nx.tgt | nx.dg << 16;
                    M.dc[p] = dc;
                }
                rs_wave_order();                               // the lanes read each other's words in the next turn
            }
            if (lane == 0) {
                M.box[0] = freeG;
                M.box[1] = freeC;
                M.box[2] = ((unsigned long long)command << 32) | exact;
                M.box[3] = exact_p;
            }
        }
        __syncthreads();
        freeG = M.box[0];
        freeC = M.box[1];
        const unsigned long long told = M.box[2];
        const uint32_t exact = (uint32_t)told, exact_p = (uint32_t)M.box[3];
        if (!(told >> 32)) break;
        const float sl_own = own < P ? M.slope[own] : 0.f;
        const uint32_t b_own = __float_as_uint(-sl_own);
        unsigned long long todo = __ballot(sl_own < 0.f && (b_own > exact || (b_own == exact && own < exact_p)));
        while (todo) {                                         // 64 / lanes of the wavefront's jobs at a time
            uint32_t l = 64u;
            for (uint32_t g = 0; g < per && todo; ++g) {
                const uint32_t first = (uint32_t)__ffsll((long long)todo) - 1u;
                todo &= todo - 1ull;
                if (g == mine) l = first;
            }
            const bool need = l < 64u;
            const uint32_t p = (need ? l : 0u) * WAVES + wave, j = M.part[need ? p : 0u];
            uint32_t dc;
            const int32_t at = PASS == 0 ? M.gi[j] : (int32_t)M.ci[j];
            const uint32_t ci = M.ci[j], g_held = PASS == 0 ? 0u : M.g[j];
            const float v = need ? L.val[p * lanes + sub] : 0.f;
            const uint32_t amt = PASS == 0 && need ? L.amt[p * lanes + sub] : 0u;
            const Step nx = few_search<PASS>(grid, M.lvl, lanes, v, amt, at, g_held, ci, M.ref[j], freeG, freeC, dc);
            if (need && sub == 0) {
                M.slope[p] = nx.slope;
                M.to[p] = nx.tgt | nx.dg << 16;
                M.dc[p] = dc;
            }
        }
        __syncthreads();
    }
}

// Where the round's jobs' segments are; for a job per thread (tid < nj).
__device__ __forceinline__ void few_jobs(const Ctx &X, const FewMem &M, uint32_t J0, uint32_t nj) {
    const uint32_t tid = threadIdx.x;
    if (tid < RK_MAX_CPU_LEVELS) M.lvl[tid] = X.grid.cpu_levels[tid];
    if (tid < nj) {
        const uint32_t ju = job_of(X, J0 + tid);
        const uint32_t s0 = X.tb.seg_off[ju];
        M.s0[tid] = s0;
        M.ns[tid] = X.tb.seg_off[ju + 1] - s0;
        M.ref[tid] = X.ref_thr[ju];
    }
}

// The memory step that ends a round, from every thread's wish (mem_wish, its cost and normalised throughput): the first
// wavefront closes the round.  M.box[0], behind the next barrier: the records in `assign` replace the wishes.
// sums: 2 * FEW_WAVES doubles in LDS.
template <int T>
__device__ __forceinline__ void few_memory(const Ctx &X, const FewMem &M, uint32_t rnd, double cost_d, double val_d, double *sums,
                                           rk_assign *assign, float *totals) {
    const uint32_t tid = threadIdx.x;
    if (__ballot(val_d != 0.0 || cost_d != 0.0)) { cost_d = wave_sum_f64(cost_d); val_d = wave_sum_f64(val_d); }
    if ((tid & 63u) == 0) { sums[tid >> 6] = cost_d; sums[FEW_WAVES + (tid >> 6)] = val_d; }
    __syncthreads();
    if (tid < 64u) {
        const bool has = tid < T / 64;
        const double wish = wave_sum_f64(has ? sums[tid] : 0.0), val = wave_sum_f64(has ? sums[FEW_WAVES + tid] : 0.0);
        const bool anew = mem_close_round(X, M.gi, M.g, M.ci, rnd, wish, val, assign, totals);
        if (tid == 0) M.box[0] = anew ? 1ull : 0ull;
    }
}
__device__ __forceinline__ rk_assign few_wish(const Ctx &X, const FewMem &M, uint32_t j, uint32_t first_seg, double &cost_d, double &val_d) {
    return mem_wish(X, M.gi[j], M.g[j], M.ci[j], M.lvl[M.ci[j]], M.s0[j], M.ns[j], first_seg, M.ref[j], cost_d, val_d);
}

// One workgroup per round; near: per-lane words in LDS.
template <int T>
__global__ __launch_bounds__(T) void k_round_few(Ctx X, JobState st, uint32_t max_jobs, uint32_t lanes0, uint32_t lanes1,
                                                           uint32_t near, rk_assign *__restrict__ assign,
                                                           float *__restrict__ totals, TableGuard guard) {
    extern __shared__ __align__(16) unsigned long long lds_few[];
    __shared__ double sums[2 * FEW_WAVES];
    if (!table_usable(guard)) return;
    const uint32_t rnd = blockIdx.x, tid = threadIdx.x;
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    const uint32_t nj = J1 - J0, jrel0 = J0 - X.jb, first_seg = X.tb.seg_off[X.jb];
    uint32_t *lds_lanes;
    const FewMem M = few_mem(lds_few, max_jobs, &lds_lanes);
    const FewLanes L = few_lane_mem(lds_lanes, near);
    few_jobs(X, M, J0, nj);
    Floor fl = {-1, 0u, RK_JOB_OUT};
    if (tid < nj) {
        fl = floor_of(st, jrel0 + tid);
        M.gi[tid] = fl.gi;
        M.g[tid] = fl.gi < 0 ? 0u : X.tb.seg_g[M.s0[tid] + (uint32_t)fl.gi];
        M.ci[tid] = fl.ci;
    }
    unsigned long long freeG, freeC;
    pass_caps<0>(X.R, cl, st, rnd, freeG, freeC);
    few_clear<T>(M);
    uint32_t P = few_compact<T>(M, nj, [&](uint32_t) { return fl.state == RK_JOB_NORMAL && freeG != 0; });
    if (P) few_pass<T, 0>(X, M, L, P, lanes0, first_seg, freeG, freeC);
    few_clear<T>(M);
    P = few_compact<T>(M, nj, [&](uint32_t j) { return fl.state == RK_JOB_NORMAL && M.gi[j] >= 0 && freeC != 0; });
    if (P) few_pass<T, 1>(X, M, L, P, lanes1, first_seg, freeG, freeC);
    double cost_d = 0.0, val_d = 0.0;
    if (tid < nj) assign[jrel0 + tid] = few_wish(X, M, tid, first_seg, cost_d, val_d);
    few_memory<T>(X, M, rnd, cost_d, val_d, sums, assign + jrel0, totals);
}

// Ticks of a simulation of at most FEW_JOBS jobs under the greedy, in one workgroup: what a job does between
// the ticks stays in its thread's registers, a round is k_round_few's.  A tick that starts from what the last round started
// from has that round's result.  As launches of their own (the round's four kernels and k_sim_step, replayed as a graph)
// a tick with a round took 40 us, most of it launches and what one kernel leaves for the next in memory: 406 jobs on 64
// GPUs, 720 ticks 19.2 ms then, 9.1 in one kernel; 30 jobs 8.2 us per tick and 2.7.
// With the walks known beforehand (KNOWN: 11,000 of a round's 44,000 cycles, and 8,000 for the pass over CPUs, which then seldom
// has to be made), 512 threads where they are enough (their registers hold a job's state) and sums by lane swaps: 5.9 ms.
// The walks of a round for many jobs keep one workgroup busy for longer than that: such a tick, and every one after it, is
// left to the launches until the rounds are for fewer jobs again.  So are the ticks after one that walked long over the CPU
// levels, for a while (as many lanes cost 4 us where curves are flat there, as the model's mostly are, and 100 where every
// level gains).  FEW_TICK_LANES and FEW_TICK_WALK are where that pays: us per tick as launches, and in this kernel alone
// whatever the round is for, on curves that gain at every amount and every CPU level, with one GPU for eight jobs, one and
// eight GPUs per job, at 5 and at 64 CPU levels:
//     4,096 lanes   256 jobs of 16   31 and 20, 56 and 40, 56 and 25    36 and 21, 97 and 79, 122 and 87
//                   128 jobs of 32   17 and 9, 41 and 25, 72 and 34     20 and 11, 48 and 34, 131 and 62
//                   64 jobs of 64    18 and 7, 43 and 30, 71 and 32     20 and 7, 55 and 34, 127 and 53
//     5,120 lanes   320 jobs of 16   27 and 20, 57 and 44, 54 and 26    37 and 26, 110 and 90, 122 and 94
//     8,192 lanes   512 jobs of 16   44 and 60, 62 and 68, 57 and 30    51 and 60, 124 and 153, 129 and 150
//                   256 jobs of 32   28 and 32, 57 and 81, 82 and 49    37 and 37, 93 and 118, 141 and 102
//                   128 jobs of 64   17 and 15, 43 and 41, 81 and 47    21 and 16, 51 and 49, 132 and 77
//     16,000 lanes  1,000 jobs of 16 58 and 132, 67 and 115, 63 and 48  62 and 145, 135 and 311, 145 and 286
// (where nobody is ever frozen 160 jobs of 32 take 37 us here and 29 as launches, 128 of them 30 and 28).  With both lines
// every one of these takes what the faster way takes, give or take 2 %, or up to 10 % of 100 ticks where they begin with
// long walks.  (All of these were measured without KNOWN; the lines still lie where the lanes' words fit the LDS.)
// first: the simulation begins with this launch; otherwise the state is where the launch before left it.
// OFTEN: rounds for more than `most` jobs and long walks may occur; FAR: a CPU pass may have more lanes than LDS (`near`), its
// words are in memory then (n_far of them).
// KNOWN: the walks over GPUs, and what a job would take of the CPUs if there were enough, are in F: where all of it fits, the pass
// over CPUs is what every job does on its own.
template <int T, bool OFTEN, bool FAR, bool KNOWN>
__global__ __launch_bounds__(T) void k_sim_few(Ctx X, SimArgs A, FewStates F, uint32_t first, uint32_t go_on, uint32_t most, uint32_t lanes0,
                                                         uint32_t lanes1, uint32_t near, uint32_t *far, uint32_t n_far,
                                                         rk_assign *__restrict__ assign) {
    extern __shared__ __align__(16) unsigned long long lds_few[];
    __shared__ double sums[2 * FEW_WAVES];
    __shared__ unsigned long long frozen[2];                   // of a tick, in two copies used in turn: CPUs | GPUs << 32
    __shared__ uint32_t frozen_n[2], used_g, wanted_c[2];
    __shared__ float round_total;
    __shared__ uint32_t out_used[SIM_FEW_TICKS], out_frozen[SIM_FEW_TICKS];
    __shared__ float out_total[SIM_FEW_TICKS];                 // the ticks' figures, written to memory when the launch ends
    const uint32_t tid = threadIdx.x, J = A.n_jobs, first_seg = X.tb.seg_off[0];
    uint32_t tick = first ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane((int)A.tick[0]);
    if (tick >= A.n_ticks) return;                             // (the simulation is over)
    if (OFTEN && go_on && A.tick[1]) return;                   // (the launch before was stopped)
    const uint32_t begin = tick;
    uint32_t end = A.n_ticks - tick > SIM_FEW_TICKS ? tick + SIM_FEW_TICKS : A.n_ticks;
    uint32_t *lds_lanes;
    const FewMem M = few_mem(lds_few, J, &lds_lanes);
    const FewLanes L = few_lane_mem(lds_lanes, near);
    few_jobs(X, M, 0u, J);
    SimJob s = {0u, 0u, RK_NO_PLAN, 0u, 0.0, 0.0, 0.0, -1.0, false};
    int32_t seg = -1;
    uint32_t lvl = 0;
    double arrival = 0.0, work = 0.0, delta = 0.0;
    const bool mine = tid < J;
    if (mine) {
        arrival = A.arrival[tid]; work = A.work[tid]; delta = A.delta[tid];
        if (!first) {
            s = SimJob{A.S.g[tid], A.S.c[tid], A.S.plan[tid], A.n_reconf[tid], A.S.owed[tid], A.held[tid], A.progress[tid],
                       A.finish[tid], A.S.done[tid] != 0};
            seg = A.S.seg[tid]; lvl = A.S.lvl[tid];
        }
    }
    if (tid < 2u) { frozen[tid] = 0ull; frozen_n[tid] = 0u; wanted_c[tid] = 0u; }
    Floor fl = {-1, 0u, RK_JOB_OUT};
    // the job's record; the amounts it is the wish for (-1: none, or another one by decisions in job order); (KNOWN) for which
    // amount the walk over the CPUs is known: CPUs it costs | level it ends on << 24; the number of amounts allowed, for which limit
    rk_assign a = {0u, 0u, 0.f, RK_NO_PLAN, 0.f};
    int32_t wish_gi = -1, end_gi = -1;
    uint32_t wish_ci = 0, end_of = 0, limit = 0xFFFFFFFFu, allowed = 0, turn = 0;
    const uint32_t lane = tid & 63u;
    __syncthreads();
    if (OFTEN && tid == 0) A.tick[1] = 0u;                     // (all have read it)
    for (bool known = false; tick < end; ++tick, known = true) {
        const double t = (double)tick * A.dt;
        const uint32_t half = tick & 1u;
        // opens the tick: who takes part, who is frozen and what they hold
        Floor now = {-1, 0u, RK_JOB_OUT};
        if (mine && arrival <= t && !s.done) {
            now.state = RK_JOB_NORMAL;
            if (sim_frozen(s.g, s.held, s.n_reconf, delta, A.gate)) now = Floor{seg, lvl, RK_JOB_FROZEN};
        }
        const bool is_frozen = now.state == RK_JOB_FROZEN;
        if (is_frozen)                                         // (what jobs hold is within the cluster, whose CPUs and GPUs are words)
            atomicAdd(&frozen[half], ((unsigned long long)s.g << 32) | (unsigned long long)M.lvl[lvl] * (X.grid.cpu_mode ? s.g : 1u));
        const unsigned long long frozen_m = __ballot(is_frozen);
        if (lane == 0 && frozen_m) atomicAdd(&frozen_n[half], (uint32_t)__popcll(frozen_m));
        const bool other = now.state != fl.state || now.gi != fl.gi || now.ci != fl.ci;
        fl = now;
        if (__syncthreads_or(other || !known)) {
            const unsigned long long held = frozen[half], hg = held >> 32, hc = held & 0xFFFFFFFFull;
            unsigned long long freeG = hg < A.cl.G ? A.cl.G - hg : 0ull, freeC = hc < A.cl.C ? A.cl.C - hc : 0ull;
            if (mine) {
                M.gi[tid] = fl.gi;
                M.g[tid] = is_frozen ? s.g : 0u;
                M.ci[tid] = fl.ci;
                if constexpr (KNOWN) {                         // the amounts that fit: GPUs, and CPUs at the lowest level
                    const uint32_t free_g = (uint32_t)freeG, free_c = (uint32_t)freeC, level = M.lvl[0];
                    const uint32_t by_cpu = X.grid.cpu_mode ? free_c / level : level <= free_c ? 0xFFFFFFFFu : 0u;
                    const uint32_t fits = by_cpu < free_g ? by_cpu : free_g;
                    if (fits != limit) { limit = fits; allowed = F.allowed[(size_t)fits * J + tid]; }
                    M.dc[tid] = allowed;
                }
            }
            if (tid == 0) used_g = 0u;
            few_clear<T>(M);
            uint32_t P = few_compact<T>(M, J, [&](uint32_t) { return fl.state == RK_JOB_NORMAL && freeG != 0; });
            if (OFTEN && (uint32_t)__builtin_amdgcn_readfirstlane((int)P) > most) {                           // (nothing of this tick is in the state yet)
                if (tid == 0) A.tick[1] = 1u;
                break;
            }
            if (P) few_pass<T, 0, false, KNOWN>(X, M, L, P, lanes0, first_seg, freeG, freeC, &F);
            bool all_fit = false;                              // every job has all the CPUs it would take
            const bool takes = fl.state == RK_JOB_NORMAL && mine && M.gi[tid] >= 0;
            if constexpr (KNOWN) {
                const int32_t gi = takes ? M.gi[tid] : -1;
                if (takes && gi != end_gi) {                   // ... and what the job would like there
                    const uint4 rec = F.cpu[(size_t)tid * (F.rows - 1u) + (uint32_t)gi];
                    const uint32_t tier = rec.z & 0xFFu, level = rec.z >> 8, g = M.g[tid];
                    end_gi = gi; end_of = rec.w | level << 24;
                    a = rk_assign{0u, 0u, 0.f, RK_NO_PLAN, 0.f};
                    if (tier != FEW_NO_TIER) {
                        float cost = X.grid.mem_levels_gb[tier];
                        if (X.grid.mem_mode) cost = cost * (float)g;
                        a = rk_assign{g, X.grid.cpu_mode ? M.lvl[level] * g : M.lvl[level], cost, rec.y, __uint_as_float(rec.x)};
                    }
                    wish_gi = gi; wish_ci = level;
                }
                uint32_t c = takes ? end_of & 0xFFFFFFu : 0u;
                if (__ballot(c != 0u)) {
                    c = wave_sum_u32(c);
                    if (lane == 0) atomicAdd(&wanted_c[turn], c);
                }
                if (tid == 0) { wanted_c[turn ^ 1u] = 0u; M.range[2] = 0u; }
                __syncthreads();
                const uint32_t wanted = wanted_c[turn];
                turn ^= 1u;
                all_fit = wanted < FEW_MANY_CPUS && wanted <= freeC;
                if (all_fit && takes) M.ci[tid] = end_of >> 24;
            }
            if (!all_fit) {
                few_clear<T>(M);
                P = few_compact<T>(M, J, [&](uint32_t j) { return fl.state == RK_JOB_NORMAL && M.gi[j] >= 0 && freeC != 0; });
                if (FAR && P * lanes1 > near) few_pass<T, 1, OFTEN>(X, M, few_lane_mem(far, n_far), P, lanes1, first_seg, freeG, freeC);
                else if (P) few_pass<T, 1, OFTEN>(X, M, L, P, lanes1, first_seg, freeG, freeC);
            }
            // memory: what the job would like, found again only where it holds something else than the last time
            double cost_d = 0.0, val_d = 0.0;
            if (mine) {
                const int32_t gi = M.gi[tid];
                const uint32_t ci = M.ci[tid];
                if (gi < 0) {
                    a = rk_assign{0u, 0u, 0.f, RK_NO_PLAN, 0.f};
                } else if (gi != wish_gi || ci != wish_ci) {
                    double unused_c = 0.0, unused_v = 0.0;
                    a = few_wish(X, M, tid, first_seg, unused_c, unused_v);
                }
                wish_gi = gi; wish_ci = ci;
                if (a.g) { cost_d = (double)a.mem_gb; val_d = (double)a.thr / (double)M.ref[tid]; }
            }
            few_memory<T>(X, M, 0u, cost_d, val_d, sums, assign, &round_total);
            __syncthreads();                                   // the round is closed
            if (OFTEN && (uint32_t)__builtin_amdgcn_readfirstlane((int)M.range[2]) > FEW_TICK_WALK) {         // (the next one is as long, as a rule)
                if (tid == 0) A.tick[1] = 1u;
                end = tick + 1u;
            }
            if (M.box[0] && mine) { a = assign[tid]; wish_gi = -1; end_gi = -1; }             // ... by decisions in job order
            uint32_t used = fl.state != RK_JOB_OUT ? a.g : 0u;
            if (__ballot(used != 0u)) {
                used = wave_sum_u32(used);
                if (lane == 0) atomicAdd(&used_g, used);
            }
        }
        // closes it
        if (fl.state != RK_JOB_OUT && sim_close(s, a, t, A.dt, delta, work)) {
            seg = s.g ? M.gi[tid] : -1;
            lvl = s.g ? M.ci[tid] : 0u;
        }
        if (tid == 0) frozen[half ^ 1u] = 0ull;
        __syncthreads();
        if (tid == 0) {
            out_used[tick - begin] = used_g;
            out_total[tick - begin] = round_total;
            out_frozen[tick - begin] = frozen_n[half];
            frozen_n[half] = 0u;
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < tick - begin; i += T) {
        if (A.out.gpus_in_use) A.out.gpus_in_use[begin + i] = out_used[i];
        if (A.out.totals) A.out.totals[begin + i] = out_total[i];
        if (A.out.frozen) A.out.frozen[begin + i] = out_frozen[i];
    }
    if (mine) {
        A.S.g[tid] = s.g; A.S.c[tid] = s.c; A.S.plan[tid] = s.plan; A.S.seg[tid] = seg; A.S.lvl[tid] = lvl;
        A.S.owed[tid] = s.owed; A.S.done[tid] = s.done ? 1 : 0;
        A.held[tid] = s.held; A.progress[tid] = s.progress; A.finish[tid] = s.finish; A.n_reconf[tid] = s.n_reconf;
    }
    if (tid == 0) {
        A.tick[0] = tick;
        if (OFTEN) {
            __hip_atomic_store(A.h_tick + 1, M.range[2] > FEW_TICK_WALK ? SIM_LONG_WALK : 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(A.h_tick, tick, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// ------------------------------------------------------------------ service-level floors
// One workgroup per round.  All threads first stage every job's demand in LDS
// (one word: GPUs, tenant, flags; one word: CPUs), so that the global-memory
// latency is paid once.  The first wavefront then takes the decisions in job
// order, 64 jobs at a time: demands that do not fit what is left right now can
// never fit later and drop out in parallel, before the first and after every
// one that is granted, so that only granted ones take a turn.  The tenants'
// quotas lie in LDS, and every lane has a copy of its job's tenant's for the
// 64 jobs.  All threads then write the floors.  1,000 jobs: 35.5 us while every
// demand that could still fit took a turn, with the quotas in registers, 23.7 now.
constexpr int FLOOR_THREADS = 1024;
constexpr uint32_t FL_CAND = 1u << 24, FL_GUAR = 1u << 25, FL_GRANTED = 1u << 31;

__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}

__global__ __launch_bounds__(FLOOR_THREADS) void k_floors(Ctx X, JobState st, SlaDev S, uint32_t max_jobs) {
    extern __shared__ uint32_t lds_floor[];
    uint32_t *word = lds_floor;                 // GPUs (16 bits) | tenant (8 bits) | flags
    uint32_t *cpus = lds_floor + max_jobs;
    __shared__ uint32_t quota[2][RK_MAX_TENANTS];            // what is left of the tenants' GPUs and CPUs
    const uint32_t rnd = blockIdx.x, tid = threadIdx.x, lane = tid & 63u;
    uint32_t J0, J1;
    rk_cluster cl;
    round_of(X.R, rnd, J0, J1, cl);
    const GridDev &grid = X.grid;
    const uint32_t nj = J1 - J0;

    static_assert(RK_MAX_TENANTS <= FLOOR_THREADS && RK_MAX_TENANTS == 256, "a tenant per thread; the word has eight bits for it");
    if (tid < RK_MAX_TENANTS) {
        const bool in = tid < S.n_tenants;
        quota[0][tid] = in ? S.quota_g[tid] : 0u;
        quota[1][tid] = in ? S.quota_c[tid] : 0u;
    }
    for (uint32_t jl = tid; jl < nj; jl += FLOOR_THREADS) {
        const uint32_t j = J0 + jl;
        uint32_t w = 0, c = 0;
        // loaded for every job, so that the loads do not wait for one another
        const bool guar = S.guaranteed[j] != 0;
        const int32_t ms = S.min_seg[j - X.jb];
        const uint32_t mc = S.min_c[j - X.jb], t = S.tenant[j];
        const uint32_t s0 = X.tb.seg_off[j], ns = X.tb.seg_off[j + 1] - s0;
        if (guar) {
            w = FL_GUAR;
            if (ms >= 0 && (uint32_t)ms < ns && mc < grid.n_cpu && t < S.n_tenants) {
                const uint32_t g = X.tb.seg_g[s0 + ms];
                const unsigned long long c64 = cpu_cost(grid, mc, g);
                if (g <= 0xFFFFu && c64 <= 0xFFFFFFFFull) {          // more can never fit a 32-bit capacity
                    w |= FL_CAND | g | (t << 16);
                    c = (uint32_t)c64;
                }
            }
        }
        word[jl] = w;
        cpus[jl] = c;
    }
    __syncthreads();

    if (tid < 64) {
        uint32_t freeG = cl.G, freeC = cl.C;
        uint32_t w = lane < nj ? word[lane] : 0u, c = lane < nj ? cpus[lane] : 0u;
        for (uint32_t base = 0; base < nj; base += 64) {
            if (freeG == 0) break;                            // every demand asks for at least one GPU
            const uint32_t jl = base + lane, next = jl + 64u;
            const uint32_t next_w = next < nj ? word[next] : 0u, next_c = next < nj ? cpus[next] : 0u;
            const uint32_t g = w & 0xFFFFu, t = (w >> 16) & 0xFFu;
            // Every lane has what is left of its job's tenant's quotas.  What does not fit now cannot fit later, so the
            // first that fits is granted and the others are asked again.
            uint32_t vg = quota[0][t], vc = quota[1][t];
            bool cand = (w & FL_CAND) != 0, granted = false, any = false;
            for (;;) {
                cand = cand && g <= vg && c <= vc && g <= freeG && c <= freeC;
                const unsigned long long fit = __ballot(cand);
                if (!fit) break;
                const uint32_t turn = (uint32_t)__ffsll((long long)fit) - 1u;
                const uint32_t tg = lane_value(g, turn), tc = lane_value(c, turn), tt = lane_value(t, turn);
                freeG -= tg; freeC -= tc;
                if (t == tt) { vg -= tg; vc -= tc; }
                if (lane == turn) { granted = true; cand = false; }
                any = true;
            }
            if (any) {
                if (granted) word[jl] = w | FL_GRANTED;
                quota[0][t] = vg; quota[1][t] = vc;           // (lanes of one tenant have the same)
                rs_wave_order();
                bool left = false;                            // is any GPU quota left at all?
#pragma unroll
                for (uint32_t r = 0; r < RK_MAX_TENANTS; r += 64) left = left || quota[0][r + lane] > 0;
                if (__ballot(left) == 0ull) break;
            }
            w = next_w; c = next_c;
        }
        if (lane == 0) { st.cap0[rnd] = freeG; st.cap0[X.R.n_rounds + rnd] = freeC; }
    }
    __syncthreads();

    for (uint32_t jl = tid; jl < nj; jl += FLOOR_THREADS) {
        const uint32_t jrel = J0 + jl - X.jb, w = word[jl];
        const bool granted = (w & FL_GRANTED) != 0;
        st.fl_gi[jrel] = granted ? S.min_seg[jrel] : -1;
        st.fl_ci[jrel] = granted ? S.min_c[jrel] : 0u;
        st.waits[jrel] = ((w & FL_GUAR) && !granted) ? RK_JOB_OUT : RK_JOB_NORMAL;
    }
}


// ------------------------------------------------------------------ Algorithm 1's Schedule as a loop
// From the state the jobs are in (paper Sec. 5.2, Algorithm 1 and the paragraph on shrinking): privileged jobs
// (below their floor) first in job order, then the others sorted once by GPU slope, CPU slope, index.  A job takes
// its next step (to its floor while below it, else the larger amount with the highest slope) when the amount can be
// gathered from what is free and from the jobs with the lowest slope among those above their own floor, each of
// which steps down to its next useful amount; a job may be shrunk when the taker's slope is higher than its own or
// the taker is below its floor, and the step is committed when all was found and (unless the taker is below its
// floor) the taker gains more than the others lose; otherwise everything is put back.
//
// One workgroup: the rule is sequential.  Its first wavefront makes a whole step of ScheduleJob by itself: the slopes of
// the jobs that can give stand together in LDS (a few hundred of thousands hold something), and a job's own steps and
// its first step down were found when its state last changed (RsNext, RsGives), so a step is a search over LDS and one
// round of loads per job that gives.  Between two barriers after a committed step all wavefronts find these again for the
// jobs that it changed; the look for the next job that has something to do needs no sort, and every thread has the values
// it asks of its own jobs in registers.
constexpr uint32_t RS_TOUCHED = 512;      // jobs changed by a step whose list is in LDS
constexpr uint32_t RS_UPDATES = 64;        // ... whose new values go from LDS to the threads that have them (beyond: from memory)
constexpr uint32_t RS_JOB_BITS = 14;       // a job or a place in the list of holders
static_assert(RK_MAX_JOBS_PER_ROUND <= 1u << RS_JOB_BITS, "a job and its place share a word");

// Threads of the workgroup and, at most, jobs of a thread (whose values are in its registers: two words each, so that
// twelve jobs a thread at 1,024 threads would leave too few registers for the rest).  Up to 1,024 jobs four wavefronts
// are enough, and their barriers are cheaper.
constexpr int RS_THREADS = 512, RS_PER = RK_MAX_JOBS_PER_ROUND / RS_THREADS;
constexpr int RS_SMALL_THREADS = 256, RS_SMALL_PER = 4;

constexpr uint32_t RS_HAS_CPU = 1u << 22, RS_HOLDS = 1u << 23;       // the job has a CPU step; it holds something
static_assert(RK_MAX_G <= 0xFFFFu && RK_MAX_CPU_LEVELS <= 64, "a step's GPUs and a level fit a word");

struct RsRound {                 // what a round of the loop works on
    JobState st;                 // gi, g, ci: the state the loop works on (and the memory step reads)
    uint32_t n_jobs;
    unsigned long long G, C;
    const uint8_t *state;        // may be null
    const int32_t *cur_seg;
    const uint32_t *cur_c;
    const int32_t *floor_seg;    // may be null
    const uint32_t *floor_c;     // may be null
    float *ug;                   // per job, as the call finds it: slope of its next GPU step (0: none)
    uint32_t *about;             // ... GPUs that step adds | level << 16 | RS_HAS_CPU | RS_HOLDS
    unsigned long long *okey;    // its place in the order (0: not in it)
    RsNext *next;                // its steps up, kept current
    RsGives *gives;              // its steps down, kept current
    uint32_t *order, *touched, *first;
    uint32_t *stats;             // may be null: steps committed, jobs on the full path, shrinks applied, steps taken back
};

struct RsArgs {                  // the kernels' argument
    Ctx X;
    RsRound r;
    // several independent rounds over the same jobs (a workgroup per round): round k works on the slice [k * n_jobs, ...)
    // of every per-job array of r, reads the state arrays from k * state_stride on and its cluster from d_clusters[k]
    uint32_t near;                   // places in the list of holders whose steps down are kept in LDS
    uint32_t state_stride;
    const rk_cluster *d_clusters;    // null: the single round's G and C
};

// What the code of a round sees: its own slice of the per-job arrays, and the table, grid and curves where the kernel
// arguments hold them (a copy of the grid's level arrays would live in scratch memory).
struct RsView : RsRound {
    const Ctx &X;
    __device__ RsView(const RsRound &r, const Ctx &x) : RsRound(r), X(x) {}
};

// The view of round k: every per-job array moved to the round's slice.
__device__ __forceinline__ RsView rs_round(const RsArgs &K, uint32_t r) {
    RsView A(K.r, K.X);
    const RsRound &B = K.r;
    const size_t at = (size_t)r * (B.n_jobs ? B.n_jobs : 1u), from = (size_t)r * K.state_stride;
    A.st.gi += at; A.st.g += at; A.st.ci += at;
    if (B.state) A.state += from;
    A.cur_seg += from; A.cur_c += from;
    if (B.floor_seg) A.floor_seg += from;
    if (B.floor_c) A.floor_c += from;
    A.ug += at; A.about += at; A.okey += at; A.next += at; A.gives += at;
    A.order += at; A.touched += at; A.first += at;
    if (B.stats) A.stats += 4 * (size_t)r;
    if (K.d_clusters) { A.G = K.d_clusters[r].G; A.C = K.d_clusters[r].C; }
    return A;
}

// rounds that share their jobs: where every round's slots begin, and the job of every slot
__global__ void k_rs_meta(uint32_t n_rounds, uint32_t n_jobs, uint32_t *round_off, uint32_t *jmap) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= n_rounds) round_off[i] = (uint32_t)(i * n_jobs);
    if (i < (size_t)n_rounds * n_jobs) jmap[i] = (uint32_t)(i % n_jobs);
}

// A wavefront has its job's rows in one round of loads where a thread follows one load with the next, so it is ahead until
// the wavefronts go over the chip several times: 7 us against 20 for 10,000 jobs, 18 against 22 for 40,000, 32 against 27 for
// 80,000, 223 against 149 for 640,000.
constexpr uint64_t RS_WAVE_JOBS = 49152;

// Every job on its own, any number of workgroups: what it holds, whether it comes first (a floor it is below), its
// cached slopes and steps.  LANES: 64, a wavefront per job, which has the job's rows at once (RsRows), or 1.
// A job's place in the order: GPU slope, then CPU slope, both descending (then index).
__device__ __forceinline__ unsigned long long rs_order_key(float ug, float uc) {
    return ((unsigned long long)rs_ordered(ug) << 32) | rs_ordered(uc);
}

template <uint32_t LANES>
__global__ void k_rs_prepare(RsArgs B) {
    const uint32_t j = (blockIdx.x * blockDim.x + threadIdx.x) / LANES, lane = threadIdx.x % LANES;
    if (j >= B.r.n_jobs) return;
    const RsView A = rs_round(B, blockIdx.y);
    int32_t gi = -1;
    uint32_t ci = 0;
    if (rs_holds(A, j) && A.cur_seg[j] >= 0 && (uint32_t)A.cur_seg[j] < rs_ns(A, j) && A.cur_c[j] < A.X.grid.n_cpu) {
        gi = A.cur_seg[j]; ci = A.cur_c[j];
    }
    const int32_t fl = rs_fl_s(A, j);
    const bool below = fl >= 0 && gi < fl;
    const uint32_t so = A.X.tb.seg_off[j], ns = A.X.tb.seg_off[j + 1] - so;
    const RsKept k = rs_keep<LANES>(A, j, so, ns, gi, ci, -1, lane, RS_ALL_PARTS, A.gives + j, nullptr);
    if (lane == 0) {
        const bool part = rs_part(A, j);
        A.st.gi[j] = gi; A.st.ci[j] = ci; A.st.g[j] = k.g;
        A.first[j] = part && below ? 1u : 0u;
        A.ug[j] = k.ug; A.about[j] = k.dg | (ci << 16) | (k.uc > 0.f ? RS_HAS_CPU : 0u) | (gi >= 0 ? RS_HOLDS : 0u);
        A.okey[j] = part && !below ? rs_order_key(k.ug, k.uc) : 0ull;
    }
}

// Dynamic LDS of k_reschedule: two slopes and the job (half a word) of every place in the list of holders; and what the
// jobs in the first places give, as many as there is room for up to RS_NEAR (the others' is in memory).
constexpr size_t RS_LDS_MOST = 136 * 1024;                  // 160 KiB less what the kernel declares
constexpr uint32_t RS_NEAR = 512;
// Lists are whole rounds of a wavefront's loads long, infinite behind the holders: no load asks whether it is inside.
constexpr uint32_t RS_LIST = 512;
static_assert(RK_MAX_JOBS_PER_ROUND % RS_LIST == 0, "the longest list is not longer for it");
__host__ __device__ inline uint32_t rs_list(uint32_t J) { return J ? (J + RS_LIST - 1u) & ~(RS_LIST - 1u) : RS_LIST; }
static inline size_t rs_list_bytes(size_t J) { return (size_t)rs_list((uint32_t)J) * (2 * sizeof(float) + sizeof(uint16_t)); }
static inline uint32_t rs_near(size_t J) {
    const size_t fit = (RS_LDS_MOST - rs_list_bytes(J)) / sizeof(RsGives), most = J < RS_NEAR ? J : RS_NEAR;
    return (uint32_t)(fit < most ? fit : most);
}

// Bound by the latency of one small decision after the other: about 0.4 us for a search for the job to shrink, 0.5 us for
// what it gives, 2.5 us for a committed step's new values (a job's rows come from memory that other chiplets wrote), 4 us
// for a look after one.  10,000 jobs on 4,096 GPUs, 15 jobs on the full path, 22 steps committed, 49 shrinks: 374 -> 242 us;
// 9,999 jobs with floors, several hundred steps: 4.2 -> 3.4 ms; while all wavefronts searched all jobs, with a barrier on
// either side of every decision, and a look read seven values of every job from memory.  Where thousands hold something a
// search by one wavefront takes longer than one by all: 4,486 holders, 5,297 steps 74.0 ms then and 60.7 now (95.3 with
// every search in two passes of single loads), 42,980 steps of a CPU level 222 and 235 (329); 1,348 holders, 13,119 such
// steps 62.7 and 62.6 (75.6); 29 holders, 244 steps 0.93 and 0.93 (1.03 with two wavefronts per changed job at all times).
// (A load that asks whether it is inside the list, and takes a constant where it is not, becomes flat loads from either
// place: 70 and 260 ms.)
template <int THREADS, int PER>
__global__ __launch_bounds__(THREADS) void k_reschedule(RsArgs B) {
    constexpr uint32_t WAVES = THREADS / 64, NONE = 0xFFFFFFFFu, JOB = (1u << RS_JOB_BITS) - 1u, MARK = 0x8000u;
    static_assert(WAVES >= 2 && WAVES <= 16, "two wavefronts find the lowest slopes, a row of 16 lanes reduces what all found");
    extern __shared__ uint4 sh_raw[];
    RsView A = rs_round(B, blockIdx.x);
    __shared__ RsNext sh_next;
    // the jobs that the step under way has changed: place << RS_JOB_BITS | job, amounts << 16 | level and the two slopes
    // before it; and the amounts << 16 | level now
    __shared__ uint4 sh_touched[RS_TOUCHED];
    __shared__ uint32_t sh_now[RS_TOUCHED], sh_so[RS_TOUCHED];          // ... where their amounts begin, and how many they are
    __shared__ uint16_t sh_ns[RS_TOUCHED];
    __shared__ uint32_t sh_upd[RS_UPDATES][4], sh_most[RK_MAX_CPU_LEVELS];
    __shared__ unsigned long long sh_free[2], sh_held[2][WAVES], sh_pick_key[WAVES];
    __shared__ uint32_t sh_pick_j[WAVES], sh_widx[WAVES];
    __shared__ RsMin sh_min[2];
    __shared__ uint32_t sh_holders, sh_changed[2], sh_nb;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const uint32_t J = A.n_jobs, room = rs_list(J), near = B.near;
    const float INF = __int_as_float(0x7F800000);
    // a place in the list of holders: what its job loses per GPU and per CPU it gives (infinite: nothing to give, or nobody
    // here), and the job, marked when the step under way has changed it
    float *const low_g = reinterpret_cast<float *>(sh_raw), *const low_c = low_g + room;
    uint16_t *const who = reinterpret_cast<uint16_t *>(low_c + room);
    RsGives *const near_gives = reinterpret_cast<RsGives *>(who + room);

    for (uint32_t i = tid; i < room / 2u; i += THREADS) {
        const uint32_t inf = 0x7F800000u;
        sh_raw[i] = uint4{inf, inf, inf, inf};
    }
    if (tid == 0) { sh_holders = 0u; sh_nb = 0u; }
    __syncthreads();
    // the state the jobs are in has been loaded (k_rs_prepare): the steps of a thread's jobs, who holds something, and what
    // they hold together
    float ug[PER];
    uint32_t about[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t j = tid + k * THREADS;
        ug[k] = j < J ? A.ug[j] : 0.f; about[k] = j < J ? A.about[j] : 0u;
        if (k % 8u == 7u) asm volatile("" ::: "memory");     // (addresses of a few jobs at a time in registers)
    }
    uint32_t changed_once = 0;                              // which of a thread's jobs have had another state
    unsigned long long hg = 0, hc = 0;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const unsigned long long m = __ballot((about[k] & RS_HOLDS) != 0u);
        if (!m) continue;
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&sh_holders, (uint32_t)__popcll(m));
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        if (about[k] & RS_HOLDS) who[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)(tid + k * THREADS);
    }
    __syncthreads();
    for (uint32_t i = tid; i < sh_holders; i += THREADS) {
        const uint32_t j = who[i], g = A.st.g[j], c = A.st.ci[j];
        const uint4 *const from = reinterpret_cast<const uint4 *>(A.gives + j);
        const uint4 n0 = from[0], n1 = from[1], n2 = from[2], n3 = from[3];
        low_g[i] = __uint_as_float(n1.y); low_c[i] = __uint_as_float(n2.w);      // (ds_g, ds_c)
        if (i < near) {
            uint4 *const to = reinterpret_cast<uint4 *>(near_gives + i);
            to[0] = n0; to[1] = n1; to[2] = n2; to[3] = n3;
        }
        A.next[j].slot = (int32_t)i;
        hg += g; hc += cpu_cost(A.X.grid, c, g);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) { hg += __shfl_xor(hg, off, 64); hc += __shfl_xor(hc, off, 64); }
    if (lane == 0) { sh_held[0][wave] = hg; sh_held[1][wave] = hc; }
    __syncthreads();
    if (tid == 0) {
        unsigned long long g = 0, c = 0;
        for (uint32_t w = 0; w < WAVES; ++w) { g += sh_held[0][w]; c += sh_held[1][w]; }
        sh_free[0] = g < A.G ? A.G - g : 0ull;
        sh_free[1] = c < A.C ? A.C - c : 0ull;
    }
    __syncthreads();

    // A wavefront finds the place with the lowest slope (the lower job among equal slopes); false: nobody gives.  Four places
    // per lane and load, two loads on their way; only where several places have the slope are they looked for again.
    auto lowest = [&](const float *low, uint32_t n, float &slope, uint32_t &place) -> bool {
        const uint32_t n4 = (n + 3u) / 4u;
        const float4 *const q4 = reinterpret_cast<const float4 *>(low);
        float4 q = q4[lane];                                 // the lane's first quad with its lowest slope, and where that is
        float least = fminf(fminf(q.x, q.y), fminf(q.z, q.w));
        uint32_t quad = lane;
        bool more = false;                                   // ... and another quad has it as well
        auto look_at = [&](const float4 &r, uint32_t at) {
            const float m = fminf(fminf(r.x, r.y), fminf(r.z, r.w));
            more = m < least ? false : more | (m == least);
            if (m < least) { least = m; quad = at; }
        };
        if (n4 > 64u) {
            look_at(q4[64u + lane], 64u + lane);
            for (uint32_t i = 128u; i < n4; i += 128u) {
                const float4 r0 = q4[i + lane], r1 = q4[i + 64u + lane];
                look_at(r0, i + lane);
                look_at(r1, i + 64u + lane);
            }
            if (quad != lane) q = q4[quad];
        }
        const uint32_t top = wave_min_u32_rows(least < INF ? rs_ordered(least) : NONE);
        if (top == NONE) return false;
        slope = rs_unordered(top);
        const unsigned long long mx = __ballot(q.x == slope), my = __ballot(q.y == slope), mz = __ballot(q.z == slope), mw = __ballot(q.w == slope);
        const unsigned long long any = mx | my | mz | mw;
        if (!(any & (any - 1ull)) && !((mx & my) | ((mx | my) & mz) | ((mx | my | mz) & mw)) && !(__ballot(more) & any)) {   // one place has it
            place = 4u * wave_lane_u32(quad, (uint32_t)__ffsll((long long)any) - 1u) + (mx ? 0u : my ? 1u : mz ? 2u : 3u);
            return true;
        }
        uint32_t job = NONE, at = 0u;
        for (uint32_t i = lane; i < n4; i += 64u) {
            q = q4[i];
            const float x[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (uint32_t c = 0; c < 4; ++c)
                if (x[c] == slope) {
                    const uint32_t w = who[4u * i + c] & JOB;
                    if (w < job) { job = w; at = 4u * i + c; }
                }
        }
        const uint32_t first = wave_min_u32_rows(job);
        place = wave_lane_u32(at, (uint32_t)__ffsll((long long)__ballot(job == first)) - 1u);
        return true;
    };
    // ... and the lowest slope but that place's
    auto lowest_but = [&](const float *low, uint32_t n, uint32_t place) -> float {
        const uint32_t n4 = (n + 3u) / 4u;
        const float4 *const q4 = reinterpret_cast<const float4 *>(low);
        float rest = INF;
        for (uint32_t i = 0u; i < n4; i += 128u) {
            float4 r[2];
#pragma unroll
            for (uint32_t u = 0; u < 2; ++u) r[u] = q4[i + 64u * u + lane];
#pragma unroll
            for (uint32_t u = 0; u < 2; ++u) {
                const uint32_t c = i + 64u * u + lane == place / 4u ? place % 4u : 4u;
                if (c == 0u) r[u].x = INF;
                if (c == 1u) r[u].y = INF;
                if (c == 2u) r[u].z = INF;
                if (c == 3u) r[u].w = INF;
                rest = fminf(rest, fminf(fminf(r[u].x, r[u].y), fminf(r[u].z, r[u].w)));
            }
        }
        return rs_unordered(wave_min_u32_rows(rs_ordered(rest)));
    };

    // ---- the first wavefront's part: a step of ScheduleJob(j).  Values without a lane are the same in all lanes.
    uint32_t moves = 0, full = 0, shrinks = 0, undone = 0, holders = sh_holders;
    unsigned long long free_g = sh_free[0], free_c = sh_free[1];
    uint32_t turn = 0;                                       // which of sh_changed: the first wavefront may be a turn ahead
    auto one = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    auto onef = [](float x) { return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x))); };
    auto two = [&](unsigned long long x) { return ((unsigned long long)one((uint32_t)(x >> 32)) << 32) | one((uint32_t)x); };
    // a job's four pieces (RsNext or RsGives), from LDS or from memory: loads of their own, for one that may be either waits
    // for both kinds
    auto pieces = [](bool near_by, const void *lds, const void *mem, uint4 (&n)[4]) {
        if (near_by) {
            const uint4 *const from = static_cast<const uint4 *>(lds);
            n[0] = from[0]; n[1] = from[1]; n[2] = from[2]; n[3] = from[3];
            asm volatile("");
        } else {
            const uint4 *const from = static_cast<const uint4 *>(mem);
            n[0] = from[0]; n[1] = from[1]; n[2] = from[2]; n[3] = from[3];
        }
    };
    // res 0: GPUs, 1: CPUs; true: committed (and the jobs it changed are listed, j the last one)
    auto step = [&](uint32_t j, const RsNext &N, uint32_t res) -> bool {
        if (!(res == 0 ? N.tgt_g >= 0 : N.uc > 0.f)) return false;
        const bool below_min = res == 0 && (N.below_ns & RS_BELOW) != 0u;
        const float slope = res == 0 ? N.ug : N.uc, gain = res == 0 ? N.gain_g : N.gain_c;
        const unsigned long long need_g = res == 0 ? N.dg : 0u, need_c = res == 0 ? N.dcg : N.dcc, need = res == 0 ? need_g : need_c;
        int32_t slot = N.slot;
        float *const low = res == 0 ? low_g : low_c;
        float own = 0.f;
        if (slot >= 0 && (res == 0 ? free_g : free_c) < need) {              // j gives nothing to itself
            own = low[slot];
            rs_wave_order();
            if (lane == 0) low[slot] = INF;
            rs_wave_order();
        }
        unsigned long long av_g = free_g, av_c = free_c;
        float lost = 0.f;
        uint32_t touched = 0;
        bool ok = true;
        const unsigned long long had = res == 0 ? free_g : free_c;
        bool again = false;                                  // a job gave more than once
        auto list = [&](uint32_t place, uint32_t v, uint32_t before, float sg, float sc, uint32_t now, uint32_t so, uint32_t ns) {
            const uint32_t word = (place << RS_JOB_BITS) | v;
            if (lane == 0) {
                if (touched < RS_TOUCHED) {
                    sh_touched[touched] = uint4{word, before, __float_as_uint(sg), __float_as_uint(sc)};
                    sh_now[touched] = now; sh_so[touched] = so; sh_ns[touched] = (uint16_t)ns;
                } else {
                    A.touched[touched] = word;
                }
            }
            touched += 1u;
        };
        while ((res == 0 ? av_g : av_c) < need) {
            // the job with the lowest slope among those that can give (GetLowestSlopeOverMinJob)
            float s;
            uint32_t place;
            if (!lowest(low, holders, s, place) || !(below_min || slope > s)) { ok = false; break; }
            const uint32_t word = one(who[place]), v = word & JOB;
            unsigned long long dg0 = 0, dc0;
            float loss, ds_g, ds_c;
            int32_t gi;
            uint32_t ci;
            if (!(word & MARK)) {                            // its step down is known
                uint4 n[4];
                pieces(place < near, near_gives + place, A.gives + v, n);
                const RsGives gv = __builtin_bit_cast(RsGives, n);
                const uint32_t gis = one(gv.gis), ci0 = one(gv.ci_ns) & 0xFFu, ns = one(gv.ci_ns) >> 8;
                if (res == 0) {
                    dg0 = one(gv.dg0); dc0 = two(gv.dc0); loss = onef(gv.loss0); ds_g = gv.ds_g0; ds_c = gv.ds_c0;
                    gi = (int32_t)(int16_t)(gis & 0xFFFFu); ci = gi < 0 ? 0u : ci0;
                } else {
                    dc0 = two(gv.dc1); loss = onef(gv.loss1); ds_g = gv.ds_g1; ds_c = gv.ds_c1;
                    gi = (int32_t)(gis >> 16); ci = ci0 - 1u;
                }
                list(place, v, (gis & 0xFFFF0000u) | ci0, gv.ds_g, gv.ds_c, ((uint32_t)gi << 16) | ci, one(gv.so), ns);
            } else {                                         // it has given in this step
                const int32_t gi0 = (int32_t)one((uint32_t)A.st.gi[v]);
                const uint32_t ci0 = one(A.st.ci[v]), so = one(A.X.tb.seg_off[v]), ns = one(A.X.tb.seg_off[v + 1]) - so;
                const RsShrunk sk = rs_shrink_wave(A, v, so, ns, res, gi0, ci0, lane);
                dg0 = two(sk.gv.dg); dc0 = two(sk.gv.dc); loss = onef(sk.gv.loss); ds_g = sk.ds_g; ds_c = sk.ds_c;
                gi = sk.gi; ci = sk.ci;
                again = true;
            }
            if (lane == 0) {
                who[place] = (uint16_t)(v | MARK);
                low_g[place] = ds_g; low_c[place] = ds_c;
                A.st.gi[v] = gi; A.st.ci[v] = ci;
            }
            av_g += dg0; av_c += dc0;
            lost = lost + loss;
            shrinks += 1u;
            rs_wave_order();
        }
        if (ok && (av_g < need_g || av_c < need_c)) ok = false;
        if (ok && !below_min && !(gain > lost)) ok = false;
        rs_wave_order();
        for (uint32_t i = lane; i < touched; i += 64u) {     // a job per lane: no longer changed, and if need be as it was
            const bool far = i >= RS_TOUCHED;
            uint4 e = sh_touched[far ? 0u : i];
            if (far) e.x = A.touched[i];
            const uint32_t v = e.x & JOB, place = e.x >> RS_JOB_BITS;
            who[place] = (uint16_t)v;
            if (ok) {
                if (again && !far) sh_now[i] = ((uint32_t)A.st.gi[v] << 16) | A.st.ci[v];
                continue;
            }
            if (far) {
                uint4 n[4];
                pieces(place < near, near_gives + place, A.gives + v, n);
                const RsGives gv = __builtin_bit_cast(RsGives, n);
                e.y = (gv.gis & 0xFFFF0000u) | (gv.ci_ns & 0xFFu); e.z = __float_as_uint(gv.ds_g); e.w = __float_as_uint(gv.ds_c);
            }
            A.st.gi[v] = (int32_t)(e.y >> 16); A.st.ci[v] = e.y & 0xFFFFu;
            low_g[place] = __uint_as_float(e.z); low_c[place] = __uint_as_float(e.w);
        }
        if (slot >= 0 && had < need && lane == 0) low[slot] = own;
        rs_wave_order();
        if (!ok) { undone += touched ? 1u : 0u; return false; }
        free_g = av_g - need_g; free_c = av_c - need_c;
        if (slot < 0) {
            slot = (int32_t)holders;
            holders += 1u;
            if (lane == 0) { who[slot] = (uint16_t)j; sh_holders = holders; }
        }
        const int32_t gi_j = res == 0 ? N.tgt_g : N.gi;
        const uint32_t ci_j = res == 0 ? N.lvl_g : N.lvl_c;
        if (lane == 0) {
            A.st.gi[j] = gi_j; A.st.ci[j] = ci_j;
            sh_free[0] = free_g; sh_free[1] = free_c;
            sh_changed[turn] = touched + 1u;
        }
        list((uint32_t)slot, j, 0u, 0.f, 0.f, ((uint32_t)gi_j << 16) | ci_j, N.so, N.below_ns & ~RS_BELOW);
        if (touched > RS_TOUCHED) __threadfence_block();     // (part of the list, and what the jobs hold now, is in memory)
        moves += 1u;
        return true;
    };

    bool others = false;                                  // the privileged jobs are through
    // ScheduleJob(j): the first wavefront steps, then all find the steps of the jobs that a committed step changed.  True
    // when one was.
    auto schedule_job = [&](uint32_t j) -> bool {
        bool any = false;
        uint32_t res = 0;
        for (;;) {
            if (wave == 0) {
                uint4 n[4];
                pieces(any, &sh_next, A.next + j, n);
#pragma unroll
                for (uint32_t i = 0; i < 4; ++i) n[i] = uint4{one(n[i].x), one(n[i].y), one(n[i].z), one(n[i].w)};
                const RsNext N = __builtin_bit_cast(RsNext, n);
                while (res < 2u && !step(j, N, res)) ++res;
                if (res == 2u && lane == 0) sh_changed[turn] = 0u;
            } else if (any) {
                __threadfence_block();                       // (what this wavefront stored of the jobs that it refreshed)
            }
            rs_lds_barrier();
            const uint32_t changed = one(sh_changed[turn]);
            turn ^= 1u;
            if (!changed) return any;
            any = true;
            // Four wavefronts per job where there are enough, one per step, otherwise two: GPUs, CPUs.
            const uint32_t each = 4u * changed <= WAVES ? 2u : 1u;           // (log2)
            for (uint32_t i = wave; i < changed << each; i += WAVES) {
                const uint32_t at = i >> each, parts = each == 2u ? 1u << (i & 3u) : i & 1u ? RS_UP_C | RS_DOWN_C : RS_UP_G | RS_DOWN_G;
                const bool far = at >= RS_TOUCHED;
                const uint32_t e = one(far ? A.touched[at] : sh_touched[at].x), v = e & JOB, place = e >> RS_JOB_BITS;
                const uint32_t now = one(far ? ((uint32_t)A.st.gi[v] << 16) | A.st.ci[v] : sh_now[at]);
                const int32_t gi = (int32_t)(int16_t)(now >> 16);
                const uint32_t so = one(far ? A.X.tb.seg_off[v] : sh_so[at]), ns = one(far ? A.X.tb.seg_off[v + 1] - so : (uint32_t)sh_ns[at]);
                const RsKept k = rs_keep<64>(A, v, so, ns, gi, now & 0xFFFFu, (int32_t)place, lane, parts,
                                             place < near ? near_gives + place : A.gives + v, v == j ? &sh_next : nullptr);
                if (lane == 0) {
                    uint32_t *const u = at < RS_UPDATES ? sh_upd[at] : nullptr;
                    if (parts & RS_UP_G) {
                        A.st.g[v] = k.g;
                        if (u) { u[0] = v; u[1] = __float_as_uint(k.ug); u[2] = k.dg | ((now & 0xFFFFu) << 16) | (gi >= 0 ? RS_HOLDS : 0u); }
                    }
                    if (parts & RS_DOWN_G) low_g[place] = k.ds_g;
                    if ((parts & RS_UP_C) && u) u[3] = k.uc > 0.f ? RS_HAS_CPU : 0u;
                    if (parts & RS_DOWN_C) low_c[place] = k.ds_c;
                    if (!others && rs_part(A, v) && !A.first[v]) {           // (the order is not yet fixed)
                        uint32_t *const key = reinterpret_cast<uint32_t *>(A.okey + v);
                        if (parts & RS_UP_G) key[1] = rs_ordered(k.ug);
                        if (parts & RS_UP_C) key[0] = rs_ordered(k.uc);
                    }
                    // (what is read behind the barrier that follows; the rest is waited for before the next one)
                    if (place >= near || changed > RS_UPDATES) __threadfence_block();
                }
            }
            rs_lds_barrier();
            if (changed > RS_UPDATES) {                      // (too many for the list: all jobs' again)
                uint32_t tid_k = tid;
                asm volatile("" : "+v"(tid_k));
#pragma unroll
                for (uint32_t k = 0; k < PER; ++k) {
                    const uint32_t j = tid_k + k * THREADS;
                    if (j < J) {
                        const RsNext &N = A.next[j];
                        ug[k] = N.ug;
                        about[k] = N.dg | (A.st.ci[j] << 16) | (N.uc > 0.f ? RS_HAS_CPU : 0u) | (N.gi >= 0 ? RS_HOLDS : 0u);
                    }
                    asm volatile("" ::: "memory");
                }
                changed_once = ~0u;
                __syncthreads();                             // (the levels have been read: the next step writes them before it knows whether it stands)
                continue;
            }
            const uint32_t mine = lane < changed ? sh_upd[lane][0] : NONE;   // the threads that have these jobs
            unsigned long long m = __ballot(mine != NONE && (mine % THREADS) / 64u == wave);
            while (m) {
                const uint32_t i = (uint32_t)__ffsll((long long)m) - 1u, v = wave_lane_u32(mine, i);
                m &= m - 1ull;
                const float g = __uint_as_float(sh_upd[i][1]);
                const uint32_t d = sh_upd[i][2] | sh_upd[i][3];
#pragma unroll
                for (uint32_t k = 0; k < PER; ++k)
                    if (tid + k * THREADS == v) { ug[k] = g; about[k] = d; changed_once |= 1u << k; }
            }
        }
    };

    // privileged jobs, in job order.  Who they are is known from the start: a job never gives below its floor, so
    // only a job that begins below it can be below it.
    if (A.floor_seg) {
        for (uint32_t base = 0; base < J; base += THREADS) {                 // their list, in job order
            const uint32_t j = base + tid;
            const bool is = j < J && A.first[j] != 0u;
            const unsigned long long in_wave = __ballot(is);
            if (lane == 0) sh_widx[wave] = (uint32_t)__popcll(in_wave);
            __syncthreads();
            uint32_t before = sh_nb, all = 0;
            for (uint32_t w = 0; w < WAVES; ++w) {
                if (w < wave) before += sh_widx[w];
                all += sh_widx[w];
            }
            if (is) A.order[before + (uint32_t)__popcll(in_wave & ((1ull << lane) - 1ull))] = j;
            __syncthreads();
            if (tid == 0) sh_nb += all;
        }
    }
    __syncthreads();
    const uint32_t n_first = sh_nb;
    uint32_t k_first = 0;
    // Most jobs of a large round find nothing to do when their turn comes: no step, or a step that needs more than is
    // free while no other job's slope is lower than theirs.  Whether that is so follows from values that change only
    // when a step is committed: the job's own next steps (kept current for every job), what is free, and the two
    // lowest slopes among the jobs that can give.  Passing over such a job changes nothing, so the jobs need not be
    // sorted: all threads look for the first job in the order, after the one served last, that is not of that kind,
    // it is served in full, and the search starts again from the new state.
    bool fresh = true;                                    // a step was committed since the last look (or this is the first)
    uint32_t maybe = 0, yes = 0, passed = 0;              // a thread's jobs that may have something to do, that have, whose turn is over or never comes,
    unsigned long long my_key = 0ull, last_key = ~0ull;   // and the first of the second kind; last_*: the job served last (before every job at first)
    uint32_t my_j = NONE, last_j = 0u;
    static_assert(PER <= 32, "a thread's jobs are the bits of a word");
    // A wavefront asks those of its jobs that may have something to do whether they have, each thread the one with the highest
    // slope first, until none is left that could come before the first that has (a thread's jobs are in its registers by an
    // index the compiler knows; what is not there is asked of memory).
    auto settle = [&]() {
        const unsigned long long fr_g = sh_free[0], fr_c = sh_free[1];
        const RsMin mg = sh_min[0], mc = sh_min[1];
        for (;;) {
            float top = -1.f;
            uint32_t at = 0;
#pragma unroll
            for (uint32_t k = 0; k < PER; ++k) {          // (the slope of a job that has not changed is its place in the order)
                const float x = (changed_once >> k) & 1u ? INF : ug[k];
                const bool more = (((maybe >> k) & 1u) != 0u) & (x > top);
                top = more ? x : top; at = more ? k : at;
            }
            const uint32_t first = wave_max_u32_rows((uint32_t)(my_key >> 32));
            const bool ask = (top >= 0.f) & (rs_ordered(top) >= first);
            if (!__any(ask)) break;
            if (!ask) continue;
            const uint32_t j = tid + at * THREADS, bit = 1u << at;
            const RsNext *const N = A.next + j;
            const unsigned long long key = A.okey[j], cg = N->dcg, cc = N->dcc;
            const float up_g = N->ug, up_c = N->uc;
            const uint32_t dg = N->dg;
            const float lowest_g = j == mg.i1 ? mg.m2 : mg.m1, lowest_c = j == mc.i1 ? mc.m2 : mc.m1;
            // GPU step: none; or GPUs are short and nobody may be shrunk for it; or the GPUs are there and its CPUs are not
            const bool gpu_idle = !(up_g > 0.f) | (fr_g < dg ? !(up_g > lowest_g) : fr_c < cg);
            const bool cpu_idle = !(up_c > 0.f) | ((fr_c < cc) & !(up_c > lowest_c));
            const bool served = (key > last_key) | ((key == last_key) & (j <= last_j)) | (key == 0ull);
            maybe &= ~bit;
            passed |= served ? bit : 0u;
            if ((gpu_idle & cpu_idle) | served) continue;
            yes |= bit;
            if (key > my_key || (key == my_key && j < my_j)) { my_key = key; my_j = j; }
        }
    };
    auto look = [&]() {
        if (!others) {                                    // the others: their order is what the slopes are now
            others = true;
            __syncthreads();                              // (they were stored by whoever found them)
        }
        bool settle_now = false;
        if (fresh) {
            if (wave < 2u) {                              // the two lowest slopes, and whose the lowest is: GPUs, CPUs
                const float *const low = wave == 0u ? low_g : low_c;
                const uint32_t n = one(sh_holders);
                RsMin m = {INF, INF, NONE};
                uint32_t place;
                if (lowest(low, n, m.m1, place)) {
                    m.i1 = one(who[place]);
                    m.m2 = lowest_but(low, n, place);
                }
                if (lane == 0) sh_min[wave] = m;
            }
            if (wave == WAVES - 1u && lane < A.X.grid.n_cpu) {               // the GPUs whose CPUs are free, at every level
                const unsigned long long fr = sh_free[1], l = A.X.grid.cpu_levels[lane];
                const unsigned long long most = A.X.grid.cpu_mode ? fr / l : fr >= l ? RK_MAX_G : 0ull;
                sh_most[lane] = most < RK_MAX_G ? (uint32_t)most : RK_MAX_G;
            }
            __syncthreads();
            const uint32_t fr_g = sh_free[0] < RK_MAX_G ? (uint32_t)sh_free[0] : RK_MAX_G;       // (no step adds more)
            const float lowest_g = sh_min[0].m1, last_ug = last_key == ~0ull ? INF : rs_unordered((uint32_t)(last_key >> 32));
            const uint32_t held = A.X.grid.cpu_mode ? 0u : RS_HOLDS;         // CPUs that a job's amounts share: who holds something has them
            maybe = 0u;
#pragma unroll
            for (uint32_t k = 0; k < PER; ++k) {          // who may have something to do, by what the registers say
                const uint32_t w = about[k], dg = w & 0xFFFFu;
                const bool cpus = (dg <= sh_most[(w >> 16) & 63u]) | ((w & held) != 0u);
                const bool gpus = (ug[k] > 0.f) & ((fr_g < dg) ? (ug[k] > lowest_g) : cpus);
                const bool later = (((changed_once >> k) & 1u) != 0u) | !(ug[k] > last_ug);
                maybe |= ((gpus | ((w & RS_HAS_CPU) != 0u)) & later) ? 1u << k : 0u;
                if (k % 4u == 3u) asm volatile("" ::: "memory");
            }
            maybe &= ~passed;
            yes = 0u; my_key = 0ull; my_j = NONE;
            settle_now = true;
        } else if (wave == (last_j % THREADS) / 64u) {    // nothing was committed: only the thread whose job it was has another
            if (tid == last_j % THREADS) {
                yes &= ~(1u << (last_j / THREADS));
                my_key = 0ull; my_j = NONE;
                for (uint32_t m = yes; m; m &= m - 1u) {
                    const uint32_t j = tid + ((uint32_t)__ffs((int)m) - 1u) * THREADS;
                    const unsigned long long key = A.okey[j];
                    if (key > my_key) { my_key = key; my_j = j; }            // (ascending jobs)
                }
            }
            settle_now = true;
        }
        // the first of the threads' jobs in the order
        if (settle_now) {
            settle();
            unsigned long long key = 0ull;
            uint32_t j = NONE;
            if (__any(my_j != NONE)) {
                const uint32_t hi = (uint32_t)(my_key >> 32), lo = (uint32_t)my_key;
                const uint32_t top_hi = wave_max_u32_rows(hi), top_lo = wave_max_u32_rows(hi == top_hi ? lo : 0u);
                j = wave_min_u32_rows(hi == top_hi && lo == top_lo ? my_j : NONE);
                key = ((unsigned long long)top_hi << 32) | top_lo;
            }
            if (lane == 0) { sh_pick_key[wave] = key; sh_pick_j[wave] = j; }
        }
        rs_lds_barrier();
        {
            const uint32_t w = lane < WAVES ? lane : 0u;
            const unsigned long long k2 = sh_pick_key[w];
            const uint32_t j2 = sh_pick_j[w], hi2 = (uint32_t)(k2 >> 32), lo2 = (uint32_t)k2;
            const uint32_t hi = NONE - wave_lane_u32(row_min_u32(NONE - hi2), 0u), lo = NONE - wave_lane_u32(row_min_u32(hi2 == hi ? NONE - lo2 : NONE), 0u);
            last_key = ((unsigned long long)hi << 32) | lo;
            last_j = wave_lane_u32(row_min_u32(k2 == last_key ? j2 : NONE), 0u);
        }
    };
    for (;;) {                                            // one job per turn; ScheduleJob appears once in the code
        uint32_t j;
        if (k_first < n_first) {
            j = one(A.order[k_first++]);
        } else {
            look();
            if (last_j == NONE) break;
            full += 1u;
            j = last_j;
        }
        const bool any = schedule_job(j);
        fresh = any || !others;
    }
    if (tid == 0 && A.stats) { A.stats[0] = moves; A.stats[1] = full; A.stats[2] = shrinks; A.stats[3] = undone; }
}

// Scratch of rk_allocate_static: one array in the library's image, so every device the library is loaded on holds
// its own copy at its own address for as long as the process lives.  The name is a host-side stand-in only: host
// code uses the address that hipGetSymbolAddress returned for the context's device (rk_ctx::static_scratch).
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)12 << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

// Where the working buffers of a call come from: the context's grow-only device buffers (base == nullptr), or
// consecutive 256-byte aligned pieces of a fixed block (no allocation; a call that needs more fails).
struct Arena {
    unsigned char *base;
    size_t used, cap;
};

template <typename T>
int32_t scratch_typed(rk_ctx *ctx, Arena &arena, int slot, size_t count, T **out) {
    if (!arena.base) return rk_scratch(ctx, slot, count * sizeof(T), reinterpret_cast<void **>(out));
    size_t bytes = count * sizeof(T);
    bytes = ((bytes ? bytes : 1) + 255) & ~(size_t)255;
    if (arena.used + bytes > arena.cap)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "the round needs more than the %zu bytes of static scratch memory", arena.cap);
    *out = reinterpret_cast<T *>(arena.base + arena.used);
    arena.used += bytes;
    return RK_OK;
}

// *closed: the pass also took the memory step that ends the round
template <int PASS>
int32_t launch_pass(rk_ctx *ctx, const Ctx &X, const JobState &st, const HullBuf &H, const Hist &hist,
                    uint32_t n_rounds, uint32_t n_jobs, uint32_t mj, uint32_t max_segs, size_t tail_lds, size_t zero_bins,
                    rk_assign *assign, float *totals, bool *closed) {
    hipStream_t s = ctx->stream;
    const uint32_t hull_blocks = (n_jobs + (HULL_THREADS / 64) - 1) / (HULL_THREADS / 64);
    const dim3 job_grid(st.blocks_per_round, n_rounds);
    *closed = false;
    if (n_jobs > 0) {
        // amounts per job: GPU counts (at most max_segs) in the GPU pass, CPU levels in the CPU pass
        const uint32_t amounts = PASS == 0 ? max_segs : X.grid.n_cpu;
        const uint32_t waves = HULL_THREADS / 64;
        if (amounts <= 16) {
            k_hull_groups<PASS, 16><<<(n_jobs + 4 * waves - 1) / (4 * waves), HULL_THREADS, 0, s>>>(X, st, H, hist, zero_bins);
        } else if (amounts <= 32) {
            k_hull_groups<PASS, 32><<<(n_jobs + 2 * waves - 1) / (2 * waves), HULL_THREADS, 0, s>>>(X, st, H, hist, zero_bins);
        } else {
            k_hull<PASS><<<hull_blocks, HULL_THREADS, 0, s>>>(X, st, H, hist, zero_bins);
        }
        RK_CHECK_LAUNCH(ctx, "k_hull");
    }
    const size_t sel_lds = tail_lds > SELECT_HIST_BYTES ? tail_lds : SELECT_HIST_BYTES;
    if (mj <= SMALL_ROUND_JOBS) {
        // (as few wavefronts as give every job a thread: a step's barrier and reductions are theirs)
        if (mj <= TAIL_THREADS / 2) k_select_small<PASS, 1, TAIL_THREADS / 2><<<n_rounds, TAIL_THREADS / 2, sel_lds, s>>>(X, mj, st, H, assign, totals);
        else if (mj <= TAIL_THREADS) k_select_small<PASS, 1, TAIL_THREADS><<<n_rounds, TAIL_THREADS, sel_lds, s>>>(X, mj, st, H, assign, totals);
        else k_select_small<PASS, SMALL_ROUND_JOBS / TAIL_THREADS, TAIL_THREADS><<<n_rounds, TAIL_THREADS, sel_lds, s>>>(X, mj, st, H, assign, totals);
        RK_CHECK_LAUNCH(ctx, "k_select_small");
        *closed = PASS == 1;
        return RK_OK;
    }
    if constexpr (PASS == 1) {
        if ((uint64_t)(X.grid.n_cpu - 1u) * mj <= CPU_ONE_WG_STEPS) {
            k_select_small<1, TAIL_KMAX, TAIL_THREADS><<<n_rounds, TAIL_THREADS, sel_lds, s>>>(X, mj, st, H, assign, totals);
            RK_CHECK_LAUNCH(ctx, "k_select_small");
            return RK_OK;
        }
    }
    if (n_jobs > 0) {
        k_hist<PASS, 0><<<job_grid, JOB_THREADS, 0, s>>>(X, st, H, hist);
        RK_CHECK_LAUNCH(ctx, "k_hist<0>");
        k_hist<PASS, 1><<<job_grid, JOB_THREADS, 0, s>>>(X, st, H, hist);
        RK_CHECK_LAUNCH(ctx, "k_hist<1>");
    }
    k_apply<PASS><<<job_grid, JOB_THREADS, 0, s>>>(X, st, H, hist);
    RK_CHECK_LAUNCH(ctx, "k_apply");
    k_tail<PASS><<<n_rounds, TAIL_THREADS, tail_lds, s>>>(X, mj, st);
    RK_CHECK_LAUNCH(ctx, "k_tail");
    return RK_OK;
}

}  // namespace

// Once per context, with its device current: the address of this device's copy of the static scratch array, and
// the dynamic LDS limits of the kernels that may need more than the default (large rounds keep per-job state in LDS;
// the single-workgroup selection adds dynamic to static LDS).  Done here so that no later call has to.
int32_t rk_allocate_setup(rk_ctx *ctx) {
    void *p = nullptr;
    RK_HIP(ctx, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    ctx->static_scratch = static_cast<unsigned char *>(p);
    const void *big[] = {reinterpret_cast<const void *>(k_tail<0>), reinterpret_cast<const void *>(k_tail<1>),
                         reinterpret_cast<const void *>(k_floors),
                         reinterpret_cast<const void *>(k_select_small<1, TAIL_KMAX, TAIL_THREADS>)};
    for (const void *f : big) RK_HIP(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 152 * 1024));
    const void *small[] = {reinterpret_cast<const void *>(k_select_small<0, SMALL_ROUND_JOBS / TAIL_THREADS, TAIL_THREADS>),
                           reinterpret_cast<const void *>(k_select_small<1, SMALL_ROUND_JOBS / TAIL_THREADS, TAIL_THREADS>),
                           reinterpret_cast<const void *>(k_select_small<0, 1, TAIL_THREADS>), reinterpret_cast<const void *>(k_select_small<1, 1, TAIL_THREADS>),
                           reinterpret_cast<const void *>(k_select_small<0, 1, TAIL_THREADS / 2>), reinterpret_cast<const void *>(k_select_small<1, 1, TAIL_THREADS / 2>)};
    const void *rounds[] = {reinterpret_cast<const void *>(k_round_few<256>), reinterpret_cast<const void *>(k_round_few<FEW_THREADS>)};
    for (const void *f : rounds) RK_HIP(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 144 * 1024));
    constexpr int ALL = FEW_THREADS, HALF = FEW_THREADS / 2;
    const void *sim[] = {reinterpret_cast<const void *>(k_sim_few<ALL, false, false, false>), reinterpret_cast<const void *>(k_sim_few<ALL, true, false, false>),
                         reinterpret_cast<const void *>(k_sim_few<ALL, true, true, false>), reinterpret_cast<const void *>(k_sim_few<ALL, false, false, true>),
                         reinterpret_cast<const void *>(k_sim_few<ALL, true, false, true>), reinterpret_cast<const void *>(k_sim_few<ALL, true, true, true>),
                         reinterpret_cast<const void *>(k_sim_few<HALF, false, false, true>), reinterpret_cast<const void *>(k_sim_few<HALF, true, false, true>),
                         reinterpret_cast<const void *>(k_sim_few<HALF, true, true, true>)};
    for (const void *f : sim) RK_HIP(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, FEW_SIM_LDS));
    for (const void *f : small) RK_HIP(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024));
    return RK_OK;
}

// jobs of a round that may hold GPUs
static uint32_t few_holders(uint32_t max_jobs, const rk_cluster *one_cluster) {
    return one_cluster && one_cluster->G < max_jobs ? one_cluster->G : max_jobs;
}
bool rk_round_is_few(const rk_alloc_grid *grid, uint32_t max_jobs, uint32_t max_segs_per_job, const rk_cluster *one_cluster, bool model_curves) {
    return max_jobs > 0 && max_jobs <= FEW_JOBS && max_segs_per_job <= 64u &&
           (uint64_t)max_jobs * few_lanes(max_segs_per_job) <= FEW_GPU_LANES &&
           (uint64_t)few_holders(max_jobs, one_cluster) * few_lanes(grid->n_cpu) <= (model_curves ? FEW_CPU_LANES_MODEL : FEW_CPU_LANES);
}

int32_t rk_launch_allocate(rk_ctx *ctx, const float *ref_thr, const TableDev &tb, const rk_alloc_grid *grid,
                           uint32_t n_rounds, const uint32_t *d_round_off, const rk_cluster *d_clusters,
                           const rk_cluster *one_cluster, uint32_t jb, uint32_t n_jobs, uint32_t max_jobs,
                           uint32_t max_segs_per_job, const float *best_thr, const uint32_t *best_plan,
                           const float *curve_thr, const SlaDev *sla, const FloorsDev *given, const uint32_t *d_jmap,
                           rk_assign *assign, float *totals, bool static_scratch, bool model_curves, const TableGuard *guard) {
    if (n_rounds == 0) return RK_OK;
    Arena arena = {nullptr, 0, 0};
    if (static_scratch) {
        if (!ctx->static_scratch) return rk_fail(ctx, RK_ERR_DEVICE, "the static scratch memory was not set up");
        arena = Arena{ctx->static_scratch, 0, STATIC_SCRATCH_BYTES};
    }
    if (d_jmap && (sla || given || jb != 0))
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "rounds that share jobs take neither floors nor a job range");
    if (max_jobs > RK_MAX_JOBS_PER_ROUND)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "a round has %u jobs, the allocation kernels take up to %u", max_jobs,
                       RK_MAX_JOBS_PER_ROUND);
    int32_t rc;
    HullBuf H;
    H.stride = n_jobs ? n_jobs : 1;
    H.width = max_segs_per_job > grid->n_cpu ? max_segs_per_job : grid->n_cpu;   // the longest walk of either pass
    if (H.width == 0) H.width = 1;
    // Rounds of few jobs take one launch, and none of the walk buffers and histograms.
    const uint32_t lanes0 = few_lanes(max_segs_per_job), lanes1 = few_lanes(grid->n_cpu);
    const uint32_t holders = few_holders(max_jobs, one_cluster);
    // (a simulation's tick that one workgroup takes well does not come here: k_sim_few)
    const bool few = !given && rk_round_is_few(grid, max_jobs, max_segs_per_job, one_cluster, model_curves);
    if (guard && !few) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "only the one launch of small rounds takes a guard");
    const size_t entries = few ? 0 : (size_t)H.stride * H.width;
    if ((rc = scratch_typed(ctx, arena, SL_HULL_KEY, entries, &H.key))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_HULL_RAW, entries, &H.raw))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_HULL_TGT, entries, &H.tgt))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_HULL_DG, entries, &H.dg))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_HULL_DC, entries, &H.dc))) return rc;
    JobState st;
    st.blocks_per_round = (max_jobs + JOB_THREADS - 1) / JOB_THREADS;
    if (st.blocks_per_round == 0) st.blocks_per_round = 1;
    if ((rc = scratch_typed(ctx, arena, SL_ST_GI, (size_t)H.stride, &st.gi))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_G, (size_t)H.stride, &st.g))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_CI, (size_t)H.stride, &st.ci))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_STEP_SLOPE, (size_t)H.stride, &st.step_slope))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_STEP_TGT, (size_t)H.stride, &st.step_tgt))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_STEP_DG, (size_t)H.stride, &st.step_dg))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_FREEG, (size_t)n_rounds * 2, &st.free_g))) return rc;   // [free G | free C] after apply
    if ((rc = scratch_typed(ctx, arena, SL_ST_FREEC, (size_t)n_rounds + ((size_t)n_rounds + 1) / 2, &st.free_c))) return rc;
    st.cpu_steps = reinterpret_cast<uint32_t *>(st.free_c + n_rounds);
    if ((rc = scratch_typed(ctx, arena, SL_ST_PARTIAL, (size_t)n_rounds * st.blocks_per_round * 2, &st.partial))) return rc;
    st.fl_gi = nullptr; st.fl_ci = nullptr; st.waits = nullptr; st.cap0 = nullptr;
    if (given) {
        st.fl_gi = given->gi; st.fl_ci = given->ci; st.waits = given->state; st.cap0 = given->cap0;
    } else if (sla) {
        if ((rc = scratch_typed(ctx, arena, SL_FL_GI, (size_t)H.stride, &st.fl_gi))) return rc;
        if ((rc = scratch_typed(ctx, arena, SL_FL_CI, (size_t)H.stride, &st.fl_ci))) return rc;
        if ((rc = scratch_typed(ctx, arena, SL_FL_WAITS, (size_t)H.stride, &st.waits))) return rc;
        if ((rc = scratch_typed(ctx, arena, SL_FL_CAP0, (size_t)n_rounds * 2, &st.cap0))) return rc;
    }
    Hist hist;
    const size_t hist_bins = few ? 0 : (size_t)n_rounds * 4 * HIST_WORDS;
    if ((rc = scratch_typed(ctx, arena, SL_HIST_G, hist_bins, &hist.g))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_HIST_C, hist_bins, &hist.c))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_HIST_CUT, few ? 0 : (size_t)n_rounds, &hist.cut))) return rc;

    Ctx X;
    X.ref_thr = ref_thr; X.tb = tb; X.grid = grid_dev(grid); X.jb = jb; X.jmap = d_jmap;
    X.best_thr = best_thr; X.best_plan = best_plan; X.curve_thr = curve_thr;
    X.R.round_off = d_round_off; X.R.clusters = d_clusters; X.R.n_rounds = n_rounds;
    X.R.inline_one = one_cluster ? 1u : 0u;
    X.R.off0 = jb; X.R.off1 = jb + n_jobs;
    X.R.cl = one_cluster ? *one_cluster : rk_cluster{0u, 0u, 0.f};

    const uint32_t mj = max_jobs ? ((max_jobs + 1u) & ~1u) : 2u;
    const size_t lds = tail_lds_bytes(mj);
    // (the kernels' dynamic LDS limits were raised when the context was made: rk_allocate_setup)
    hipStream_t s = ctx->stream;
    // Histograms start at zero: the first walk kernel clears them for both passes on its way (fill code, no
    // memset, so the sequence can be captured in a graph).  Rounds large enough to use them have jobs, so that
    // kernel always runs.
    const bool hists = mj > SMALL_ROUND_JOBS;
    if (sla && !given) {
        k_floors<<<n_rounds, FLOOR_THREADS, (size_t)mj * 8, s>>>(X, st, *sla, mj);
        RK_CHECK_LAUNCH(ctx, "k_floors");
    }
    if (few) {
        const uint32_t jobs = (max_jobs + 3u) & ~3u, gpu = max_jobs * lanes0, cpu = holders * lanes1, near = gpu > cpu ? gpu : cpu;
        // fewer wavefronts at the barriers where four have all the lanes (8 jobs 36.3 and 35.6 us a round; 64 jobs of 16 lanes
        // 41.1, with 512 threads 42.8, with 256 48.2)
        const int threads = gpu <= 256u && cpu <= 256u && max_jobs <= 256u ? 256 : FEW_THREADS;
        const size_t few_lds = FEW_FIXED_BYTES + (size_t)jobs * FEW_JOB_BYTES + (size_t)near * FEW_LANE_BYTES;
        auto *kernel = threads == 256 ? k_round_few<256> : k_round_few<FEW_THREADS>;
        kernel<<<n_rounds, threads, few_lds, s>>>(X, st, max_jobs, lanes0, lanes1, near, assign, totals, guard ? *guard : TableGuard{});
        RK_CHECK_LAUNCH(ctx, "k_round_few");
        return RK_OK;
    }
    bool closed = false;
    if ((rc = launch_pass<0>(ctx, X, st, H, hist, n_rounds, n_jobs, mj, max_segs_per_job, lds, hists ? hist_bins : 0, assign,
                             totals, &closed))) return rc;
    if ((rc = launch_pass<1>(ctx, X, st, H, hist, n_rounds, n_jobs, mj, max_segs_per_job, lds, 0, assign, totals,
                             &closed))) return rc;
    if (closed) return RK_OK;                                   // the CPU pass's selection took the memory step
    if (max_jobs > 0) {
        k_mem_wish<<<dim3(st.blocks_per_round, n_rounds), JOB_THREADS, 0, s>>>(X, st, assign);
        RK_CHECK_LAUNCH(ctx, "k_mem_wish");
    }
    k_mem_finish<<<n_rounds, 64, 0, s>>>(X, st, assign, totals);
    RK_CHECK_LAUNCH(ctx, "k_mem_finish");
    return RK_OK;
}

// LDS of k_sim_few but the words per lane, and the lanes that fit beside it.
static size_t few_sim_job_lds(uint32_t n_jobs) { return FEW_FIXED_BYTES + (size_t)((n_jobs + 3u) & ~3u) * FEW_JOB_BYTES; }
static uint32_t few_sim_room(uint32_t n_jobs) { return (uint32_t)((FEW_SIM_LDS - few_sim_job_lds(n_jobs)) / FEW_LANE_BYTES) & ~63u; }

SimFew rk_sim_few(uint32_t n_jobs, uint32_t max_segs_per_job, const rk_alloc_grid *grid, const rk_cluster *cluster, uint32_t *most) {
    *most = 0;
    if (n_jobs > FEW_JOBS || max_segs_per_job > 64u) return SIM_NOT_FEW;
    const uint32_t lanes0 = few_lanes(max_segs_per_job), line = lanes0 == 16u ? FEW_TICK_LANES_16 : FEW_TICK_LANES, room = few_sim_room(n_jobs);
    *most = (line < room ? line : room) / lanes0;              // (the GPU pass is in LDS)
    const uint32_t holders = cluster->G < n_jobs ? cluster->G : n_jobs, lanes = holders * few_lanes(grid->n_cpu);
    const uint32_t turns = (lanes + FEW_THREADS - 1u) / FEW_THREADS;
    return n_jobs <= *most && lanes <= room && turns * grid->n_cpu <= FEW_TICK_WALK ? SIM_ALWAYS_FEW : SIM_OFTEN_FEW;
}

int32_t rk_launch_sim_few(rk_ctx *ctx, const SimArgs &A, const float *ref_thr, const rk_alloc_grid *grid, uint32_t max_segs_per_job,
                          const float *best_thr, const uint32_t *best_plan, const float *curve_thr, rk_assign *assign,
                          uint32_t n_launches, bool begin, bool often, uint32_t most) {
    const uint32_t J = A.n_jobs, lanes0 = few_lanes(max_segs_per_job), lanes1 = few_lanes(grid->n_cpu);
    Ctx X;
    X.ref_thr = ref_thr; X.tb = A.tb; X.grid = A.grid; X.jb = 0; X.jmap = nullptr;
    X.best_thr = best_thr; X.best_plan = best_plan; X.curve_thr = curve_thr;
    X.R = RoundArgs{nullptr, nullptr, 1u, 1u, 0u, J, A.cl};
    const uint32_t part = J < most ? J : most, holders = A.cl.G < part ? A.cl.G : part, gpu = part * lanes0, cpu = holders * lanes1;
    const uint32_t need = gpu > cpu ? gpu : cpu, room = few_sim_room(J), near = need < room ? need : room;
    uint32_t *far = nullptr;
    int32_t rc;
    if (cpu > near && (rc = rk_scratch(ctx, SL_HULL_KEY, (size_t)cpu * FEW_LANE_BYTES, (void **)&far))) return rc;
    // What the jobs do in a round from nothing is found beforehand where that is not too much for memory or for the ticks: 6,900
    // walks take 10 us, a round is 8 us shorter.
    FewStates T = {nullptr, nullptr, nullptr, max_segs_per_job + 1u, A.cl.G};
    const uint64_t walks = (uint64_t)J * T.rows, walk_bytes = walks * lanes0 * sizeof(uint4), cpu_bytes = (uint64_t)J * max_segs_per_job * sizeof(uint4);
    const uint64_t allowed_bytes = ((uint64_t)A.cl.G + 1u) * J;
    const bool known = A.n_ticks > 1u && max_segs_per_job > 0u && walk_bytes <= FEW_WALK_BYTES && allowed_bytes <= FEW_WALK_BYTES / 8u &&
                       walks <= (uint64_t)FEW_WALKS_PER_TICK * A.n_ticks;
    if (known) {
        char *mem;
        if ((rc = rk_scratch(ctx, SL_FEW_STATES, walk_bytes + cpu_bytes + allowed_bytes, (void **)&mem))) return rc;
        uint4 *walk = reinterpret_cast<uint4 *>(mem), *cpu_end = reinterpret_cast<uint4 *>(mem + walk_bytes);
        uint8_t *allowed = reinterpret_cast<uint8_t *>(mem + walk_bytes + cpu_bytes);
        T.walk = walk; T.cpu = cpu_end; T.allowed = allowed;
        if (begin) {
            k_few_states<<<J, 256, 0, ctx->stream>>>(X, lanes0, lanes1, T, walk, cpu_end, allowed);
            RK_CHECK_LAUNCH(ctx, "k_few_states");
        }
    }
    constexpr int ALL = FEW_THREADS, HALF = FEW_THREADS / 2;
    const bool half = known && J <= HALF;
    auto *kernel = !often ? (half ? k_sim_few<HALF, false, false, true> : known ? k_sim_few<ALL, false, false, true> : k_sim_few<ALL, false, false, false>)
                   : far  ? (half ? k_sim_few<HALF, true, true, true> : known ? k_sim_few<ALL, true, true, true> : k_sim_few<ALL, true, true, false>)
                          : (half ? k_sim_few<HALF, true, false, true> : known ? k_sim_few<ALL, true, false, true> : k_sim_few<ALL, true, false, false>);
    for (uint32_t i = 0; i < n_launches; ++i) {                // (the pass over GPUs is always in LDS: rk_sim_few)
        kernel<<<1, half ? HALF : ALL, few_sim_job_lds(J) + (size_t)near * FEW_LANE_BYTES, ctx->stream>>>(
            X, A, T, begin && i == 0 ? 1u : 0u, i ? 1u : 0u, most, lanes0, lanes1, near, far, cpu, assign);
        RK_CHECK_LAUNCH(ctx, "k_sim_few");
    }
    return RK_OK;
}

extern "C" int32_t rk_reschedule(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                 const rk_alloc_grid *grid, const rk_cluster *cluster, const float *best_thr,
                                 const uint32_t *best_plan, const float *curve_thr, const rk_job_state *jobs_state,
                                 rk_assign *assign, float *total, uint32_t *stats) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if ((rc = rk_check_table(ctx, table, 0, table ? table->n_jobs : 0))) return rc;
    if ((rc = rk_check_grid(ctx, grid))) return rc;
    if (!cluster || !total || !jobs_state) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    const uint32_t J = table->n_jobs;
    if (J > 0 && (!ref_thr || !assign || !jobs_state->cur_seg || !jobs_state->cur_c ||
                  (table->n_segs > 0 && (!best_thr || !best_plan || !curve_thr))))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (!(cluster->host_mem_gb >= 0.f)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "host_mem_gb negative or NaN");
    if (table->max_segs_per_job > 32767u) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 32767 segments per job");
    if (J > RK_MAX_JOBS_PER_ROUND)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u jobs, the allocation kernels take up to %u", J, RK_MAX_JOBS_PER_ROUND);
    RK_HIP(ctx, hipSetDevice(ctx->device));
    return rk_launch_reschedule(ctx, ref_thr, table, grid, cluster, best_thr, best_plan, curve_thr, jobs_state, assign, total,
                                stats);
}

// n_rounds independent rounds over the same jobs (clusters [host] n_rounds entries; round r reads the state arrays from
// r * state_stride on and writes assign[r * n_jobs ...], totals[r], stats[4 r ...]); one round: the plain loop
static int32_t launch_reschedule_rounds(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                        const rk_alloc_grid *grid, uint32_t n_rounds, const rk_cluster *clusters,
                                        const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                                        const rk_job_state *jobs_state, uint32_t state_stride, rk_assign *assign,
                                        float *totals, uint32_t *stats) {
    const uint32_t J = table->n_jobs;
    int32_t rc;
    Arena arena = {nullptr, 0, 0};
    const size_t n = J ? J : 1, all = n * n_rounds;
    RsArgs K;
    RsRound &A = K.r;
    JobState &st = A.st;
    st = JobState{};
    st.blocks_per_round = (J + JOB_THREADS - 1) / JOB_THREADS;
    if (st.blocks_per_round == 0) st.blocks_per_round = 1;
    if ((rc = scratch_typed(ctx, arena, SL_ST_GI, all, &st.gi))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_G, all, &st.g))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_CI, all, &st.ci))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_ST_PARTIAL, (size_t)st.blocks_per_round * 2 * n_rounds, &st.partial))) return rc;
    uint32_t *u32;
    if ((rc = scratch_typed(ctx, arena, SL_RS_U32, all * 5, &u32))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_RS_U64, all, &A.okey))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_RS_NEXT, all, &A.next))) return rc;
    if ((rc = scratch_typed(ctx, arena, SL_RS_GIVES, all, &A.gives))) return rc;
    A.ug = reinterpret_cast<float *>(u32);
    A.about = u32 + all; A.order = u32 + 2 * all; A.touched = u32 + 3 * all; A.first = u32 + 4 * all;
    Ctx &X = K.X;
    X.ref_thr = ref_thr; X.tb = table_dev(table); X.grid = grid_dev(grid); X.jb = 0; X.jmap = nullptr;
    X.best_thr = best_thr; X.best_plan = best_plan; X.curve_thr = curve_thr;
    X.R.round_off = nullptr; X.R.clusters = nullptr; X.R.n_rounds = n_rounds; X.R.inline_one = 1u;
    X.R.off0 = 0; X.R.off1 = J; X.R.cl = clusters[0];
    A.n_jobs = J; A.G = clusters[0].G; A.C = clusters[0].C;
    A.state = jobs_state->state; A.cur_seg = jobs_state->cur_seg; A.cur_c = jobs_state->cur_c;
    A.floor_seg = jobs_state->floor_seg; A.floor_c = jobs_state->floor_c;
    A.stats = stats;
    K.state_stride = state_stride; K.d_clusters = nullptr;
    hipStream_t s = ctx->stream;
    if (n_rounds > 1) {                                        // the rounds' slots, the job of every slot, the clusters
        const size_t off_bytes = (((size_t)n_rounds + 1) * 4 + 15) & ~(size_t)15;
        char *d_meta;
        uint32_t *d_jmap;
        if ((rc = rk_scratch(ctx, SL_ROUND_META, off_bytes + (size_t)n_rounds * sizeof(rk_cluster), (void **)&d_meta))) return rc;
        if ((rc = rk_scratch(ctx, SL_JMAP, all * 4, (void **)&d_jmap))) return rc;
        RK_HIP(ctx, hipMemcpyAsync(d_meta + off_bytes, clusters, (size_t)n_rounds * sizeof(rk_cluster), hipMemcpyHostToDevice, s));
        const size_t most = all > (size_t)n_rounds + 1 ? all : (size_t)n_rounds + 1;
        k_rs_meta<<<(uint32_t)((most + 255) / 256), 256, 0, s>>>(n_rounds, J, reinterpret_cast<uint32_t *>(d_meta), d_jmap);
        RK_CHECK_LAUNCH(ctx, "k_rs_meta");
        X.R.round_off = reinterpret_cast<const uint32_t *>(d_meta);
        X.R.clusters = reinterpret_cast<const rk_cluster *>(d_meta + off_bytes);
        X.R.inline_one = 0u;
        X.jmap = d_jmap;
        K.d_clusters = X.R.clusters;
    }
    if (J > 0) {
        if ((uint64_t)J * n_rounds <= RS_WAVE_JOBS) k_rs_prepare<64><<<dim3((J + 3) / 4, n_rounds), 256, 0, s>>>(K);
        else k_rs_prepare<1><<<dim3((J + 255) / 256, n_rounds), 256, 0, s>>>(K);
        RK_CHECK_LAUNCH(ctx, "k_rs_prepare");
    }
    K.near = rs_near(J);
    const size_t lds = rs_list_bytes(J ? J : 1u) + (size_t)K.near * sizeof(RsGives);
    if (lds > 32 * 1024 && !ctx->loop_lds_raised) {
        const auto most = hipFuncAttributeMaxDynamicSharedMemorySize;
        RK_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(k_reschedule<RS_THREADS, RS_PER>), most, (int)RS_LDS_MOST));
        RK_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(k_reschedule<RS_SMALL_THREADS, RS_SMALL_PER>), most, (int)RS_LDS_MOST));
        ctx->loop_lds_raised = true;
    }
    if (J <= RS_SMALL_THREADS * RS_SMALL_PER) k_reschedule<RS_SMALL_THREADS, RS_SMALL_PER><<<n_rounds, RS_SMALL_THREADS, lds, s>>>(K);
    else k_reschedule<RS_THREADS, RS_PER><<<n_rounds, RS_THREADS, lds, s>>>(K);
    RK_CHECK_LAUNCH(ctx, "k_reschedule");
    if (J > 0) {
        k_mem_wish<<<dim3(st.blocks_per_round, n_rounds), JOB_THREADS, 0, s>>>(X, st, assign);
        RK_CHECK_LAUNCH(ctx, "k_mem_wish");
    }
    k_mem_finish<<<n_rounds, 64, 0, s>>>(X, st, assign, totals);
    RK_CHECK_LAUNCH(ctx, "k_mem_finish");
    return RK_OK;
}

int32_t rk_launch_reschedule(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table, const rk_alloc_grid *grid,
                             const rk_cluster *cluster, const float *best_thr, const uint32_t *best_plan,
                             const float *curve_thr, const rk_job_state *jobs_state, rk_assign *assign, float *total,
                             uint32_t *stats) {
    return launch_reschedule_rounds(ctx, ref_thr, table, grid, 1, cluster, best_thr, best_plan, curve_thr, jobs_state, 0, assign,
                                    total, stats);
}

extern "C" int32_t rk_reschedule_rounds(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                        const rk_alloc_grid *grid, uint32_t n_rounds, const rk_cluster *clusters,
                                        const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                                        const rk_job_state *jobs_state, uint32_t state_stride, rk_assign *assign,
                                        float *totals, uint32_t *stats) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if ((rc = rk_check_table(ctx, table, 0, table ? table->n_jobs : 0))) return rc;
    if ((rc = rk_check_grid(ctx, grid))) return rc;
    if (!clusters || !totals || !jobs_state) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (n_rounds == 0) return RK_OK;
    const uint32_t J = table->n_jobs;
    if (J > 0 && (!ref_thr || !assign || !jobs_state->cur_seg || !jobs_state->cur_c ||
                  (table->n_segs > 0 && (!best_thr || !best_plan || !curve_thr))))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (state_stride != 0 && state_stride != J)
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "state_stride must be 0 (one state for all rounds) or n_jobs (one per round)");
    for (uint32_t r = 0; r < n_rounds; ++r)
        if (!(clusters[r].host_mem_gb >= 0.f)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "host_mem_gb negative or NaN");
    if (table->max_segs_per_job > 32767u) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 32767 segments per job");
    if (J > RK_MAX_JOBS_PER_ROUND)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u jobs, the allocation kernels take up to %u", J, RK_MAX_JOBS_PER_ROUND);
    if ((uint64_t)n_rounds * (J ? J : 1) > (1ull << 26) || n_rounds > 65535u)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "rounds x jobs above 2^26, or more than 65535 rounds");
    RK_HIP(ctx, hipSetDevice(ctx->device));
    return launch_reschedule_rounds(ctx, ref_thr, table, grid, n_rounds, clusters, best_thr, best_plan, curve_thr, jobs_state,
                                    state_stride, assign, totals, stats);
}

static int32_t allocate_one_round(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                  const rk_alloc_grid *grid, const rk_cluster *cluster, uint32_t jb, uint32_t je,
                                  const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                                  rk_assign *assign, float *total, bool static_scratch) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if ((rc = rk_check_table(ctx, table, jb, je))) return rc;
    if ((rc = rk_check_grid(ctx, grid))) return rc;
    if (!cluster || !total) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    // (a table without any segment has empty value arrays, which may be null)
    if (je > jb && (!ref_thr || !assign || (table->n_segs > 0 && (!best_thr || !best_plan || !curve_thr))))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (!(cluster->host_mem_gb >= 0.f)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "host_mem_gb negative or NaN");
    if (table->max_segs_per_job > 32767u) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 32767 segments per job");
    if (static_scratch) {
        const uint64_t width = table->max_segs_per_job > grid->n_cpu ? table->max_segs_per_job : grid->n_cpu;
        if ((uint64_t)(je - jb) * width > RK_STATIC_MAX_STEPS)
            return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u jobs x %llu amounts per job: rk_allocate_static takes up to %u",
                           je - jb, (unsigned long long)width, RK_STATIC_MAX_STEPS);
    }
    RK_HIP(ctx, hipSetDevice(ctx->device));
    return rk_launch_allocate(ctx, ref_thr, table_dev(table), grid, 1, nullptr, nullptr, cluster, jb, je - jb, je - jb,
                              table->max_segs_per_job, best_thr, best_plan, curve_thr, nullptr, nullptr, nullptr, assign,
                              total, static_scratch);
}

extern "C" int32_t rk_allocate(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                               const rk_alloc_grid *grid, const rk_cluster *cluster, uint32_t jb, uint32_t je,
                               const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                               rk_assign *assign, float *total) {
    return allocate_one_round(ctx, ref_thr, table, grid, cluster, jb, je, best_thr, best_plan, curve_thr, assign, total,
                              false);
}

extern "C" int32_t rk_allocate_static(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                      const rk_alloc_grid *grid, const rk_cluster *cluster, uint32_t jb, uint32_t je,
                                      const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                                      rk_assign *assign, float *total) {
    return allocate_one_round(ctx, ref_thr, table, grid, cluster, jb, je, best_thr, best_plan, curve_thr, assign, total,
                              true);
}

int32_t rk_check_sla(rk_ctx *ctx, const rk_sla *sla, bool need_request) {
    if (!sla) return rk_fail(ctx, RK_ERR_INVALID_ARG, "sla is null");
    if (!sla->guaranteed || !sla->tenant) return rk_fail(ctx, RK_ERR_INVALID_ARG, "sla: guaranteed or tenant is null");
    if (sla->n_tenants > RK_MAX_TENANTS)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u tenants, at most %u", sla->n_tenants, RK_MAX_TENANTS);
    if (sla->n_tenants > 0 && (!sla->quota_g || !sla->quota_c)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "sla: quota array is null");
    if (need_request && (!sla->req_g || !sla->req_c || !sla->req_m || !sla->base_thr))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "sla: request or baseline array is null");
    return RK_OK;
}

extern "C" int32_t rk_allocate_sla(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                   const rk_alloc_grid *grid, const rk_cluster *cluster, uint32_t jb, uint32_t je,
                                   const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                                   const rk_sla *sla, const int32_t *min_seg, const uint32_t *min_c,
                                   rk_assign *assign, float *total) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if ((rc = rk_check_table(ctx, table, jb, je))) return rc;
    if ((rc = rk_check_grid(ctx, grid))) return rc;
    if (!cluster || !total) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (je > jb && (!ref_thr || !assign || !min_seg || !min_c ||
                    (table->n_segs > 0 && (!best_thr || !best_plan || !curve_thr))))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (je > jb && (rc = rk_check_sla(ctx, sla, false))) return rc;
    if (!(cluster->host_mem_gb >= 0.f)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "host_mem_gb negative or NaN");
    if (table->max_segs_per_job > 32767u) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 32767 segments per job");
    RK_HIP(ctx, hipSetDevice(ctx->device));
    SlaDev S = {};
    if (je > jb) S = SlaDev{sla->guaranteed, sla->tenant, min_seg, min_c, sla->n_tenants, sla->quota_g, sla->quota_c};
    return rk_launch_allocate(ctx, ref_thr, table_dev(table), grid, 1, nullptr, nullptr, cluster, jb, je - jb, je - jb,
                              table->max_segs_per_job, best_thr, best_plan, curve_thr, je > jb ? &S : nullptr, nullptr,
                              nullptr, assign, total, false);
}
