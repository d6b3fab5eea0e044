// Algorithm 1's Schedule with ScheduleJob searching the cluster node by node (paper Sec. 5.2, Algorithm 1 and the
// paragraph on shrinking): on each node the job first takes what is free, then the job with the lowest slope among
// the jobs ON THAT NODE that are above their own minimum is shrunk while that is permitted, then the next node.
// State, order of the jobs, steps, slopes, permit cases and commit rule are those of the loop over the cluster's
// totals (k_reschedule); this kernel adds where things are.
//
// Nodes: per node what is free (GPUs, CPUs) and the list of its residents (job, GPUs of that job here); a node of n
// GPUs has at most n residents, so the lists are a fixed table.  The CPU levels are CPUs per GPU: a part of k GPUs at
// level l holds cpu_levels[l] * k CPUs of its node.  A job's parts are not stored per job; they are found by looking
// the job up on every node (all threads, a node or a few per thread) in the few places that need them.
//
// k_nd_init clears the nodes and k_nd_prepare loads every job on its own, over the whole chip: what it holds, its parts
// booked on the nodes, its cached slopes and next steps.  The loop itself is one workgroup: the rule is sequential.
// Parallel are: the refresh of the jobs a committed step changed (a wavefront per job), the walk over the nodes as
// long as nobody has to be asked (a node per thread: what each offers, a prefix sum that cuts the offers at what the
// job lacks, and the first node where the job still lacks GPUs and somebody may be shrunk), the parts a shrunk job
// gives up elsewhere (a suffix sum over the nodes), the look-ahead that passes over jobs with nothing to do, and
// everything about memory and the records.
// Before a step touches anything the node tables are copied; a step that is not committed copies them back.
#include <type_traits>

#include "rk_internal.h"
#include "rk_model.h"
#include "rk_loop.h"
#include "rk_sim.h"

namespace {

constexpr int ND_THREADS = 1024;
constexpr int ND_WAVES = ND_THREADS / 64;
constexpr uint32_t ND_NONE = 0xFFFFFFFFu;
constexpr uint32_t ND_PER = (RK_MAX_NODES + ND_THREADS - 1) / ND_THREADS;   // nodes per thread, at most
// The workgroup of rounds whose jobs are in LDS too: 512 threads find the new values of up to four jobs at once after a
// committed step (406 jobs: 256 threads are 3 % slower), 256 have the cheaper barriers where a thread has one job at most
// (60 jobs: 512 threads are 2 % slower).
constexpr int ND_SMALL_THREADS = 512, ND_FEW_THREADS = 256;
constexpr size_t ND_LDS_MOST = 156 * 1024;                                    // dynamic LDS of a workgroup: 160 KiB less what the kernels declare
constexpr uint32_t ND_MAX_GPUS = 1u << 20;                                   // nodes x GPUs per node

struct NdCurves {
    const float *ref_thr;
    TableDev tb;
    GridDev grid;
    const float *best_thr;
    const uint32_t *best_plan;
    const float *curve_thr;
};
struct NdHold { int32_t *gi; uint32_t *ci; };

struct NdBody {
    NdHold st;                       // what every job holds: index of its GPU count (-1 nothing), CPU level
    unsigned long long G;            // GPUs of the cluster
    uint32_t n_jobs, n_nodes, gpn, cpn;
    float mem_gb;                    // host memory of a node
    const uint8_t *state;            // may be null
    const int32_t *cur_seg;
    const uint32_t *cur_c;
    const int32_t *floor_seg;        // may be null
    const uint32_t *floor_c;         // may be null
    const uint32_t *prev_off;        // may be null (then nobody may hold anything)
    const rk_place_entry *prev_entries;
    uint64_t n_prev;                 // records in prev_entries
    // nodes: one block of words [free_g | free_c | cnt | res], and its copy; a resident is (job << 16 | its GPUs here),
    // ND_EMPTY past a node's last one (in the tables kept in LDS)
    uint32_t *free_g, *free_c, *cnt, *res;
    uint32_t *keep_nodes;
    uint32_t nodes_words;
    // per job: cached slopes (see rk_loop.h), the order, what a step touched
    float *ds_g, *ds_c, *ug, *uc, *sg, *sc, *keep_ds;
    float *gain_g, *gain_c;          // ... and of a job's next GPU / CPU step: its gain,
    int32_t *tgt_g;                  // the GPU step's target amount,
    uint32_t *lvl_g, *lvl_c;         // the CPU level each step ends on (no GPU step: tgt_g -1; no CPU step: uc 0)
    uint32_t *udg, *touched, *stamp, *first, *keep_ci, *np, *tmp_off;
    int32_t *keep_gi;
    RsGives *gives;                  // its step down in GPUs, kept for the first time a step asks for it (k_nodes_lds; the first half and
    uint4 *give;                     // `ci_ns, so`); in LDS with the jobs: GPUs, loss, amount after, slope after,
    float *give_c;                   // and CPU slope after (then give is not null)
    unsigned long long *udc_c, *okey;   // okey: a job's place in the order (k_nodes_lds)
    uint32_t *plist;                 // parts of one job: (node, GPUs) pairs, ascending node
    uint32_t *tmp_parts;             // parts of all jobs, (node << 16 | GPUs), grouped by job, in no order
    rk_assign *assign;
    uint32_t *place_off;
    rk_place_entry *entries;
    float *total;
    uint32_t *stats;                 // may be null
    const uint32_t *seg_off;         // the plan table's, or its copy in LDS
    bool book;                       // k_nd_prepare books the parts on the nodes (the kernel with the nodes in LDS does it itself)
};
// What the device code sees: the body by value (registers), the table, grid and curves where the kernel arguments
// hold them (a copy of the grid's level arrays would live in scratch memory).
struct NdArgs : NdBody {
    const NdCurves &X;
    __device__ NdArgs(const NdBody &b, const NdCurves &x) : NdBody(b), X(x) {}
};
struct NdKernArgs { NdCurves X; NdBody b; };       // the kernels' argument

__device__ __forceinline__ uint32_t nd_cpl(const NdArgs &A, uint32_t lvl) { return A.X.grid.cpu_levels[lvl]; }

// where job `job` is in node n's list, -1: not there
__device__ __forceinline__ int nd_find(const NdArgs &A, uint32_t n, uint32_t job) {
    const uint32_t c = A.cnt[n];
    const uint32_t *r = A.res + (size_t)n * A.gpn;
    for (uint32_t i = 0; i < c; ++i)
        if ((r[i] >> 16) == job) return (int)i;
    return -1;
}
__device__ __forceinline__ uint32_t nd_part(const NdArgs &A, uint32_t n, uint32_t job) {
    const int i = nd_find(A, n, job);
    return i < 0 ? 0u : A.res[(size_t)n * A.gpn + (uint32_t)i] & 0xFFFFu;
}
// job takes k free GPUs of node n, each with per_gpu CPUs (the caller has checked that they are free)
__device__ __forceinline__ void nd_add(const NdArgs &A, uint32_t n, uint32_t job, uint32_t k, uint32_t per_gpu) {
    A.free_g[n] -= k; A.free_c[n] -= k * per_gpu;
    const size_t base = (size_t)n * A.gpn;
    const int i = nd_find(A, n, job);
    if (i >= 0) { A.res[base + (uint32_t)i] += k; return; }
    const uint32_t c = A.cnt[n];
    if (c < A.gpn) { A.res[base + c] = (job << 16) | k; A.cnt[n] = c + 1u; }   // (always: a resident holds a GPU)
}
// job gives k GPUs of node n back, each with per_gpu CPUs
__device__ __forceinline__ void nd_drop(const NdArgs &A, uint32_t n, uint32_t job, uint32_t k, uint32_t per_gpu) {
    const int i = nd_find(A, n, job);
    if (i < 0) return;
    const size_t base = (size_t)n * A.gpn;
    A.free_g[n] += k; A.free_c[n] += k * per_gpu;
    const uint32_t left = (A.res[base + (uint32_t)i] & 0xFFFFu) - k;
    if (left) { A.res[base + (uint32_t)i] = (job << 16) | left; return; }
    const uint32_t c = A.cnt[n] - 1u;
    A.res[base + (uint32_t)i] = A.res[base + c];
    A.cnt[n] = c;
}
// GetLowestSlopeOverMinJob(n, resType): lowest cached slope among the residents of n other than j (infinite: gives
// nothing); lower job index among equal slopes; who = ND_NONE when nobody can give
__device__ __forceinline__ float nd_lowest_on(const NdArgs &A, uint32_t n, uint32_t j, const float *ds, uint32_t &who) {
    const float INF = __int_as_float(0x7F800000);
    float best = INF;
    who = ND_NONE;
    const uint32_t c = A.cnt[n];
    const uint32_t *r = A.res + (size_t)n * A.gpn;
    for (uint32_t i = 0; i < c; ++i) {
        const uint32_t v = r[i] >> 16;
        if (v == j) continue;
        const float s = ds[v];
        if (s < best || (s == best && s < INF && v < who)) { best = s; who = v; }
    }
    return best;
}

// The same for a whole wavefront, a resident per lane (64 at a time): the residents' slopes are asked for together.
__device__ __forceinline__ float nd_lowest_on_wave(const NdArgs &A, uint32_t n, uint32_t j, const float *ds, uint32_t &who,
                                                   uint32_t lane) {
    const float INF = __int_as_float(0x7F800000);
    const uint32_t c = A.cnt[n];
    const uint32_t *r = A.res + (size_t)n * A.gpn;
    unsigned long long low = ~0ull;                          // (slope as a word that orders like it, job)
    for (uint32_t b = 0; b < c; b += 64u) {
        const uint32_t i = b + lane;
        const uint32_t v = i < c ? r[i] >> 16 : j;
        const float s = v != j ? ds[v] : INF;
        const unsigned long long key = ((unsigned long long)rs_ordered(s) << 32) | v;
        if (s < INF && key < low) low = key;
    }
    low = wave_min_u64_rows(low);
    who = low == ~0ull ? ND_NONE : (uint32_t)low;
    return low == ~0ull ? INF : rs_unordered((uint32_t)(low >> 32));
}

// What job v, which holds (gi, ci), gives as a: kept for k_nodes_lds.
__device__ __forceinline__ void nd_keep_give(const NdArgs &A, uint32_t v, uint32_t so, uint32_t ns, int32_t gi, uint32_t ci, const RsGive &a, const RsShrunk &s) {
    if (A.give) {
        A.give[v] = uint4{(uint32_t)a.dg, __float_as_uint(a.loss), (uint32_t)s.gi, __float_as_uint(s.ds_g)};
        A.give_c[v] = s.ds_c;
    } else if (gi >= 0) {
        uint4 *const to = reinterpret_cast<uint4 *>(A.gives + v);
        to[0] = uint4{(uint32_t)a.dg, __float_as_uint(a.loss), ((uint32_t)gi << 16) | ((uint32_t)s.gi & 0xFFFFu), __float_as_uint(s.ds_g)};
        to[1] = uint4{__float_as_uint(s.ds_c), __float_as_uint(a.any ? a.slope : __int_as_float(0x7F800000)), ci | (ns << 8), so};
    }
}

// All cached values of job v from its present state: what it gives (rs_refresh_give) and its next steps in full, so
// that ScheduleJob need not search them again.  `lanes` threads share the search (1, or the 64 of a wavefront).
__device__ __forceinline__ void nd_refresh(const NdArgs &A, uint32_t v, uint32_t lane, uint32_t lanes) {
    const int32_t gi = A.st.gi[v];
    const uint32_t ci = A.st.ci[v], so = A.seg_off[v], ns = A.seg_off[v + 1] - so;
    const RsGive a = rs_down_gpu_at(A, v, gi, ci, lane, lanes), b = rs_down_cpu_at(A, v, gi, ci);
    const RsStep ug = rs_up_gpu(A, v, gi, ci, lane, lanes), uc = rs_up_cpu(A, v, gi, ci, lane, lanes);
    RsShrunk s = {a, -1, 0u, 0.f, 0.f};
    if (a.any) s = rs_shrunk_at(A, v, 0, gi, ci, a, lane, lanes);
    if (lane != 0) return;
    nd_keep_give(A, v, so, ns, gi, ci, a, s);
    A.ds_g[v] = a.any ? a.slope : __int_as_float(0x7F800000);
    A.ds_c[v] = b.any ? b.slope : __int_as_float(0x7F800000);
    A.ug[v] = ug.any ? ug.slope : 0.f; A.udg[v] = (uint32_t)ug.dg;   // (a step that exists has its slope here)
    A.uc[v] = uc.any ? uc.slope : 0.f; A.udc_c[v] = uc.dc;
    A.gain_g[v] = ug.gain; A.gain_c[v] = uc.gain; A.tgt_g[v] = ug.tgt; A.lvl_g[v] = ug.lvl; A.lvl_c[v] = uc.lvl;
}
// nd_refresh for a whole wavefront: a job of at most 64 amounts that is not below its floor has its rows loaded at
// once, an amount per lane, and every step comes from the registers (rs_rows).  The steps in GPUs and in CPUs may be
// left to two wavefronts (with_g, with_c).
__device__ __forceinline__ void nd_refresh_wave(const NdArgs &A, uint32_t v, int32_t gi, uint32_t ci, uint32_t lane, bool with_g = true, bool with_c = true) {
    const int32_t fl = rs_fl_s(A, v);
    const uint32_t so = A.seg_off[v], ns = A.seg_off[v + 1] - so;
    if (ns > 64u || (fl >= 0 && gi < fl)) { if (with_g) nd_refresh(A, v, lane, 64); return; }
    const RsRows R = rs_rows(A, v, so, ns, gi, ci, lane);
    if (with_g) {
        const RsGive a = rs_down_gpu_rows(A, R, R.curve, gi, ci, lane);
        const RsStep ug = rs_up_gpu_rows(A, R, gi, ci, lane);
        RsShrunk s = {a, -1, 0u, 0.f, 0.f};
        if (a.any) s = rs_shrunk_rows(A, R, 0, gi, ci, a, lane);
        if (lane == 0) {
            nd_keep_give(A, v, so, ns, gi, ci, a, s);
            A.ds_g[v] = a.any ? a.slope : __int_as_float(0x7F800000);
            A.ug[v] = ug.any ? ug.slope : 0.f; A.udg[v] = (uint32_t)ug.dg;
            A.gain_g[v] = ug.gain; A.tgt_g[v] = ug.tgt; A.lvl_g[v] = ug.lvl;
        }
    }
    if (with_c) {
        const RsGive b = rs_down_cpu_rows(A, R, gi, ci, rs_lane_f(R.best, gi), rs_lane_f(R.best_lo, gi));
        const RsStep uc = rs_up_cpu_rows(A, R, gi, ci, lane);
        if (lane == 0) {
            A.ds_c[v] = b.any ? b.slope : __int_as_float(0x7F800000);
            A.uc[v] = uc.any ? uc.slope : 0.f; A.udc_c[v] = uc.dc;
            A.gain_c[v] = uc.gain; A.lvl_c[v] = uc.lvl;
        }
    }
}
// the cached next step of job j: res 0 GPUs, 1 CPU level
__device__ __forceinline__ RsStep nd_cached_step(const NdArgs &A, uint32_t j, uint32_t res) {
    RsStep st;
    if (res == 0) {
        st.tgt = A.tgt_g[j]; st.any = st.tgt >= 0 ? 1u : 0u; st.lvl = A.lvl_g[j]; st.slope = A.ug[j]; st.gain = A.gain_g[j];
        st.dg = A.udg[j]; st.dc = 0ull;        // (a GPU step's CPUs come with its GPUs)
    } else {
        st.tgt = A.st.gi[j]; st.lvl = A.lvl_c[j]; st.slope = A.uc[j]; st.any = st.slope > 0.f ? 1u : 0u; st.gain = A.gain_c[j];
        st.dg = 0ull; st.dc = A.udc_c[j];
    }
    return st;
}

// The nodes, all free and empty (for k_reschedule_nodes).
__global__ void k_nd_init(NdKernArgs K) {
    const NdArgs A(K.b, K.X);
    const uint32_t n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n < A.n_nodes) { A.free_g[n] = A.gpn; A.free_c[n] = A.cpn; A.cnt[n] = 0u; }
}

// Every job on its own, a wavefront per job: what it holds, whether it comes first (bit 0 of `first`), whether its
// parts are a placement (bit 1: they are not), its cached slopes; with A.book its parts are booked on the nodes (atomics;
// a node that ends up holding more than it has is seen by the main kernel).
__global__ void k_nd_prepare(NdKernArgs K) {
    const NdArgs A(K.b, K.X);
    const uint32_t j = (blockIdx.x * blockDim.x + threadIdx.x) >> 6, lane = threadIdx.x & 63u;
    if (j >= A.n_jobs) return;
    const uint32_t N = A.n_nodes;
    int32_t gi = -1;
    uint32_t ci = 0;
    const int32_t seg = A.cur_seg[j];
    const uint32_t lvl = A.cur_c[j];
    if (rs_holds(A, j) && seg >= 0 && (uint32_t)seg < rs_ns(A, j) && lvl < A.X.grid.n_cpu) { gi = seg; ci = lvl; }
    const int32_t fl = rs_fl_s(A, j);
    bool good = true;
    if (gi >= 0) {
        good = A.prev_off != nullptr && A.prev_entries != nullptr;
        const uint32_t a = good ? A.prev_off[j] : 0u, b = good ? A.prev_off[j + 1] : 0u;
        if (a > b || b > A.n_prev) good = false;
        if (good) {
            const uint32_t per_gpu = nd_cpl(A, ci);
            unsigned long long sum = 0;
            bool ok = true;
            for (uint32_t i = a + lane; i < b; i += 64u) {
                const rk_place_entry e = A.prev_entries[i];
                const long long last = i > a ? (long long)A.prev_entries[i - 1].node : -1;
                if (e.node >= N || (long long)e.node <= last || e.g == 0u || e.g > A.gpn || e.c > A.cpn ||
                    (unsigned long long)e.c != (unsigned long long)per_gpu * e.g) ok = false;
                sum += e.g;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, 64);
            good = __ballot(!ok) == 0ull && sum == rs_g(A, j, gi);
        }
        if (good && A.book)
            for (uint32_t i = a + lane; i < b; i += 64u) {
                const rk_place_entry e = A.prev_entries[i];
                const uint32_t slot = atomicAdd(&A.cnt[e.node], 1u);
                if (slot < A.gpn) A.res[(size_t)e.node * A.gpn + slot] = (j << 16) | e.g;
                // (wraps below zero when the node holds more than it has; the main kernel sees that)
                atomicSub(&A.free_g[e.node], e.g);
                atomicSub(&A.free_c[e.node], e.c);
            }
    }
    if (lane == 0) {
        A.st.gi[j] = gi; A.st.ci[j] = ci;
        A.first[j] = ((rs_part(A, j) && fl >= 0 && gi < fl) ? 1u : 0u) | (good ? 0u : 2u);
    }
    asm volatile("" ::: "memory");               // (nd_refresh's other lanes read what the first one stored)
    nd_refresh_wave(A, j, gi, ci, lane);
}

// What is kept of a job in a state (nothing or one of its amounts, a CPU level) does not depend on the other jobs, and a
// simulation's jobs have few states: they are all found once, over the whole chip, before the first tick.
// ND_STATE_WORDS words per state, in the order of NdField, and a record of what the job would run as at its best tier
// (throughput, plan, tier or ND_NONE, GPUs).  A job's states, `per_job` places: nothing at every level (only level 0 is
// used), then its amounts, each at every level.
enum NdField : uint32_t { ND_UG, ND_UDG, ND_GAIN_G, ND_TGT_G, ND_UC, ND_GAIN_C, ND_LVL_C, ND_DC_LO, ND_DC_HI, ND_DS_G, ND_DS_C,
                          ND_GIVES, ND_LOSS, ND_TO, ND_DS_G1, ND_DS_C1, ND_STATE_WORDS };
struct NdStates { uint32_t *words; uint4 *best; uint32_t per_job; };
__device__ __forceinline__ size_t nd_state_at(const NdStates &T, uint32_t j, uint32_t n_cpu, int32_t gi, uint32_t ci) {
    return j * T.per_job + (uint32_t)(gi + 1) * n_cpu + (gi < 0 ? 0u : ci);
}
// A workgroup per job and CPU level, a wavefront per amount.  406 jobs of up to 16 amounts at 5 levels: 34,000 states.
__global__ __launch_bounds__(256) void k_nd_states(NdKernArgs K, NdStates to) {
    const NdArgs A(K.b, K.X);
    const uint32_t j = blockIdx.x, ci = blockIdx.y, lane = threadIdx.x & 63u;
    const uint32_t so = A.seg_off[j], ns = A.seg_off[j + 1] - so, n_cpu = A.X.grid.n_cpu, n_mem = A.X.grid.n_mem;
    const float INF = __int_as_float(0x7F800000);
    for (int32_t gi = (int32_t)(threadIdx.x >> 6) - 1; gi < (int32_t)ns; gi += 4) {
        if (gi < 0 && ci > 0) continue;
        RsGive a, b;
        RsStep ug, uc;
        RsShrunk s;
        if (ns <= 64u) {
            const RsRows R = rs_rows(A, j, so, ns, gi, ci, lane);
            a = rs_down_gpu_rows(A, R, R.curve, gi, ci, lane);
            b = rs_down_cpu_rows(A, R, gi, ci, rs_lane_f(R.best, gi), rs_lane_f(R.best_lo, gi));
            ug = rs_up_gpu_rows(A, R, gi, ci, lane);
            uc = rs_up_cpu_rows(A, R, gi, ci, lane);
            s = RsShrunk{a, -1, 0u, 0.f, 0.f};
            if (a.any) s = rs_shrunk_rows(A, R, 0, gi, ci, a, lane);
        } else {
            a = rs_down_gpu_at(A, j, gi, ci, lane, 64);
            b = rs_down_cpu_at(A, j, gi, ci);
            ug = rs_up_gpu(A, j, gi, ci, lane, 64);
            uc = rs_up_cpu(A, j, gi, ci, lane, 64);
            s = RsShrunk{a, -1, 0u, 0.f, 0.f};
            if (a.any) s = rs_shrunk_at(A, j, 0, gi, ci, a, lane, 64);
        }
        const size_t at = nd_state_at(to, j, n_cpu, gi, ci);
        uint4 best = {0u, RK_NO_PLAN, ND_NONE, 0u};
        if (gi >= 0) {
            best.w = A.X.tb.seg_g[so + (uint32_t)gi];
            float top = 0.f;
            for (uint32_t m = 0; m < n_mem; ++m) {
                const uint64_t slot = (uint64_t)n_cpu * n_mem * so + ((uint64_t)ci * n_mem + m) * ns + (uint32_t)gi;
                const float v = A.X.best_thr[slot];
                if (v > top) { top = v; best.x = __float_as_uint(v); best.y = A.X.best_plan[slot]; best.z = m; }
            }
        }
        if (lane == 0) {
            uint4 *const w = reinterpret_cast<uint4 *>(to.words + at * ND_STATE_WORDS);
            w[0] = uint4{__float_as_uint(ug.any ? ug.slope : 0.f), (uint32_t)ug.dg, __float_as_uint(ug.gain), (uint32_t)ug.tgt};
            w[1] = uint4{__float_as_uint(uc.any ? uc.slope : 0.f), __float_as_uint(uc.gain), uc.lvl, (uint32_t)uc.dc};
            w[2] = uint4{(uint32_t)(uc.dc >> 32), __float_as_uint(a.any ? a.slope : INF), __float_as_uint(b.any ? b.slope : INF), (uint32_t)a.dg};
            w[3] = uint4{__float_as_uint(a.loss), (uint32_t)s.gi, __float_as_uint(s.ds_g), __float_as_uint(s.ds_c)};
            to.best[at] = best;
        }
    }
}

// exclusive prefix sum over the threads of the workgroup (thread order) and the sum of all; all threads call it
template <int THREADS>
__device__ __forceinline__ uint32_t nd_block_scan(uint32_t val, uint32_t &all, uint32_t *sh_scan) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t inc = val;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(inc, off, 64);
        if ((int)lane >= off) inc += o;
    }
    if (lane == 63) sh_scan[wave] = inc;
    __syncthreads();
    uint32_t base = 0;
    all = 0;
#pragma unroll
    for (uint32_t w = 0; w < THREADS / 64; ++w) { const uint32_t x = sh_scan[w]; if (w < wave) base += x; all += x; }
    __syncthreads();
    return base + inc - val;
}

// Nothing is scheduled: the state is no placement on these nodes.
template <int THREADS>
__device__ __forceinline__ void nd_refuse(const NdArgs &A) {
    for (uint32_t j = threadIdx.x; j < A.n_jobs; j += THREADS) {
        A.assign[j] = rk_assign{0u, 0u, 0.f, RK_NO_PLAN, 0.f};
        A.place_off[j] = 0u;
    }
    if (threadIdx.x == 0) {
        A.place_off[A.n_jobs] = 0u; *A.total = 0.f;
        if (A.stats) { A.stats[0] = 0u; A.stats[1] = 0u; A.stats[2] = 0u; A.stats[3] = 0u; A.stats[4] = 1u; }
    }
}

// Memory, then the records, from what the jobs hold and who is on the nodes.  np, off [n_jobs], parts [GPUs of all
// nodes], wish [n_jobs], list [jobs that hold something; may be where the residents are] and mem [n_nodes] are working
// memory, in LDS or not.  All threads call it.
template <int THREADS>
__device__ __forceinline__ void nd_finish(const NdArgs &A, uint32_t *np, uint32_t *off, uint32_t *parts, uint32_t *wish, uint32_t *list, float *mem,
                                          uint32_t *sh_scan) {
    constexpr uint32_t WAVES = THREADS / 64;
    __shared__ uint32_t sh_fit, sh_wide, sh_list;
    __shared__ double sh_sum[ND_WAVES];
    double *const share = reinterpret_cast<double *>(A.okey);                // [n_jobs] thr / ref_thr (the order has been served)
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t J = A.n_jobs, N = A.n_nodes, gpus = N * A.gpn;
    __syncthreads();
    for (uint32_t j = tid; j < J; j += THREADS) np[j] = 0u;
    for (uint32_t n = tid; n < N; n += THREADS) mem[n] = 0.f;
    if (tid == 0) { sh_fit = A.gpn <= 4096u ? 1u : 0u; sh_wide = 0u; sh_list = 0u; }
    __syncthreads();
    // the parts of all jobs, grouped by job (in no order yet): an entry of the nodes' tables per thread
    for (uint32_t i = tid; i < gpus; i += THREADS) {
        const uint32_t n = i / A.gpn;
        if (i - n * A.gpn < A.cnt[n]) atomicAdd(&np[A.res[i] >> 16], 1u);
    }
    __syncthreads();
    const uint32_t jobs_per_thread = (J + THREADS - 1) / THREADS;
    auto offsets = [&](uint32_t *to) {                                       // where every job's parts begin; returns their number
        uint32_t local = 0, all;
        for (uint32_t i = 0; i < jobs_per_thread; ++i) {
            const uint32_t j = tid * jobs_per_thread + i;
            if (j < J) local += np[j] & 0xFFFFu;
        }
        uint32_t at = nd_block_scan<THREADS>(local, all, sh_scan);
        for (uint32_t i = 0; i < jobs_per_thread; ++i) {
            const uint32_t j = tid * jobs_per_thread + i;
            if (j < J) { to[j] = at; at += np[j] & 0xFFFFu; }
        }
        return all;
    };
    offsets(off);
    __syncthreads();
    for (uint32_t i = tid; i < gpus; i += THREADS) {                         // (moves off[j] to the end of job j's parts)
        const uint32_t n = i / A.gpn;
        if (i - n * A.gpn < A.cnt[n]) {
            const uint32_t word = A.res[i];
            parts[atomicAdd(&off[word >> 16], 1u)] = (n << 16) | (word & 0xFFFFu);
        }
    }
    __syncthreads();
    // the jobs that hold something, listed in no order; the others' records
    for (uint32_t j0 = 0; j0 < J; j0 += THREADS) {
        const uint32_t j = j0 + tid;
        const bool holds = j < J && np[j] != 0u;
        const unsigned long long m = __ballot(holds);
        uint32_t base = 0;
        if (lane == 0 && m) base = atomicAdd(&sh_list, (uint32_t)__popcll(m));
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        if (holds) list[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = j;
        else if (j < J) A.assign[j] = rk_assign{0u, 0u, 0.f, RK_NO_PLAN, 0.f};
    }
    __syncthreads();
    const uint32_t n_list = sh_list;
    const uint64_t rows = (uint64_t)A.X.grid.n_cpu * A.X.grid.n_mem;
    const uint32_t n_mem = A.X.grid.n_mem;
    auto tier_cost = [&](uint32_t m, uint32_t g) {
        float v = A.X.grid.mem_levels_gb[m];
        if (A.X.grid.mem_mode) v = v * (float)g;
        return v;
    };
    auto slot_of = [&](uint32_t j, uint32_t m) {                             // of what job j holds, at tier m, in the curves' layout
        const uint32_t so = A.seg_off[j], ns = A.seg_off[j + 1] - so;
        return rows * so + ((uint64_t)A.st.ci[j] * n_mem + m) * ns + (uint32_t)A.st.gi[j];
    };
    auto gpus_of = [&](uint32_t j) { return A.X.tb.seg_g[A.seg_off[j] + (uint32_t)A.st.gi[j]]; };
    // np[j] holds the job's tier above its parts; a job without a tier is dropped: it has no parts
    auto settle = [&](uint32_t j, uint32_t bm) {
        if (bm != ND_NONE) np[j] = (np[j] & 0xFFFFu) | (bm << 16);
        else { off[j] -= np[j] & 0xFFFFu; np[j] = 0u; }
    };
    // the tier every job would like (highest throughput, smallest such tier), and what that asks of the nodes
    for (uint32_t h = tid; h < n_list; h += THREADS) {
        const uint32_t j = list[h], P = np[j], a = off[j] - P, g = gpus_of(j);
        uint32_t bm = ND_NONE;
        float bv = 0.f;
        for (uint32_t m = 0; m < n_mem; ++m) {
            const float v = A.X.best_thr[slot_of(j, m)];
            if (v > bv) { bv = v; bm = m; }
        }
        if (bm != ND_NONE) {
            const float cost = tier_cost(bm, g);
            for (uint32_t i = a; i < a + P; ++i) atomicAdd(&mem[parts[i] >> 16], (cost * (float)(parts[i] & 0xFFFFu)) / (float)g);
        }
        wish[h] = bm;
    }
    __syncthreads();
    for (uint32_t n = tid; n < N; n += THREADS)
        if (!(mem[n] <= A.mem_gb * 0.999f)) atomicAnd(&sh_fit, 0u);
    __syncthreads();
    if (sh_fit) {
        for (uint32_t h = tid; h < n_list; h += THREADS) settle(list[h], wish[h]);
    } else {                                                 // some node's memory can bind: job by job, in order
        for (uint32_t n = tid; n < N; n += THREADS) mem[n] = A.mem_gb;
        __syncthreads();
        if (wave == 0) {
            for (uint32_t j0 = 0; j0 < J; j0 += 64u) {       // what 64 jobs have to say is loaded together, a job per lane
                const uint32_t mine = j0 + lane;
                const bool holds = mine < J && np[mine] != 0u;
                unsigned long long todo = __ballot(holds);
                if (!todo) continue;
                const uint32_t my_p = holds ? np[mine] : 0u, my_a = holds ? off[mine] - my_p : 0u, my_g = holds ? gpus_of(mine) : 1u;
                float my_v[RK_MAX_MEM_LEVELS];
#pragma unroll
                for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) {
                    my_v[m] = 0.f;
                    if (m < n_mem && holds) my_v[m] = A.X.best_thr[slot_of(mine, m)];
                }
                uint32_t my_tier = ND_NONE;
                while (todo) {
                    const uint32_t s = (uint32_t)__ffsll((long long)todo) - 1u;
                    todo &= todo - 1ull;
                    const uint32_t P = wave_lane_u32(my_p, s), a = wave_lane_u32(my_a, s), g = wave_lane_u32(my_g, s);
                    float bv = 0.f;
                    uint32_t bm = ND_NONE;
#pragma unroll
                    for (uint32_t m = 0; m < RK_MAX_MEM_LEVELS; ++m) {
                        if (m >= n_mem) break;
                        const float v = rs_lane_f(my_v[m], (int32_t)s);
                        if (!(v > bv)) continue;
                        const float cost = tier_cost(m, g);
                        bool bad = false;
                        for (uint32_t i = lane; i < P; i += 64u)
                            if (!((cost * (float)(parts[a + i] & 0xFFFFu)) / (float)g <= mem[parts[a + i] >> 16])) bad = true;
                        if (__ballot(bad)) continue;
                        bv = v; bm = m;
                    }
                    if (bm != ND_NONE) {
                        const float cost = tier_cost(bm, g);
                        for (uint32_t i = lane; i < P; i += 64u) {
                            const uint32_t n = parts[a + i] >> 16;
                            mem[n] = mem[n] - (cost * (float)(parts[a + i] & 0xFFFFu)) / (float)g;
                        }
                    }
                    if (lane == s) my_tier = bm;
                    asm volatile("" ::: "memory");           // (the next job's lanes read what these ones stored)
                }
                if (holds) settle(mine, my_tier);
            }
        }
    }
    __syncthreads();
    // the records: a job's parts in node order
    {
        const uint32_t all = offsets(A.place_off);
        if (tid == 0) A.place_off[J] = all;
    }
    __syncthreads();
    for (uint32_t h = tid; h < n_list; h += THREADS) {
        const uint32_t j = list[h];
        rk_assign out = {0u, 0u, 0.f, RK_NO_PLAN, 0.f};
        const uint32_t m = np[j] >> 16, P = np[j] & 0xFFFFu, a = off[j] - P;
        if (P) {
            const uint32_t g = gpus_of(j);
            const uint32_t per_gpu = nd_cpl(A, A.st.ci[j]);
            const float cost = tier_cost(m, g);
            out.g = g; out.c = per_gpu * g; out.mem_gb = cost;
            out.plan = A.X.best_plan[slot_of(j, m)];
            out.thr = A.X.best_thr[slot_of(j, m)];
            share[j] = (double)out.thr / (double)A.X.ref_thr[j];
            const uint32_t to = A.place_off[j];
            if (P <= 8u) {                                   // few parts: this thread ranks them
                for (uint32_t i = 0; i < P; ++i) {
                    const uint32_t node = parts[a + i] >> 16, k = parts[a + i] & 0xFFFFu;
                    uint32_t rank = 0;
                    for (uint32_t q = 0; q < P; ++q) rank += (parts[a + q] >> 16) < node ? 1u : 0u;
                    A.entries[to + rank] = rk_place_entry{node, k, per_gpu * k, (cost * (float)k) / (float)g};
                }
            } else {
                wish[atomicAdd(&sh_wide, 1u)] = j;           // (the wishes have been read)
            }
        }
        A.assign[j] = out;
    }
    __syncthreads();
    const uint32_t n_wide = sh_wide;
    for (uint32_t w = wave; w < n_wide; w += WAVES) {         // many parts: a wavefront ranks them
        const uint32_t j = wish[w];
        const uint32_t m = np[j] >> 16, P = np[j] & 0xFFFFu;
        const uint32_t g = gpus_of(j);
        const uint32_t per_gpu = nd_cpl(A, A.st.ci[j]);
        const float cost = tier_cost(m, g);
        const uint32_t a = off[j] - P, to = A.place_off[j];
        for (uint32_t i = lane; i < P; i += 64u) {
            const uint32_t node = parts[a + i] >> 16, k = parts[a + i] & 0xFFFFu;
            uint32_t rank = 0;
            for (uint32_t q = 0; q < P; ++q) rank += (parts[a + q] >> 16) < node ? 1u : 0u;
            A.entries[to + rank] = rk_place_entry{node, k, per_gpu * k, (cost * (float)k) / (float)g};
        }
    }
    // The total, in one order of its float64 additions whatever THREADS is and in whatever order the list was made:
    // ND_THREADS partial sums over the jobs, then over 64 lanes, then one after the other.
    constexpr uint32_t PER = ND_WAVES / WAVES;
    double sum[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        sum[k] = 0.0;
        for (uint32_t j = tid + k * THREADS; j < J; j += ND_THREADS) {
            const uint32_t some = np[j];
            const double x = share[j];                       // (nothing of use where the job has no parts)
            sum[k] += some ? x : 0.0;
        }
    }
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) sum[k] = wave_sum_f64(sum[k]);
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) if (lane == 0) sh_sum[k * WAVES + wave] = sum[k];
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
#pragma unroll
        for (uint32_t w = 0; w < ND_WAVES; ++w) s += sh_sum[w];
        *A.total = (float)s;
    }
}

// Inclusive prefix sum over the wavefront: within rows of 16 lanes by row shifts, then each row's sum is broadcast to
// the rows behind it.  All 64 lanes must be active.
__device__ __forceinline__ uint32_t nd_wave_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);     // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);     // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);     // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);     // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);     // row_bcast:15 into rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);     // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ uint32_t nd_wave_sum(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)nd_wave_scan(v), 63); }

// Words of dynamic LDS that k_nodes_lds needs: the nodes and their copy, the cached slopes, memory, and (LJ) everything
// else a job has.
constexpr uint32_t ND_LDS_JOB_WORDS = 22;
constexpr uint32_t ND_TOUCHED = 64;                        // jobs changed by a step that are remembered in registers (the others in memory)
constexpr uint32_t ND_LDS_SIM_WORDS = 4;                   // ... more per job for ticks of a simulation
// whole 16-byte pieces: copied and searched four words at a time
static inline size_t nd_nodes_words(size_t N, size_t gpus) { return (((3 * N + 3) & ~(size_t)3) + gpus + 3) & ~(size_t)3; }
static inline size_t nd_lds_words(size_t J, size_t N, size_t nodes_words, bool lj, bool sim = false) {
    return 2 * nodes_words + 2 * (J + 1) + N + (J + 31) / 32 + (lj ? ND_LDS_JOB_WORDS * J + 1 : 0) + (sim ? ND_LDS_SIM_WORDS * J : 0);
}

// Where every state of every job is found before the first tick (k_nd_states) the ticks of a simulation need in LDS, beside
// those words, who is on the nodes when a round begins, every job's state and, per job on the nodes, what its memory costs and
// its GPUs; with few nodes also what every job asks of every node (share).
constexpr uint32_t ND_SHARES = 2048;
constexpr uint32_t ND_CHANGED = 48;                        // jobs whose place in the order is found one by one; more: all are sorted
static inline size_t nd_share_words(size_t N, size_t gpus) { return N <= 64 && N * gpus <= ND_SHARES ? N * gpus : 0; }
static inline size_t nd_tab_words(size_t threads, size_t N, size_t gpus, size_t nodes_words) {     // a job per thread
    return nd_lds_words(threads, N, nodes_words, true, true) + 3 * gpus + nd_share_words(N, gpus) + threads / 4 + 8;
}

// The loop with the nodes in LDS.  It is a chain of small decisions, so what bounds it is the latency of one after
// the other.  Here the first wavefront makes a whole step of ScheduleJob by itself, a node per lane on the walk, a
// resident per lane where somebody is shrunk, 64 entries of the nodes' tables at a time where a job's parts are
// looked up: nothing is exchanged between wavefronts within a step, every table it reads and writes is in LDS, and
// what the others do (the look for the next job, the slopes of the jobs that a step changed, the copy of the nodes)
// stands between two barriers after it.  LJ: what the jobs hold and their cached steps are in LDS too.
// What a job gives first in a step was found when its state last changed (nd_keep_give), what a step changed is
// remembered a job per lane, and a shrunk job's other parts are looked for 256 entries at a time: 10,000 jobs on 512 nodes,
// the round from the descriptors: 1,174 -> 1,058 and 2,980 -> 2,620 us on two drawn states.
// SIM (with LJ): a round is a tick of a simulation.  The ticks after it that need no round are closed, then the jobs'
// values are brought up to date for the next round, up to S.rounds of them per launch: nodes, jobs and cached steps stay
// where they are, and only jobs that came, went or thawed have theirs found again.  As launches of their own, replayed as
// a graph, the preparation, the round and the tick took 5, 102 and 9 us with 9 us between them, of which loading the
// nodes and jobs was 5; 406 jobs, 720 ticks: 57.4 -> 46.7 ms, 60 jobs, 100 ticks: 2.59 -> 1.56 ms.
// GPN: the GPUs of a node where they are known (0: not): divisions by it are shifts, loops over a node's residents are unrolled.
template <int THREADS, bool LJ, bool SIM, bool TAB, uint32_t GPN, class KernArgs>
__device__ __forceinline__ void nodes_lds(const KernArgs &K) {
    static_assert((LJ || !SIM) && (SIM || !TAB), "ticks of a simulation have the jobs in LDS; the states are found for them");
    extern __shared__ uint4 sh_raw[];
    constexpr uint32_t WAVES = THREADS / 64;
    __shared__ uint32_t sh_scan[WAVES], sh_take[RK_MAX_CPU_LEVELS], sh_free_c, sh_cpl[RK_MAX_CPU_LEVELS], sh_list;
    __shared__ float sh_rcp[RK_MAX_CPU_LEVELS];             // 1 / a level's CPUs per GPU
    __shared__ unsigned long long sh_pick_key[WAVES];
    __shared__ uint32_t sh_pick_j[WAVES], sh_low[2][WAVES][3];
    __shared__ uint32_t sh_did, sh_touched;                 // what the first wavefront's steps ended in
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
    NdArgs A(K.b, K.X);
    if constexpr (TAB) { A.floor_seg = nullptr; A.floor_c = nullptr; }      // (nobody has a floor in a simulation)
    const uint32_t J = A.n_jobs, N = A.n_nodes, gpn = GPN ? GPN : A.gpn, gpus = N * gpn;
    const uint32_t EMPTY = (J << 16) | 0xFFFFu;              // no resident: a job that has no index, whose slopes are infinite
    const float INF = __int_as_float(0x7F800000);
    uint32_t tick = 0;
    if constexpr (SIM) {
        tick = *K.S.tick;
        if (tick >= K.S.n_ticks) return;                     // (the simulation is over)
    }

    // ---- everything into LDS.  TAB: room for a job per thread, and what the jobs have comes first, so that the addresses
    // are known beforehand (a wavefront that works alone pays for every instruction).  Otherwise what every node has comes before
    // the jobs' words (behind them 900 jobs on 512 nodes took 62.6 ms instead of 62.0).
    const uint32_t JL = TAB ? (uint32_t)THREADS : J;
    uint32_t *at = reinterpret_cast<uint32_t *>(sh_raw);
    auto take = [&](size_t words) { uint32_t *p = at; at += words; return p; };
    uint32_t *nodes = at;
    if constexpr (!TAB) at += 2 * A.nodes_words;
    if constexpr (LJ) A.give = reinterpret_cast<uint4 *>(take(4 * (size_t)JL));
    if constexpr (LJ) { A.udc_c = reinterpret_cast<unsigned long long *>(take(2 * (size_t)JL)); A.okey = reinterpret_cast<unsigned long long *>(take(2 * (size_t)JL)); }
    float *const sh_ds = reinterpret_cast<float *>(take(2 * ((size_t)JL + 1)));
    float *sh_mem = nullptr;
    uint32_t *sh_mark = nullptr;
    if constexpr (!TAB) { sh_mem = reinterpret_cast<float *>(take(N)); sh_mark = take((J + 31u) / 32u); }
    if constexpr (LJ) {
        auto words = [&](auto &p) { p = reinterpret_cast<std::decay_t<decltype(p)>>(take(JL)); };        // a per-job array of words in LDS
        words(A.st.gi); words(A.st.ci); words(A.ug); words(A.uc); words(A.udg); words(A.gain_g); words(A.gain_c);
        words(A.tgt_g); words(A.lvl_g); words(A.lvl_c); words(A.first);
        words(A.touched); words(A.give_c);
    }
    uint32_t *const so = LJ ? take((size_t)JL + 1) : nullptr;
    uint32_t *fin_np = reinterpret_cast<uint32_t *>(sh_ds), *fin_off = fin_np + J, *fin_list = nullptr, *old_state = nullptr;
    if constexpr (SIM) { fin_np = take(JL); fin_off = take(JL); fin_list = take(JL); if (!TAB) old_state = take(JL); }   // (what the next round needs again is not working memory of this one's end)
    uint8_t *state8 = nullptr;
    if constexpr (TAB) {
        state8 = reinterpret_cast<uint8_t *>(take(THREADS / 4));
        at += (4u - (uint32_t)(at - nodes) % 4u) % 4u;       // (whole pieces)
        nodes = take(2 * A.nodes_words);
    }
    uint32_t *const keep = nodes + A.nodes_words;
    if constexpr (TAB) { sh_mem = reinterpret_cast<float *>(take(N)); sh_mark = take((J + 31u) / 32u); }         // a bit per job: changed by the step under way and remembered in memory
    uint32_t *start_res = nullptr, *held_g = nullptr;        // (TAB)
    float *held_cost = nullptr, *share = nullptr;
    A.free_g = nodes; A.free_c = nodes + N; A.cnt = nodes + 2 * N; A.res = nodes + ((3 * N + 3) & ~3u);
    for (uint32_t i = tid; i < (J + 31u) / 32u; i += THREADS) sh_mark[i] = 0u;
    for (uint32_t i = tid; i < A.nodes_words; i += THREADS) nodes[i] = i < N ? gpn : i < 2 * N ? A.cpn : i < 3 * N ? 0u : EMPTY;
    if (tid < A.X.grid.n_cpu) {
        const uint32_t l = A.X.grid.cpu_levels[tid];
        sh_cpl[tid] = l; sh_rcp[tid] = 1.f / (float)l;
    }
    if (tid == 0) sh_list = 0u;
    if constexpr (LJ) {
        for (uint32_t j = tid; j < J; j += THREADS) {        // (all of a job's loads before the first store)
            const NdBody &b = K.b;
            const int32_t gi = b.st.gi[j], tgt = b.tgt_g[j];
            const uint32_t ci = b.st.ci[j], udg = b.udg[j], lg = b.lvl_g[j], lc = b.lvl_c[j], first = b.first[j], o = K.X.tb.seg_off[j];
            const float ug = b.ug[j], uc = b.uc[j], gg = b.gain_g[j], gc = b.gain_c[j];
            const unsigned long long dc = b.udc_c[j];
            const uint4 *const gives = reinterpret_cast<const uint4 *>(b.gives + j);
            const uint4 g0 = gi >= 0 ? gives[0] : uint4{0u, 0u, 0u, 0u};
            const uint32_t g1 = gi >= 0 ? gives[1].x : 0u;
            A.give[j] = uint4{g0.x, g0.y, (uint32_t)(int32_t)(int16_t)(g0.z & 0xFFFFu), g0.w}; A.give_c[j] = __uint_as_float(g1);
            A.st.gi[j] = gi; A.st.ci[j] = ci; A.ug[j] = ug; A.uc[j] = uc; A.udg[j] = udg; A.gain_g[j] = gg; A.gain_c[j] = gc;
            A.tgt_g[j] = tgt; A.lvl_g[j] = lg; A.lvl_c[j] = lc; A.first[j] = first; A.udc_c[j] = dc; so[j] = o;
        }
        if (tid == 0) so[J] = A.X.tb.seg_off[J];
        A.seg_off = so;
    }
    if constexpr (!SIM) fin_list = A.res;
    if constexpr (SIM && !TAB) for (uint32_t j = tid; j < J; j += THREADS) old_state[j] = A.state[j];
    if constexpr (TAB) {
        start_res = take(gpus); held_cost = reinterpret_cast<float *>(take(gpus)); held_g = take(gpus);
        if (K.shares) share = reinterpret_cast<float *>(take((size_t)N * gpus));
        for (uint32_t j = tid; j < J; j += THREADS) state8[j] = A.state[j];
        A.state = state8;
        A.lvl_g = A.st.ci;                                   // (a GPU step stays on the level)
    }
    uint32_t bad = 0, any_first = 0;
    for (uint32_t j = tid; j < J; j += THREADS) {
        sh_ds[j] = A.ds_g[j]; sh_ds[JL + 1 + j] = A.ds_c[j];
        bad |= A.first[j] & 2u; any_first |= A.first[j] & 1u;
    }
    A.ds_g = sh_ds; A.ds_c = sh_ds + JL + 1;
    if (tid == 0) sh_ds[J] = sh_ds[JL + 1 + J] = INF;
    __syncthreads();
    // the jobs' parts are booked (k_nd_prepare has checked them): a job per thread, or a wavefront where a job has many.
    // These are listed where the copy of the nodes will be; parts that fit the nodes are three GPUs or more a job, so a
    // list that is too long says that the nodes are booked beyond what they have.
    auto book = [&](uint32_t j, const rk_place_entry &e) {
        const uint32_t slot = atomicAdd(&A.cnt[e.node], 1u);
        if (slot < gpn) A.res[e.node * gpn + slot] = (j << 16) | e.g;
        atomicSub(&A.free_g[e.node], e.g);                   // (wraps below zero when the node holds more than it has)
        atomicSub(&A.free_c[e.node], e.c);
    };
    for (uint32_t j0 = tid; j0 < J; j0 += 4 * THREADS) {     // (four jobs' offsets, then four parts, in flight)
        uint32_t a[4], b[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t j = j0 + k * THREADS;
            const bool holds = j < J && A.st.gi[j] >= 0 && !(A.first[j] & 2u);
            a[k] = holds ? A.prev_off[j] : 0u;
            b[k] = holds ? A.prev_off[j + 1] : 0u;
        }
        rk_place_entry e[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) if (a[k] < b[k] && b[k] - a[k] <= 2u) e[k] = A.prev_entries[a[k]];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t j = j0 + k * THREADS;
            if (b[k] - a[k] > 2u) {
                const uint32_t to = atomicAdd(&sh_list, 1u);
                if (to < A.nodes_words) keep[to] = j;
                continue;
            }
            if (a[k] < b[k]) book(j, e[k]);
            if (a[k] + 1u < b[k]) book(j, A.prev_entries[a[k] + 1u]);
        }
    }
    __syncthreads();
    const uint32_t listed = sh_list;
    if (listed > A.nodes_words) { nd_refuse<THREADS>(A); return; }
    for (uint32_t i = wave; i < listed; i += WAVES) {
        const uint32_t j = keep[i];
        const uint32_t a = A.prev_off[j], b = A.prev_off[j + 1];
        for (uint32_t x = a + lane; x < b; x += 64u) book(j, A.prev_entries[x]);
    }
    __syncthreads();
    for (uint32_t n = tid; n < N; n += THREADS)
        if (A.cnt[n] > gpn || A.free_g[n] > gpn || A.free_c[n] > A.cpn) bad |= 1u;
    if (__syncthreads_or((int)bad)) { nd_refuse<THREADS>(A); return; }
    const bool with_first = __syncthreads_or((int)any_first) != 0;
    auto copy_nodes = [&](uint32_t *to, const uint32_t *from) {          // (nodes_words is a multiple of four)
        const uint4 *src = reinterpret_cast<const uint4 *>(from);
        uint4 *dst = reinterpret_cast<uint4 *>(to);
        for (uint32_t i = tid; i < A.nodes_words / 4u; i += THREADS) dst[i] = src[i];
    };
    copy_nodes(keep, nodes);
    __syncthreads();

    // ---- the first wavefront's part: a step of ScheduleJob.  Values without a lane are the same in all lanes.
    uint32_t moves = 0, full = 0, shrinks = 0, undone = 0;   // (the first wavefront's counts)
    uint32_t touched = 0;                                    // jobs this step has changed so far
    float lost = 0.f;
    bool dirty = false;                                      // the nodes are not as they were when the step began
    // job v as it was before this step changed it for the first time: a job per lane, then in memory (all lanes call)
    uint32_t was_j = ND_NONE, was = 0;                       // the job; its amount << 16 | level
    float was_g = 0.f, was_c = 0.f;                          // its slopes
    auto remember = [&](uint32_t v, int32_t gi, uint32_t ci) {
        if (touched < ND_TOUCHED) {
            if (lane == touched) { was_j = v; was = ((uint32_t)gi << 16) | ci; was_g = A.ds_g[v]; was_c = A.ds_c[v]; }
        } else if (lane == 0) {
            K.b.keep_gi[touched] = gi; K.b.keep_ci[touched] = ci;
            K.b.keep_ds[2 * touched] = A.ds_g[v]; K.b.keep_ds[2 * touched + 1] = A.ds_c[v];
            sh_mark[v >> 5] |= 1u << (v & 31u);
        }
        if (lane == 0) A.touched[touched] = v;
        touched += 1u;
    };
    auto remembered = [&](uint32_t v) {
        return __ballot(was_j == v) != 0ull ||
               (touched > ND_TOUCHED && (((uint32_t)__builtin_amdgcn_readfirstlane((int)sh_mark[v >> 5]) >> (v & 31u)) & 1u));
    };
    auto begin_jobs = [&]() { touched = 0u; lost = 0.f; was_j = ND_NONE; };
    // the step is over: when it was not committed the jobs are as they were
    auto end_jobs = [&](bool committed) {
        rs_wave_order();
        if (touched > ND_TOUCHED) {
            for (uint32_t i = ND_TOUCHED + lane; i < touched; i += 64u) {
                const uint32_t v = A.touched[i];
                atomicAnd(&sh_mark[v >> 5], ~(1u << (v & 31u)));
                if (committed) continue;
                A.st.gi[v] = K.b.keep_gi[i]; A.st.ci[v] = K.b.keep_ci[i];
                A.ds_g[v] = K.b.keep_ds[2 * i]; A.ds_c[v] = K.b.keep_ds[2 * i + 1];
            }
            rs_wave_order();
        }
        if (committed) return;
        if (was_j != ND_NONE) {
            A.st.gi[was_j] = (int32_t)(was >> 16); A.st.ci[was_j] = was & 0xFFFFu;
            A.ds_g[was_j] = was_g; A.ds_c[was_j] = was_c;
        }
        undone += touched ? 1u : 0u;
    };
    // job v's entries of the nodes' tables, in ascending order of the nodes (DOWN: descending), until what(index of the lane's
    // entry, the entry, the lanes that have one of v's) says no.  1,024 entries are looked through at a time, four loads of
    // a lane in flight; 256 of them are handed on together where a lane's four are one node's, of which v has one at most.
    const uint4 *const res4 = reinterpret_cast<const uint4 *>(A.res);
    const uint32_t n4 = (gpus + 3u) / 4u;
    auto for_parts = [&](uint32_t v, auto down, auto what) {
        constexpr bool DOWN = decltype(down)::value;
        const uint32_t blocks = (n4 + 255u) / 256u;
        for (uint32_t x = 0; x < blocks; ++x) {
            const uint32_t blk = DOWN ? blocks - 1u - x : x;
            uint32_t with = 0;                               // which of the four groups of 256 entries hold some of the job
            {
                uint4 q[4];
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u) {
                    const uint32_t at4 = blk * 256u + u * 64u + lane;
                    q[u] = at4 < n4 ? res4[at4] : uint4{EMPTY, EMPTY, EMPTY, EMPTY};
                }
#pragma unroll
                for (uint32_t u = 0; u < 4; ++u)
                    if (__ballot((q[u].x >> 16) == v || (q[u].y >> 16) == v || (q[u].z >> 16) == v || (q[u].w >> 16) == v)) with |= 1u << u;
            }
            while (with) {
                const uint32_t u = DOWN ? 31u - (uint32_t)__clz((int)with) : (uint32_t)__ffs((int)with) - 1u;
                with &= ~(1u << u);
                if ((gpn & 3u) == 0u) {
                    const uint32_t at4 = blk * 256u + u * 64u + lane;
                    const uint4 q = at4 < n4 ? res4[at4] : uint4{EMPTY, EMPTY, EMPTY, EMPTY};
                    uint32_t word = q.x, c = 0u;
                    if ((q.y >> 16) == v) { word = q.y; c = 1u; }
                    if ((q.z >> 16) == v) { word = q.z; c = 2u; }
                    if ((q.w >> 16) == v) { word = q.w; c = 3u; }
                    if (!what(4u * at4 + c, word, __ballot((word >> 16) == v))) return;
                    continue;
                }
#pragma unroll 1
                for (uint32_t y = 0; y < 4; ++y) {           // ... and where
                    const uint32_t b = 4u * (blk * 256u + u * 64u) + 64u * (DOWN ? 3u - y : y);
                    const uint32_t word = b + lane < gpus ? A.res[b + lane] : EMPTY;
                    const unsigned long long m = __ballot((word >> 16) == v);
                    if (m && !what(b + lane, word, m)) return;
                }
            }
        }
    };
    auto one = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    auto one_i = [](int32_t x) { return __builtin_amdgcn_readfirstlane(x); };
    // a / b from 1 / b for a < 2^21: (a + 1/2) / b is further from a whole number than the product's error
    auto over = [&](uint32_t a, float rcp) { return (uint32_t)(((float)a + 0.5f) * rcp); };
    const float rcp_gpn = 1.f / (float)gpn;
    auto node_of = [&](uint32_t i) { if constexpr (GPN != 0u) return i / GPN; else return over(i, rcp_gpn); };
    enum : uint32_t { DID_NOTHING = 0, DID_GPUS = 1, DID_CPUS = 2, DID_UNDO = 4 };
    // A GPU step of job j: DID_GPUS when it is committed, else DID_NOTHING (jobs put back; the nodes are `dirty` or as before)
    auto gpu_step = [&](uint32_t j) -> uint32_t {
        dirty = false;
        const RsStep st = nd_cached_step(A, j, 0);
        if (!st.any) return DID_NOTHING;
        begin_jobs();
        const int32_t fl = rs_fl_s(A, j), gi_j = A.st.gi[j];
        const uint32_t ci_j = TAB ? st.lvl : A.st.ci[j];
        const bool below_min = fl >= 0 && gi_j < fl;
        const uint32_t per_gpu = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh_cpl[st.lvl]);
        const float rcp = sh_rcp[st.lvl];
        uint32_t lack = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)st.dg);
        bool ok = true;
        if (gi_j >= 0 && st.lvl != ci_j) {                   // its parts go to the step's level: their CPUs must be free
            const uint32_t more = per_gpu - sh_cpl[ci_j];
            dirty = true;
            for_parts(j, std::false_type{}, [&](uint32_t i, uint32_t word, unsigned long long m) {
                bool short_of = false;
                if ((m >> lane) & 1ull) {
                    const uint32_t n = node_of(i), have = A.free_c[n];
                    const unsigned long long need = (unsigned long long)more * (word & 0xFFFFu);
                    if (have < need) short_of = true;
                    else A.free_c[n] = have - (uint32_t)need;
                }
                if (__ballot(short_of)) ok = false;
                return ok;
            });
            rs_wave_order();
        }
        const float own = A.ds_g[j];                         // j gives nothing to itself
        rs_wave_order();
        if (lane == 0) A.ds_g[j] = INF;
        rs_wave_order();
        uint32_t n0 = 0;
        while (ok && lack > 0 && n0 < N) {                   // the walk over the nodes, a node per lane
            const uint32_t n = n0 + lane;
            const bool in = n < N;
            uint32_t offer = 0, c = 0, fg = 0, fc = 0;
            float low = INF;                                 // the lowest slope among the others on the node (j's own is infinite now)
            const uint32_t base_n = n * gpn;
            if (in) {
                fg = A.free_g[n]; fc = A.free_c[n]; c = A.cnt[n];
                if ((gpn & 7u) == 0u) {                      // eight residents at a time, all their loads unconditional
                    for (uint32_t i = 0; i < gpn; i += 8u) {
                        const uint4 q = res4[(base_n + i) / 4u], r = res4[(base_n + i) / 4u + 1u];
                        const float s0 = A.ds_g[q.x >> 16], s1 = A.ds_g[q.y >> 16], s2 = A.ds_g[q.z >> 16], s3 = A.ds_g[q.w >> 16];
                        const float s4 = A.ds_g[r.x >> 16], s5 = A.ds_g[r.y >> 16], s6 = A.ds_g[r.z >> 16], s7 = A.ds_g[r.w >> 16];
                        low = fminf(fminf(fminf(low, fminf(s0, s1)), fminf(s2, s3)), fminf(fminf(s4, s5), fminf(s6, s7)));
                    }
                } else {
                    for (uint32_t i = 0; i < c; ++i) low = fminf(low, A.ds_g[A.res[base_n + i] >> 16]);
                }
                const uint32_t by_cpu = over(fc, rcp);
                offer = fg < by_cpu ? fg : by_cpu;
            }
            const bool ask = low < INF && (below_min || st.slope > low);     // somebody here may be shrunk
            const uint32_t upto = nd_wave_scan(offer), before = upto - offer;
            const unsigned long long done_m = __ballot(in && upto >= lack), ask_m = __ballot(ask && upto < lack);
            const uint32_t done_t = done_m ? (uint32_t)__ffsll((long long)done_m) - 1u : 64u;
            const uint32_t ask_t = ask_m ? (uint32_t)__ffsll((long long)ask_m) - 1u : 64u;
            const uint32_t last = done_t < ask_t ? done_t : ask_t;           // the nodes up to here give what they offer
            if (__ballot(lane <= last && offer > 0u)) dirty = true;
            if (lane <= last && offer) {
                const uint32_t k = offer < lack - before ? offer : lack - before;
                A.free_g[n] = fg - k; A.free_c[n] = fc - k * per_gpu;
                int at = -1;                             // (a newcomer is on no node that the walk comes to)
                if (gi_j >= 0) {
                    if ((gpn & 7u) == 0u) {
                        for (uint32_t i = 0; i < gpn; i += 8u) {
                            const uint4 q = res4[(base_n + i) / 4u], r = res4[(base_n + i) / 4u + 1u];
                            const uint32_t w[8] = {q.x, q.y, q.z, q.w, r.x, r.y, r.z, r.w};
#pragma unroll
                            for (uint32_t x = 0; x < 8; ++x) at = (w[x] >> 16) == j ? (int)(i + x) : at;
                        }
                    } else {
                        at = nd_find(A, n, j);
                    }
                }
                if (at >= 0) A.res[base_n + (uint32_t)at] += k;
                else if (c < gpn) { A.res[base_n + c] = (j << 16) | k; A.cnt[n] = c + 1u; }
            }
            const uint32_t got = wave_lane_u32(upto, last < 64u ? last : 63u);
            lack -= got < lack ? got : lack;
            rs_wave_order();
            if (ask_t >= done_t) { n0 += 64u; continue; }    // (nobody to ask; when the step has its GPUs the walk ends)
            const uint32_t f = n0 + ask_t, base = f * gpn;
            n0 = f + 1u;
            while (lack > 0) {                               // node f: a resident per lane (a node has at most 64 here)
                const uint32_t cf = (uint32_t)__builtin_amdgcn_readfirstlane((int)A.cnt[f]);
                const uint32_t free_g = A.free_g[f], free_c = A.free_c[f];
                const uint32_t word = lane < gpn ? A.res[base + lane] : EMPTY;
                const uint32_t rv = word >> 16;
                const float sl = A.ds_g[rv];
                // the lowest slope (as a word that orders like it), then the lowest job that has it
                uint32_t key = sl < INF ? rs_ordered(sl) : ND_NONE, least, who;
                if (gpn <= 16u) {
                    least = (uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(key), 0);
                    who = (uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(key == least ? rv : ND_NONE), 0);
                } else {
                    least = wave_min_u32_rows(key);
                    who = wave_min_u32_rows(key == least ? rv : ND_NONE);
                }
                if (least == ND_NONE || !(below_min || st.slope > rs_unordered(least))) break;
                // what it gives: kept, unless this step has changed it already
                const bool again = remembered(who);
                int32_t gi0, gi1;
                uint32_t ci0, dg;
                float loss, ds_g1, ds_c1;
                if (!again) {
                    if constexpr (LJ) {
                        const uint4 w = A.give[who];
                        ds_c1 = A.give_c[who];
                        gi0 = one_i(A.st.gi[who]); ci0 = one(A.st.ci[who]);
                        dg = one(w.x); loss = __uint_as_float(one(w.y)); gi1 = one_i((int32_t)w.z); ds_g1 = __uint_as_float(w.w);
                    } else {
                        const uint4 *const from = reinterpret_cast<const uint4 *>(A.gives + who);
                        const uint4 w = from[0], x = from[1];
                        const uint32_t gis = one(w.z);
                        dg = one(w.x); loss = __uint_as_float(one(w.y)); gi0 = (int32_t)(gis >> 16); gi1 = (int32_t)(int16_t)(gis & 0xFFFFu);
                        ds_g1 = __uint_as_float(w.w); ds_c1 = __uint_as_float(x.x); ci0 = one(x.z) & 0xFFu;
                    }
                    remember(who, gi0, ci0);
                } else {
                    gi0 = one_i(A.st.gi[who]); ci0 = one(A.st.ci[who]);
                    if constexpr (TAB) {
                        const uint32_t w = K.states.words[nd_state_at(K.states, who, A.X.grid.n_cpu, gi0, ci0) * ND_STATE_WORDS + (lane & 15u)];
                        dg = wave_lane_u32(w, ND_GIVES); loss = __uint_as_float(wave_lane_u32(w, ND_LOSS)); gi1 = (int32_t)wave_lane_u32(w, ND_TO);
                        ds_g1 = __uint_as_float(wave_lane_u32(w, ND_DS_G1)); ds_c1 = __uint_as_float(wave_lane_u32(w, ND_DS_C1));
                    } else {
                        const uint32_t so = one(A.seg_off[who]), ns = one(A.seg_off[who + 1]) - so;
                        const RsShrunk sk = rs_shrink_wave(A, who, so, ns, 0, gi0, ci0, lane);
                        dg = one((uint32_t)sk.gv.dg); loss = sk.gv.loss; gi1 = sk.gi; ds_g1 = sk.ds_g; ds_c1 = sk.ds_c;
                    }
                }
                const uint32_t slot = (uint32_t)__ffsll((long long)__ballot(lane < cf && rv == who)) - 1u;
                const uint32_t here_has = wave_lane_u32(word, slot) & 0xFFFFu, per_v = sh_cpl[ci0];
                const uint32_t here = dg < here_has ? dg : here_has;
                dirty = true;
                shrinks += 1u;
                lost = lost + loss;
                // the node afterwards, from what the lanes hold: who gives `here` of its GPUs, j takes what it can
                const uint32_t fg = free_g + here, fc = free_c + here * per_v;
                const uint32_t by_cpu = over(fc, rcp), offer2 = fg < by_cpu ? fg : by_cpu;
                const uint32_t t = offer2 < lack ? offer2 : lack;
                const bool goes = here == here_has;          // it leaves the node: the last resident takes its entry
                const uint32_t c1 = cf - (goes ? 1u : 0u);
                const uint32_t last_word = wave_lane_u32(word, cf - 1u);
                uint32_t mine = word;
                if (lane == slot) mine = goes ? last_word : word - here;
                if (lane >= c1) mine = EMPTY;
                const unsigned long long j_m = __ballot(lane < c1 && (mine >> 16) == j);
                uint32_t c2 = c1;
                if (t) {
                    if (j_m) { if ((j_m >> lane) & 1ull) mine += t; }
                    else if (c1 < gpn) { if (lane == c1) mine = (j << 16) | t; c2 = c1 + 1u; }
                }
                if (lane < gpn) A.res[base + lane] = mine;
                if (lane == 0) {
                    A.free_g[f] = fg - t; A.free_c[f] = fc - t * per_gpu; A.cnt[f] = c2;
                    A.st.gi[who] = gi1; A.st.ci[who] = gi1 < 0 ? 0u : ci0;
                    A.ds_g[who] = ds_g1; A.ds_c[who] = ds_c1;
                }
                lack -= t;
                uint32_t rest = dg - here;
                rs_wave_order();
                if (rest > 0)                                // the rest from its other parts, the last one first
                    for_parts(who, std::true_type{}, [&](uint32_t i, uint32_t w, unsigned long long m) {
                        const uint32_t k = (m >> lane) & 1ull ? w & 0xFFFFu : 0u, upto = nd_wave_scan(k), all = wave_lane_u32(upto, 63u);
                        const uint32_t behind = all - upto;  // what the entries after this one have
                        if (k && behind < rest) {
                            const uint32_t give = k < rest - behind ? k : rest - behind, n1 = node_of(i);
                            A.free_g[n1] += give; A.free_c[n1] += give * per_v;
                            if (give < k) A.res[i] = w - give;
                            else {                           // (a job is on a node once: no other lane's node, no entry still to come)
                                const uint32_t l = A.cnt[n1] - 1u;
                                A.res[i] = A.res[n1 * gpn + l];
                                A.res[n1 * gpn + l] = EMPTY;
                                A.cnt[n1] = l;
                            }
                        }
                        rs_wave_order();
                        rest -= all < rest ? all : rest;
                        return rest > 0;
                    });
                rs_wave_order();
            }
        }
        if (lane == 0) A.ds_g[j] = own;
        const bool committed = ok && lack == 0u && (below_min || st.gain > lost);
        end_jobs(committed);
        if (!committed) return DID_NOTHING;
        if (lane == 0) { A.st.gi[j] = st.tgt; A.st.ci[j] = st.lvl; }
        moves += 1u;
        return DID_GPUS;
    };
    // A CPU step of job j likewise, on every node the job is on (DID_CPUS)
    auto cpu_step = [&](uint32_t j) -> uint32_t {
        dirty = false;
        const RsStep st = nd_cached_step(A, j, 1);
        if (!st.any) return DID_NOTHING;
        begin_jobs();
        const uint32_t more = sh_cpl[st.lvl] - sh_cpl[A.st.ci[j]];
        bool ok = true;
        for_parts(j, std::false_type{}, [&](uint32_t i, uint32_t word, unsigned long long m) {
            while (m) {
                const uint32_t s = (uint32_t)__ffsll((long long)m) - 1u, n = node_of(wave_lane_u32(i, s));
                m &= m - 1ull;
                const unsigned long long need = (unsigned long long)more * (wave_lane_u32(word, s) & 0xFFFFu);
                for (;;) {
                    const uint32_t free_here = A.free_c[n];
                    if (free_here >= need) {
                        if (lane == 0) A.free_c[n] = free_here - (uint32_t)need;
                        dirty = true;
                        rs_wave_order();
                        break;
                    }
                    uint32_t who;
                    const float low = nd_lowest_on_wave(A, n, j, A.ds_c, who, lane);
                    if (who == ND_NONE || !(st.slope > low)) { ok = false; return false; }
                    const int32_t gi0 = __builtin_amdgcn_readfirstlane(A.st.gi[who]);
                    const uint32_t ci0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)A.st.ci[who]);
                    const uint32_t so = A.seg_off[who], ns = A.seg_off[who + 1] - so;
                    const RsShrunk sk = rs_shrink_wave(A, who, so, ns, 1, gi0, ci0, lane);
                    if (!remembered(who)) remember(who, gi0, ci0);
                    dirty = true;
                    shrinks += 1u;
                    lost = lost + sk.gv.loss;
                    if (lane == 0) {
                        A.st.ci[who] = sk.ci;
                        A.ds_g[who] = sk.ds_g; A.ds_c[who] = sk.ds_c;
                    }
                    const uint32_t less = sh_cpl[ci0] - sh_cpl[ci0 - 1u];
                    for_parts(who, std::false_type{}, [&](uint32_t i2, uint32_t w2, unsigned long long m2) {     // it gives a level on all its nodes
                        if ((m2 >> lane) & 1ull) A.free_c[node_of(i2)] += less * (w2 & 0xFFFFu);
                        return true;
                    });
                    rs_wave_order();
                }
            }
            return true;
        });
        const bool committed = ok && st.gain > lost;
        end_jobs(committed);
        if (!committed) return DID_NOTHING;
        if (lane == 0) A.st.ci[j] = st.lvl;
        moves += 1u;
        return DID_CPUS;
    };

    // ScheduleJob(j): the first wavefront steps, then all refresh what a committed step changed, or put the nodes back
    auto schedule_job = [&](uint32_t j) {
        bool gpus_done = false, done = false;                // (the first wavefront's)
        for (;;) {
            if (wave == 0) {
                uint32_t did = DID_NOTHING;
                if (!gpus_done) {
                    did = gpu_step(j);
                    if (did == DID_NOTHING) {
                        gpus_done = true;
                        if (dirty) {                         // (the CPU steps' turn comes when the nodes are back)
                            did = DID_UNDO;
                            done = !(A.uc[j] > 0.f);
                        }
                    }
                }
                if (did == DID_NOTHING) {
                    did = cpu_step(j);
                    if (did == DID_NOTHING) { done = true; if (dirty) did = DID_UNDO; }
                }
                if (lane == 0) { sh_did = did | (done ? 8u : 0u); sh_touched = touched; }
            }
            __syncthreads();
            const uint32_t did = sh_did, n_touched = sh_touched;
            if (did & (DID_GPUS | DID_CPUS)) {
                for (uint32_t i = wave; i < 2u * (n_touched + 1u); i += WAVES) { // two wavefronts per job whose state changed: GPUs, CPUs
                    const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)(i < 2u * n_touched ? A.touched[i >> 1] : j));
                    nd_refresh_wave(A, v, __builtin_amdgcn_readfirstlane(A.st.gi[v]), (uint32_t)__builtin_amdgcn_readfirstlane((int)A.st.ci[v]), lane,
                                    (i & 1u) == 0u, (i & 1u) != 0u);
                }
                copy_nodes(keep, nodes);
            } else if (did & DID_UNDO) {
                copy_nodes(nodes, keep);
            }
            __syncthreads();
            if (did & 8u) break;
        }
    };

    auto round = [&]() {
    // ---- privileged jobs (below their floor) come first, in job order: their list (tmp_off serves as the list)
    uint32_t n_first = 0;
    if (with_first) {
        for (uint32_t base = 0; base < J; base += THREADS) {
            const uint32_t j = base + tid;
            const bool is = j < J && A.first[j] != 0u;
            uint32_t all;
            const uint32_t to = nd_block_scan<THREADS>(is ? 1u : 0u, all, sh_scan);
            if (is) A.tmp_off[n_first + to] = j;
            n_first += all;
        }
        __syncthreads();
    }
    // ---- then the others, in an order that is fixed when these are through (by slopes; the cached ones are current); jobs
    // with nothing to do are passed over (k_reschedule_nodes says when that is)
    unsigned long long last_key = ~0ull, my_key = 0ull;      // my_*: the first job of this thread's to serve
    uint32_t last_j = 0u, my_j = ND_NONE;
    bool fresh = true;                                       // a step was committed since the last look (or this is the first)
    RsMin low[2];                                            // the two lowest slopes per resource, and whose the lowest is
    low[0] = low[1] = RsMin{INF, INF, ND_NONE};
    bool others = false;
    auto look = [&]() {                                      // leaves the job to serve in last_j
        if (!others) {
            for (uint32_t j = tid; j < J; j += THREADS)      // 0: not in the list
                A.okey[j] = rs_part(A, j) && !A.first[j] ? ((unsigned long long)rs_ordered(A.ug[j]) << 32) | rs_ordered(A.uc[j]) : 0ull;
            others = true;
        }
        if (fresh) {
            // what the nodes can give at every CPU level, and all free CPUs: a wavefront per sum
            for (uint32_t l = wave; l <= A.X.grid.n_cpu; l += WAVES) {
                const bool cpus = l == A.X.grid.n_cpu;
                const float rcp = cpus ? 1.f : sh_rcp[l];
                uint32_t t = 0;
                for (uint32_t n = lane; n < N; n += 64u) {
                    const uint32_t by_cpu = over(A.free_c[n], rcp), fg = A.free_g[n];
                    t += cpus || by_cpu < fg ? by_cpu : fg;
                }
                t = nd_wave_sum(t);
                if (lane == 0) { if (cpus) sh_free_c = t; else sh_take[l] = t; }
            }
            // the two lowest slopes (as words that order like them) and the job of the lowest: every thread's, every
            // wavefront's, then all wavefronts' by everybody
            float a[2] = {INF, INF}, b[2] = {INF, INF};
            uint32_t ia[2] = {ND_NONE, ND_NONE};
            for (uint32_t v = tid; v < J; v += THREADS)
#pragma unroll
                for (uint32_t r = 0; r < 2; ++r) {           // ascending jobs: the lower one stays among equals
                    const float y = sh_ds[r * (JL + 1) + v];
                    if (y < a[r]) { b[r] = a[r]; a[r] = y; ia[r] = v; }
                    else if (y < b[r]) b[r] = y;
                }
#pragma unroll
            for (uint32_t r = 0; r < 2; ++r) {
                const uint32_t mine = rs_ordered(a[r]), least = wave_min_u32_rows(mine);
                const uint32_t whose = wave_min_u32_rows(mine == least ? ia[r] : ND_NONE);
                const uint32_t second = wave_min_u32_rows(ia[r] != ND_NONE && ia[r] == whose ? rs_ordered(b[r]) : mine);
                if (lane == 0) { sh_low[r][wave][0] = least; sh_low[r][wave][1] = whose; sh_low[r][wave][2] = second; }
            }
            rs_lds_barrier();
#pragma unroll
            for (uint32_t r = 0; r < 2; ++r) {
                const uint32_t w = lane < WAVES ? lane : 0u;
                const uint32_t mine = sh_low[r][w][0], i = sh_low[r][w][1], s2 = sh_low[r][w][2];
                const uint32_t least = (uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(mine), 0);
                low[r].i1 = (uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(mine == least ? i : ND_NONE), 0);
                low[r].m1 = rs_unordered(least);
                low[r].m2 = rs_unordered((uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(i == low[r].i1 ? s2 : mine), 0));
            }
        }
        // the job's place in the order when it is still to be served and finds something to do, else 0
        const uint32_t free_c = sh_free_c;
        auto place_of = [&](uint32_t j, unsigned long long key, float ug, float uc, uint32_t dg, uint32_t lv, unsigned long long dc) {
            const float lowest_g = j == low[0].i1 ? low[0].m2 : low[0].m1, lowest_c = j == low[1].i1 ? low[1].m2 : low[1].m1;
            const bool gpu_idle = !(ug > 0.f) || (sh_take[lv] < dg && !(ug > lowest_g));
            const bool cpu_idle = !(uc > 0.f) || (free_c < dc && !(uc > lowest_c));
            return (gpu_idle && cpu_idle) || key > last_key || (key == last_key && j <= last_j) ? 0ull : key;
        };
        if (fresh) {
            constexpr uint32_t UN = 4;                       // jobs whose values are in flight
            my_key = 0ull; my_j = ND_NONE;
            for (uint32_t j0 = tid; j0 < J; j0 += UN * THREADS) {
                unsigned long long key[UN], dc[UN];
                float ug[UN], uc[UN];
                uint32_t dg[UN], lv[UN];
#pragma unroll
                for (uint32_t k = 0; k < UN; ++k) {
                    const uint32_t j = j0 + k * THREADS;
                    const bool in = j < J;
                    key[k] = in ? A.okey[j] : 0ull;
                    ug[k] = in ? A.ug[j] : 0.f; uc[k] = in ? A.uc[j] : 0.f;
                    dg[k] = in ? A.udg[j] : 0u; lv[k] = in ? A.st.ci[j] : 0u; dc[k] = in ? A.udc_c[j] : 0ull;
                }
#pragma unroll
                for (uint32_t k = 0; k < UN; ++k) {
                    const uint32_t j = j0 + k * THREADS;
                    const unsigned long long place = place_of(j, key[k], ug[k], uc[k], dg[k], lv[k], dc[k]);
                    if (place > my_key) { my_key = place; my_j = j; }        // (ascending jobs)
                }
            }
        } else if (wave == (last_j % THREADS) / 64u) {
            // nothing was committed: every thread's first job stays it, but the one's that has been served.  Its wavefront
            // looks through that thread's jobs, a job per lane (at most 48)
            const uint32_t owner = last_j % THREADS, j = owner + lane * THREADS;
            unsigned long long place = 0ull;
            if (j < J) place = place_of(j, A.okey[j], A.ug[j], A.uc[j], A.udg[j], A.st.ci[j], A.udc_c[j]);
            const uint32_t hi = (uint32_t)(place >> 32), lo = (uint32_t)place;
            const uint32_t top_hi = wave_max_u32_rows(hi), top_lo = wave_max_u32_rows(hi == top_hi ? lo : 0u);
            const unsigned long long top = ((unsigned long long)top_hi << 32) | top_lo;
            const uint32_t first = wave_min_u32_rows(top && place == top ? j : ND_NONE);
            if (tid == owner) { my_key = top; my_j = first; }
        }
        {                                                    // the first of the threads' jobs in the order
            const uint32_t hi = (uint32_t)(my_key >> 32), lo = (uint32_t)my_key;
            const uint32_t top_hi = wave_max_u32_rows(hi), top_lo = wave_max_u32_rows(hi == top_hi ? lo : 0u);
            const uint32_t first = wave_min_u32_rows(hi == top_hi && lo == top_lo ? my_j : ND_NONE);
            if (lane == 0) { sh_pick_key[wave] = ((unsigned long long)top_hi << 32) | top_lo; sh_pick_j[wave] = first; }
            rs_lds_barrier();
            const uint32_t w = lane < WAVES ? lane : 0u;     // (at most 16 wavefronts: a row of lanes)
            const unsigned long long k2 = sh_pick_key[w];
            const uint32_t j2 = sh_pick_j[w], hi2 = (uint32_t)(k2 >> 32), lo2 = (uint32_t)k2;
            const uint32_t best_hi = 0xFFFFFFFFu - (uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(0xFFFFFFFFu - hi2), 0);
            const uint32_t best_lo = 0xFFFFFFFFu - (uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(hi2 == best_hi ? 0xFFFFFFFFu - lo2 : 0xFFFFFFFFu), 0);
            last_key = ((unsigned long long)best_hi << 32) | best_lo;
            last_j = (uint32_t)__builtin_amdgcn_readlane((int)row_min_u32(k2 == last_key ? j2 : ND_NONE), 0);
        }
    };
    for (uint32_t k_first = 0;;) {                           // one job per turn; ScheduleJob appears once in the code, which
        uint32_t j;                                          // the instruction cache then holds
        const bool is_first = k_first < n_first;
        if (is_first) {
            j = one(A.tmp_off[k_first++]);
        } else {
            look();
            if (last_j == ND_NONE) break;
            full += 1u;
            j = last_j;
        }
        const uint32_t before = moves;
        schedule_job(j);
        fresh = __syncthreads_or(is_first || (wave == 0 && moves != before)) != 0;
    }
    };
    if constexpr (TAB) {

        // Ticks of a simulation whose jobs' states are all known: the first wavefront makes a round by itself, without barriers,
        // since what a committed step changes of a job is a look into the table, and who comes next is found in a list that
        // is in order before the round.  A job per thread has in registers what the ticks need of it.  What bounds it is how
        // many instructions that one wavefront needs, 6.7 cycles each: addresses that are known beforehand, nodes of eight GPUs
        // as a case of their own, and the order kept from round to round took a third of them away.  406 jobs on 8 nodes, 720
        // ticks: 41.0 ms with searches between barriers, 28.5 with the states looked up, 18.8 now; 200 jobs on 16 nodes, 60
        // ticks: 1.81 and 0.78 ms; 900 on 128 nodes: 27.1 and 19.2.
        const SimArgs &S = K.S;
        __shared__ uint32_t sh_open[3], sh_used, sh_gone, sh_changed[WAVES], sh_who[ND_CHANGED], sh_before[ND_CHANGED];
        __shared__ unsigned long long sh_was[ND_CHANGED], sh_now[ND_CHANGED];
        __shared__ double sh_part[ND_WAVES];
        const uint32_t n_cpu = A.X.grid.n_cpu, n_mem = A.X.grid.n_mem;
        const bool mine = tid < J;
        auto barrier = [&]() { rs_lds_barrier(); };          // (what the wavefronts tell each other lies in LDS)
        // where a state's word (lane & 15) goes: the job's place in an array of words
        const uint32_t field = lane & 15u;
        uint32_t to = 0, stride = 1u;
        uint32_t *const words0 = reinterpret_cast<uint32_t *>(sh_raw);
        {
            auto at_word = [&](const void *p) { return (uint32_t)(reinterpret_cast<const uint32_t *>(p) - words0); };
            const uint32_t places[ND_STATE_WORDS] = {at_word(A.ug), at_word(A.udg), at_word(A.gain_g), at_word(A.tgt_g), at_word(A.uc), at_word(A.gain_c),
                                                     at_word(A.lvl_c), at_word(A.udc_c), at_word(A.udc_c) + 1u, at_word(A.ds_g), at_word(A.ds_c),
                                                     at_word(A.give), at_word(A.give) + 1u, at_word(A.give) + 2u, at_word(A.give) + 3u, at_word(A.give_c)};
#pragma unroll
            for (uint32_t f = 0; f < ND_STATE_WORDS; ++f) to = field == f ? places[f] : to;
            if (field == ND_DC_LO || field == ND_DC_HI) stride = 2u;
            if (field == ND_GIVES || field == ND_LOSS || field == ND_TO || field == ND_DS_G1) stride = 4u;
        }
        const bool slope = field == ND_DS_G || field == ND_DS_C;
        auto state_word = [&](uint32_t v, int32_t gi, uint32_t ci) { return K.states.words[nd_state_at(K.states, v, n_cpu, gi, ci) * ND_STATE_WORDS + field]; };
        auto refresh = [&](uint32_t v, bool on) {            // job v of the lane's row of 16, from what it holds
            const int32_t gi = A.st.gi[v];
            const uint32_t ci = A.st.ci[v], state = state8[v];
            if (!on) return;
            uint32_t w = state_word(v, gi, ci);
            if (slope && state != RK_JOB_NORMAL) w = __float_as_uint(INF);     // (who takes no part gives nothing)
            words0[to + v * stride] = w;
        };
        auto copy_alone = [&](uint32_t *dst, const uint32_t *src) {            // the nodes, by the first wavefront
            for (uint32_t i = lane; i < A.nodes_words / 4u; i += 64u) reinterpret_cast<uint4 *>(dst)[i] = reinterpret_cast<const uint4 *>(src)[i];
            rs_wave_order();
        };
        const uint32_t NO_SLOPE = 0xFF800000u;               // an infinite slope as a word that orders like it
        uint32_t *const list = fin_list;                     // the jobs that may be served, in the loop's order
        auto round_alone = [&](uint32_t n_list) {
            uint32_t pos = 0, free_c = 0;                    // the first job of the list that has not been looked at
            bool fresh = true, with_c = false;               // (with_c: the CPUs' slopes are those of the present state)
            RsMin low[2];
            low[0] = low[1] = RsMin{INF, INF, ND_NONE};
            // the two lowest slopes of a resource and whose the lowest is, among those who are on the nodes (nobody else gives)
            auto lowest = [&](uint32_t r) {
                const float *const ds = sh_ds + r * (JL + 1);
                uint32_t v = A.res[lane < gpus ? lane : 0u] >> 16, x = rs_ordered(ds[v]), y = NO_SLOPE;    // (nobody: infinite slopes)
                for (uint32_t i = lane + 64u; i < gpus; i += 64u) {
                    const uint32_t w = A.res[i] >> 16, z = rs_ordered(ds[w]);
                    const bool first = z < x || (z == x && w < v);
                    const uint32_t behind = first ? x : z;   // the one that is not, if it is another job's
                    y = w != v && behind < y ? behind : y;
                    if (first) { x = z; v = w; }
                }
                const uint32_t least = wave_min_u32_rows(x), whose = wave_min_u32_rows(x == least ? v : ND_NONE);
                const uint32_t second = wave_min_u32_rows(v == whose ? y : x);
                low[r] = RsMin{rs_unordered(least), rs_unordered(second), least == NO_SLOPE ? ND_NONE : whose};
            };
            for (;;) {
                if (fresh) {
                    // what the nodes can give at every CPU level, and all free CPUs
                    if (n_cpu > 16u) {                       // a level per lane, one node after the other
                        const float rcp = lane < n_cpu ? sh_rcp[lane] : 1.f;
                        uint32_t t = 0, all = 0;
                        for (uint32_t n = 0; n < N; ++n) {
                            const uint32_t fg = A.free_g[n], fc = A.free_c[n], by_cpu = over(fc, rcp);
                            t += by_cpu < fg ? by_cpu : fg;
                            all += fc;
                        }
                        if (lane < n_cpu) sh_take[lane] = t;
                        free_c = one(all);
                    } else if (N <= 16u) {                   // a level per row of lanes, a node per lane
                        const uint32_t n = lane & 15u, fg = n < N ? A.free_g[n] : 0u, fc = n < N ? A.free_c[n] : 0u;
                        for (uint32_t l0 = 0; l0 <= n_cpu; l0 += 4u) {
                            const uint32_t l = l0 + (lane >> 4);
                            const uint32_t by_cpu = l < n_cpu ? over(fc, sh_rcp[l]) : fc;
                            uint32_t t = l >= n_cpu || by_cpu < fg ? by_cpu : fg;
                            t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x111, 0xF, 0xF, true);     // row_shr:1, 2, 4, 8
                            t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x112, 0xF, 0xF, true);
                            t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x114, 0xF, 0xF, true);
                            t += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)t, 0x118, 0xF, 0xF, true);
                            if (n == 15u && l < n_cpu) sh_take[l] = t;
                            if (l0 + 4u > n_cpu) free_c = wave_lane_u32(t, (n_cpu - l0) * 16u + 15u);
                        }
                    } else {
                        for (uint32_t l = 0; l <= n_cpu; ++l) {
                            const float rcp = l < n_cpu ? sh_rcp[l] : 1.f;
                            uint32_t t = 0;
                            for (uint32_t n = lane; n < N; n += 64u) {
                                const uint32_t fg = A.free_g[n], fc = A.free_c[n], by_cpu = l < n_cpu ? over(fc, rcp) : fc;
                                t += l >= n_cpu || by_cpu < fg ? by_cpu : fg;
                            }
                            t = nd_wave_sum(t);
                            if (l < n_cpu) sh_take[l] = t;
                            else free_c = t;
                        }
                    }
                    lowest(0);
                    with_c = false;
                    rs_wave_order();
                }
                // the next job of the list that finds something to do
                uint32_t last_j = ND_NONE;
                while (pos < n_list) {
                    const bool in = pos + lane < n_list;
                    const uint32_t jj = list[in ? pos + lane : pos];
                    const float ug = A.ug[jj], uc = A.uc[jj];
                    const uint32_t dg = A.udg[jj], ci = A.st.ci[jj];
                    const unsigned long long dc = A.udc_c[jj];
                    const float lowest_g = jj == low[0].i1 ? low[0].m2 : low[0].m1;
                    bool busy = ug > 0.f && (sh_take[ci] >= dg || ug > lowest_g);
                    if (__ballot(uc > 0.f && free_c < dc) && !with_c) { lowest(1); with_c = true; }
                    const float lowest_c = jj == low[1].i1 ? low[1].m2 : low[1].m1;
                    busy = busy || (uc > 0.f && (free_c >= dc || uc > lowest_c));
                    const unsigned long long m = __ballot(in && busy);
                    if (!m) { pos += 64u; continue; }
                    const uint32_t s = (uint32_t)__ffsll((long long)m) - 1u;
                    pos += s + 1u;
                    last_j = wave_lane_u32(jj, s);
                    break;
                }
                if (last_j == ND_NONE) break;
                // ScheduleJob
                const uint32_t j = last_j, before = moves;
                bool gpus_done = false;
                for (;;) {
                    uint32_t did = DID_NOTHING, after = 0;   // after: the job's values if the step is committed, on their way meanwhile
                    if (!gpus_done) {
                        after = state_word(j, A.tgt_g[j], A.st.ci[j]);
                        did = gpu_step(j);
                        if (did == DID_NOTHING) {
                            gpus_done = true;
                            if (dirty) copy_alone(nodes, keep);
                        }
                    }
                    if (did == DID_NOTHING) {
                        did = cpu_step(j);
                        if (did == DID_NOTHING) {
                            if (dirty) copy_alone(nodes, keep);
                            break;
                        }
                    }
                    rs_wave_order();
                    for (uint32_t i0 = 0; i0 < touched; i0 += 4u) {            // a row of lanes per job that gave something
                        const uint32_t i = i0 + (lane >> 4);
                        refresh(A.touched[i < touched ? i : i0], i < touched);
                    }
                    if (did == DID_CPUS) refresh(j, lane < 16u);
                    else if (lane < 16u) words0[to + j * stride] = after;      // (who takes a step takes part)
                    rs_wave_order();
                    copy_alone(keep, nodes);
                }
                fresh = moves != before;
            }
        };

        SimJob s = {0u, 0u, RK_NO_PLAN, 0u, 0.0, 0.0, 0.0, -1.0, false};
        int32_t seg = -1;
        uint32_t lvl = 0, state = RK_JOB_OUT;
        double arrival = 0.0, work = 0.0, delta = 0.0;
        float ref = 1.f;
        if (mine) {
            arrival = S.arrival[tid]; work = S.work[tid]; delta = S.delta[tid]; ref = A.X.ref_thr[tid];
            s = SimJob{S.S.g[tid], S.S.c[tid], S.S.plan[tid], S.n_reconf[tid], S.S.owed[tid], S.held[tid], S.progress[tid], S.finish[tid],
                       S.S.done[tid] != 0};
            seg = S.S.seg[tid]; lvl = S.S.lvl[tid]; state = state8[tid];
        }
        if (tid < 3u) sh_open[tid] = 0u;
        if (tid == 0) { sh_list = 0u; sh_used = 0u; sh_gone = 0u; }
        rk_assign a = {0u, 0u, 0.f, RK_NO_PLAN, 0.f};
        float total = 0.f;
        uint32_t turn = 0, place = 0;
        unsigned long long place_key = 0ull;                 // the job's key in the order (0: not in it) and its place
        __syncthreads();
        for (uint32_t done = 0;;) {
            // ---- a round: who may be served, and who is where when it begins
            for (uint32_t i = tid; i < gpus; i += THREADS) start_res[i] = A.res[i];
            for (uint32_t n = tid; n < N; n += THREADS) sh_mem[n] = 0.f;
            if (share) for (uint32_t i = tid; i < N * gpus; i += THREADS) share[i] = 0.f;
            // The jobs that find something to do now, by both slopes descending, then the lower job; then those that only may
            // (they hold something and have no step up), whose slopes are all zero.  From round to round few jobs' slopes
            // change: the others move past those that left their place or came to one (144 jobs, 10 of them changed: 3,500
            // cycles; counting what comes before each of them 12,000).
            uint32_t n_list = 0, n_idle = 0;
            {
                const float ug = mine ? A.ug[tid] : 0.f, uc = mine ? A.uc[tid] : 0.f;
                const bool in = state == RK_JOB_NORMAL && (ug > 0.f || uc > 0.f), idle = state == RK_JOB_NORMAL && !in && A.st.gi[tid] >= 0;
                const unsigned long long key = in ? ((unsigned long long)rs_ordered(ug) << 32) | rs_ordered(uc) : 0ull;
                const bool changed = key != place_key;
                const unsigned long long m = __ballot(in), m_idle = __ballot(idle), m_changed = __ballot(changed), below = (1ull << lane) - 1ull;
                if (lane == 0) {
                    sh_scan[wave] = (uint32_t)__popcll(m) | (uint32_t)__popcll(m_idle) << 16;
                    sh_changed[wave] = (uint32_t)__popcll(m_changed);
                }
                barrier();
                uint32_t p = (uint32_t)__popcll(m & below), p_idle = (uint32_t)__popcll(m_idle & below), p_changed = (uint32_t)__popcll(m_changed & below);
                uint32_t n_changed = 0;
#pragma unroll
                for (uint32_t w = 0; w < WAVES; ++w) {
                    const uint32_t n = sh_scan[w], before = w < wave ? n : 0u, c = sh_changed[w];
                    p += before & 0xFFFFu; p_idle += before >> 16; p_changed += w < wave ? c : 0u;
                    n_list += n & 0xFFFFu; n_idle += n >> 16; n_changed += c;
                }
                n_list = one(n_list); n_idle = one(n_idle); n_changed = one(n_changed);
                if (idle) list[n_list + p_idle] = tid;
                if (n_changed <= ND_CHANGED) {
                    if (changed) { sh_was[p_changed] = place_key; sh_now[p_changed] = key; sh_who[p_changed] = tid; sh_before[p_changed] = 0u; }
                    barrier();
                    const bool stays = in && !changed;
                    for (uint32_t c = 0; c < n_changed; ++c) {
                        const unsigned long long was = sh_was[c], now = sh_now[c];
                        const bool lower = sh_who[c] < tid;
                        const bool left = was > key || (was == key && lower), came = now > key || (now == key && lower);
                        place += (came ? 1u : 0u) - (left ? 1u : 0u);
                        const unsigned long long ahead = __ballot(stays && !came);
                        if (lane == 0 && ahead) atomicAdd(&sh_before[c], (uint32_t)__popcll(ahead));
                    }
                    if (n_changed) barrier();
                    if (in && changed) {
                        place = sh_before[p_changed];
                        for (uint32_t c = 0; c < n_changed; ++c) {
                            const unsigned long long now = sh_now[c];
                            place += now > key || (now == key && sh_who[c] < tid) ? 1u : 0u;
                        }
                    }
                    if (in) list[place] = tid;
                } else {
                    if (in) { A.okey[p] = key; list[p] = tid; }
                    barrier();
                    uint32_t most = 128u;
                    while (most < n_list) most <<= 1;
                    // bitonic, every step the same way round (what is beyond the list comes last and never moves); steps that
                    // stay within the 128 places of a wavefront need no barrier
                    auto exchange = [&](uint32_t x, uint32_t y) {
                        if (y >= n_list) return;
                        const unsigned long long kx = A.okey[x], ky = A.okey[y];
                        const uint32_t jx = list[x], jy = list[y];
                        if (kx > ky || (kx == ky && jx < jy)) return;
                        A.okey[x] = ky; A.okey[y] = kx;
                        list[x] = jy; list[y] = jx;
                    };
                    for (uint32_t k = 2u; k <= most; k <<= 1)
                        for (uint32_t d = k >> 1; d > 0; d >>= 1) {
                            if (tid < most / 2u) {
                                const uint32_t x = 2u * d * (tid / d) + tid % d;       // (powers of two)
                                exchange(x, d == k >> 1 ? x - tid % d + k - 1u - tid % d : x + d);
                            }
                            if ((k > 128u && (d >= 128u || d == k >> 1)) || (d == 1u && k >= 128u)) barrier(); else rs_wave_order();
                        }
                    for (uint32_t i = tid; i < n_list; i += THREADS) fin_np[list[i]] = i;
                    barrier();
                    if (in) place = fin_np[tid];
                }
                place_key = key;
            }
            barrier();
            if (wave == 0) round_alone(n_list + n_idle);
            barrier();
            // ---- memory, then the record of every job that holds something, in job order
            const int32_t gi = mine ? A.st.gi[tid] : -1;
            const uint32_t ci = mine ? A.st.ci[tid] : 0u;
            const bool holds = gi >= 0;
            uint4 best = {0u, RK_NO_PLAN, ND_NONE, 0u};
            float cost = 0.f;
            if (holds) best = K.states.best[nd_state_at(K.states, tid, n_cpu, gi, ci)];
            if (holds && best.z != ND_NONE) { cost = A.X.grid.mem_levels_gb[best.z]; if (A.X.grid.mem_mode) cost = cost * (float)best.w; }
            const unsigned long long holders = __ballot(holds);
            if (lane == 0) sh_scan[wave] = (uint32_t)__popcll(holders);
            if (tid == 0) { sh_list = 0u; sh_used = 0u; }
            barrier();
            uint32_t h = (uint32_t)__popcll(holders & ((1ull << lane) - 1ull)), n_holders = 0;
#pragma unroll
            for (uint32_t w = 0; w < WAVES; ++w) { const uint32_t n = sh_scan[w]; h += w < wave ? n : 0u; n_holders += n; }
            if (holds) {                                     // (each is on a node: at most as many as GPUs)
                fin_off[tid] = h;
                held_cost[h] = best.z == ND_NONE ? -1.f : cost;
                held_g[h] = best.w;
            }
            barrier();
            for (uint32_t i = tid; i < gpus; i += THREADS) {
                const uint32_t n = i / gpn;
                if (i - n * gpn < A.cnt[n]) {
                    const uint32_t word = A.res[i], hv = fin_off[word >> 16];
                    const float c = held_cost[hv];
                    if (c >= 0.f) {
                        const float asks = (c * (float)(word & 0xFFFFu)) / (float)held_g[hv];
                        atomicAdd(&sh_mem[n], asks);
                        if (share) share[hv * N + n] = asks;
                    }
                }
            }
            barrier();
            uint32_t short_of = 0;
            for (uint32_t n = lane; n < N; n += 64u) short_of |= !(sh_mem[n] <= A.mem_gb * 0.999f) ? 1u : 0u;
            bool dropped = holds && best.z == ND_NONE;
            if (__ballot(short_of != 0u)) {                  // (the same in all wavefronts) some node's memory can bind: job by job
                if (n_mem == 1u && share) {
                    if (wave == 0) {
                        float left = A.mem_gb, next = lane < N && n_holders ? share[lane] : 0.f;
                        for (uint32_t q = 0; q < n_holders; ++q) {
                            const float asks = next;
                            next = lane < N && q + 1u < n_holders ? share[(q + 1u) * N + lane] : 0.f;
                            const bool bad = __ballot(!(asks <= left)) != 0ull;
                            if (!bad) left = left - asks;
                            else if (lane == 0) held_g[q] = 0u;
                        }
                    }
                    barrier();
                    dropped = dropped || (holds && held_g[h] == 0u);
                } else {
                    nd_finish<THREADS>(A, fin_np, fin_off, keep, A.touched, fin_list, sh_mem, sh_scan);
                    __syncthreads();
                    if (mine) a = A.assign[tid];
                    dropped = holds && a.g == 0u;
                    best.x = __float_as_uint(a.thr); best.y = a.plan; cost = a.mem_gb;
                }
            }
            a = rk_assign{0u, 0u, 0.f, RK_NO_PLAN, 0.f};
            if (holds && !dropped) { a.g = best.w; a.c = sh_cpl[ci] * best.w; a.mem_gb = cost; a.plan = best.y; a.thr = __uint_as_float(best.x); }
            if (dropped) A.st.gi[tid] = -1;               // (its parts are still on the nodes, and its level is theirs)
            // the total: the additions of nd_finish, a job per thread
            {
                double x = a.g ? (double)a.thr / (double)ref : 0.0;
                if (__ballot(x != 0.0)) x = wave_sum_f64(x);
                const uint32_t used = nd_wave_sum(state != RK_JOB_OUT ? a.g : 0u);
                if (lane == 0) { sh_part[wave] = x; if (used) atomicAdd(&sh_used, used); }
            }
            barrier();
            // ---- is anybody somewhere else than when the round began?
            bool other = false;
            for (uint32_t i = tid; i < gpus; i += THREADS) {
                uint32_t word = A.res[i];
                const uint32_t v = word >> 16;
                if (v < J && A.st.gi[v] < 0) word = EMPTY;
                other |= word != start_res[i];
            }
            if (tid == 0) {
                double sum = 0.0;
#pragma unroll
                for (uint32_t w = 0; w < WAVES; ++w) sum += sh_part[w];
                total = (float)sum;
            }
            const uint32_t used = sh_used;
            // ---- the tick is closed and the next one opened, and those after it that start from what this round started from
            const uint32_t round_state = state;
            bool more = true;
            for (;;) {
                const double t = (double)tick * S.dt;
                if (state != RK_JOB_OUT && sim_close(s, a, t, S.dt, delta, work)) {
                    other = true;
                    seg = s.g ? gi : -1;
                    lvl = s.g ? ci : 0u;
                }
                if (tid == 0) {
                    if (S.out.gpus_in_use) S.out.gpus_in_use[tick] = used;
                    if (S.out.totals) S.out.totals[tick] = total;
                }
                if (++tick == S.n_ticks) { more = false; break; }
                const double t1 = (double)tick * S.dt;
                uint32_t now = RK_JOB_OUT;
                if (mine && arrival <= t1 && !s.done) now = sim_frozen(s.g, s.held, s.n_reconf, delta, S.gate) ? RK_JOB_FROZEN : RK_JOB_NORMAL;
                other |= now != state;
                state = now;
                const uint32_t frozen = (uint32_t)__popcll(__ballot(now == RK_JOB_FROZEN));
                const bool any = __ballot(other) != 0ull;
                if (lane == 0 && frozen) atomicAdd(&sh_open[turn], frozen);
                if (lane == 0 && any) atomicOr(&sh_open[turn], 0x80000000u);
                if (tid == 0) sh_open[turn == 2u ? 0u : turn + 1u] = 0u;       // (read by all before the barrier before)
                barrier();
                const uint32_t open = sh_open[turn];
                turn = turn == 2u ? 0u : turn + 1u;
                if (tid == 0 && S.out.frozen) S.out.frozen[tick] = open & 0x7FFFFFFFu;
                if (open & 0x80000000u) break;
            }
            if (!more || ++done == K.rounds) break;
            // ---- what the next round starts from: those who leave free their parts, changed jobs' values are looked up
            {
                const bool stays = state != RK_JOB_OUT && seg >= 0;
                const int32_t gi_now = mine ? A.st.gi[tid] : -1;
                const bool leaves = gi >= 0 && !stays;       // (dropped, or it has come to its end)
                if (mine) {
                    if (state != round_state || leaves) {
                        fin_np[atomicAdd(&sh_list, 1u)] = tid;
                        state8[tid] = (uint8_t)state;
                    }
                    if (leaves) { if (gi_now >= 0) A.st.gi[tid] = -1; sh_gone = 1u; }
                }
                barrier();
                const uint32_t n_changed = sh_list;
                if (sh_gone)
                    for (uint32_t n = tid; n < N; n += THREADS) {
                        uint32_t c = A.cnt[n], fg = 0, fc = 0;
                        for (uint32_t i = 0; i < c;) {
                            const uint32_t word = A.res[n * gpn + i], v = word >> 16;
                            if (A.st.gi[v] >= 0) { ++i; continue; }
                            fg += word & 0xFFFFu; fc += (word & 0xFFFFu) * sh_cpl[A.st.ci[v]];
                            c -= 1u;
                            A.res[n * gpn + i] = A.res[n * gpn + c];
                            A.res[n * gpn + c] = EMPTY;
                        }
                        if (fg) { A.cnt[n] = c; A.free_g[n] += fg; A.free_c[n] += fc; }
                    }
                for (uint32_t i0 = 4u * wave; i0 < n_changed; i0 += 4u * WAVES) {
                    const uint32_t i = i0 + (lane >> 4);
                    refresh(fin_np[i < n_changed ? i : i0], i < n_changed);
                }
                barrier();
                if (leaves) A.st.ci[tid] = 0u;
                if (tid == 0) { sh_list = 0u; sh_gone = 0u; }
                copy_nodes(keep, nodes);
                barrier();
            }
        }
        // ---- the state, for the next launch
        if (mine) {
            S.S.g[tid] = s.g; S.S.c[tid] = s.c; S.S.plan[tid] = s.plan; S.S.seg[tid] = seg; S.S.lvl[tid] = lvl;
            S.S.owed[tid] = s.owed; S.S.done[tid] = s.done ? 1 : 0;
            S.held[tid] = s.held; S.progress[tid] = s.progress; S.finish[tid] = s.finish; S.n_reconf[tid] = s.n_reconf;
            S.F.state[tid] = (uint8_t)state;
        }
        {                                                    // where the jobs are: a job's parts in node order
            const bool on = mine && A.st.gi[tid] >= 0;
            auto parts = [&](uint32_t at, bool write) {
                uint32_t p = 0;
                for (uint32_t n = 0; n < N; ++n)
                    for (uint32_t i = 0; i < A.cnt[n]; ++i) {
                        const uint32_t word = A.res[n * gpn + i];
                        if ((word >> 16) != tid) continue;
                        const uint32_t k = word & 0xFFFFu;
                        if (write) S.at_ent[at + p] = rk_place_entry{n, k, sh_cpl[A.st.ci[tid]] * k, 0.f};
                        ++p;
                    }
                return p;
            };
            const uint32_t p = on ? parts(0u, false) : 0u;
            uint32_t all;
            const uint32_t at = nd_block_scan<THREADS>(p, all, sh_scan);
            if (mine) S.at_off[tid] = at;
            if (tid == 0) S.at_off[J] = all;
            if (on) (void)parts(at, true);
        }
        if (tid == 0) {
            *S.tick = tick;
            __hip_atomic_store(S.h_tick, tick, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    } else if constexpr (!SIM) {
        round();
        nd_finish<THREADS>(A, fin_np, fin_off, keep, A.touched, fin_list, sh_mem, sh_scan);
        if (tid == 0 && A.stats) { A.stats[0] = moves; A.stats[1] = full; A.stats[2] = shrinks; A.stats[3] = undone; A.stats[4] = 0u; }
    } else {
        const SimArgs &S = K.S;
        for (uint32_t done = 0;;) {
            round();
            nd_finish<THREADS>(A, fin_np, fin_off, keep, A.touched, fin_list, sh_mem, sh_scan);
            __syncthreads();
            const bool moved = sim_placed<THREADS>(S);
            const bool more = sim_ticks<THREADS>(S, tick, false, moved);
            if (tid == 0) sh_list = 0u;
            __syncthreads();
            if (!more || ++done == K.rounds) break;
            // who holds something else than the round left them with, or takes part in another way
            for (uint32_t j = tid; j < J; j += THREADS) {
                const uint32_t state = A.state[j], lvl = A.cur_c[j], ci = A.st.ci[j];
                const int32_t seg = A.cur_seg[j], gi = A.st.gi[j];
                const bool holds = rs_holds(A, j) && seg >= 0 && (uint32_t)seg < A.seg_off[j + 1] - A.seg_off[j] && lvl < A.X.grid.n_cpu;
                if (state != old_state[j] || (holds ? seg != gi || lvl != ci : gi >= 0)) fin_list[atomicAdd(&sh_list, 1u)] = j;
                old_state[j] = state;
                A.st.gi[j] = holds ? seg : -1;
                if (holds) A.st.ci[j] = lvl;                 // (a job that leaves keeps its level until its parts are free)
            }
            __syncthreads();
            for (uint32_t n = tid; n < N; n += THREADS) {    // the parts of those that left
                uint32_t c = A.cnt[n], fg = 0, fc = 0;
                for (uint32_t i = 0; i < c;) {
                    const uint32_t word = A.res[n * gpn + i], v = word >> 16;
                    if (A.st.gi[v] >= 0) { ++i; continue; }
                    fg += word & 0xFFFFu; fc += (word & 0xFFFFu) * sh_cpl[A.st.ci[v]];
                    c -= 1u;
                    A.res[n * gpn + i] = A.res[n * gpn + c];
                    A.res[n * gpn + c] = EMPTY;
                }
                if (fg) { A.cnt[n] = c; A.free_g[n] += fg; A.free_c[n] += fc; }
            }
            __syncthreads();
            const uint32_t n_changed = sh_list;
            for (uint32_t i = tid; i < n_changed; i += THREADS) if (A.st.gi[fin_list[i]] < 0) A.st.ci[fin_list[i]] = 0u;
            copy_nodes(keep, nodes);
            __syncthreads();
            for (uint32_t i = wave; i < 2u * n_changed; i += WAVES) {
                const uint32_t v = one(fin_list[i >> 1]);
                nd_refresh_wave(A, v, one_i(A.st.gi[v]), one(A.st.ci[v]), lane, (i & 1u) == 0u, (i & 1u) != 0u);
            }
            __syncthreads();
        }
        if (tid == 0) {
            *S.tick = tick;
            __hip_atomic_store(S.h_tick, tick, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

template <int THREADS, bool LJ>
__global__ __launch_bounds__(THREADS) void k_nodes_lds(NdKernArgs K) { nodes_lds<THREADS, LJ, false, false, 0u>(K); }

struct NdSimArgs : NdKernArgs { SimArgs S; uint32_t rounds, shares; NdStates states; };     // rounds of a launch, at most; TAB: shares, states
template <int THREADS, bool TAB, uint32_t GPN>
__global__ __launch_bounds__(THREADS) void k_sim_nodes(NdSimArgs K) { nodes_lds<THREADS, true, true, TAB, GPN>(K); }

__global__ __launch_bounds__(ND_THREADS) void k_reschedule_nodes(NdKernArgs K) {
    // what every job loses per GPU / CPU it gives, [2][n_jobs]: read at every look at a node's residents and at every
    // look for the next job, so the kernel keeps them in LDS (k_nd_prepare left them in memory)
    extern __shared__ float sh_ds[];
    NdArgs A(K.b, K.X);
    for (uint32_t j = threadIdx.x; j < A.n_jobs; j += ND_THREADS) {
        sh_ds[j] = K.b.ds_g[j];
        sh_ds[A.n_jobs + j] = K.b.ds_c[j];
    }
    A.ds_g = sh_ds;
    A.ds_c = sh_ds + A.n_jobs;
    __shared__ RsStep sh_step;
    __shared__ float sh_lost;
    __shared__ unsigned long long sh_pick_key[ND_WAVES + 1];
    __shared__ uint32_t sh_pick_j[ND_WAVES + 1];
    __shared__ uint32_t sh_scan[ND_WAVES];
    __shared__ uint32_t sh_lack, sh_ok, sh_go, sh_touched, sh_epoch, sh_moves, sh_full, sh_shrinks, sh_undone;
    __shared__ uint32_t sh_vnode, sh_next, sh_v, sh_rest, sh_per_v, sh_flag, sh_np, sh_bad, sh_done, sh_ask;
    __shared__ unsigned long long sh_take[RK_MAX_CPU_LEVELS], sh_free_c;
    __shared__ RsMin sh_min[2];
    __shared__ unsigned long long sh_two_k[2 * (ND_WAVES + 1)];
    __shared__ uint32_t sh_two_s[2 * (ND_WAVES + 1)];
    __shared__ float sh_mem[RK_MAX_NODES];                  // memory of the nodes: sums of wishes, then what is left
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t J = A.n_jobs, N = A.n_nodes;
    const float INF = __int_as_float(0x7F800000);
    const uint32_t per_thread = (N + ND_THREADS - 1) / ND_THREADS;          // <= ND_PER

    auto block_scan = [&](uint32_t val, uint32_t &all) { return nd_block_scan<ND_THREADS>(val, all, sh_scan); };

    // ---- the state the jobs are in has been loaded (k_nd_init, k_nd_prepare); no node may hold more than it has
    if (tid == 0) { sh_bad = 0u; sh_epoch = 0u; sh_moves = 0u; sh_full = 0u; sh_shrinks = 0u; sh_undone = 0u; }
    __syncthreads();
    for (uint32_t n = tid; n < N; n += ND_THREADS)
        if (A.cnt[n] > A.gpn || A.free_g[n] > A.gpn || A.free_c[n] > A.cpn) atomicOr(&sh_bad, 1u);
    for (uint32_t j = tid; j < J; j += ND_THREADS) {
        A.stamp[j] = 0u;
        if (A.first[j] & 2u) atomicOr(&sh_bad, 1u);
    }
    __syncthreads();
    if (sh_bad) { nd_refuse<ND_THREADS>(A); return; }
    // the node tables and their copy, four words at a time, two pieces in flight (nodes_words is a multiple of four)
    auto copy_nodes = [&](uint32_t *to, const uint32_t *from) {
        const uint4 *src = reinterpret_cast<const uint4 *>(from);
        uint4 *dst = reinterpret_cast<uint4 *>(to);
        const uint32_t n4 = A.nodes_words / 4u;
        for (uint32_t i = tid; i < n4; i += 2 * ND_THREADS) {
            const uint4 a = src[i];
            const bool two = i + ND_THREADS < n4;
            const uint4 b = two ? src[i + ND_THREADS] : a;
            dst[i] = a;
            if (two) dst[i + ND_THREADS] = b;
        }
    };
    auto keep_nodes = [&]() { copy_nodes(A.keep_nodes, A.free_g); };
    auto restore_nodes = [&]() { copy_nodes(A.free_g, A.keep_nodes); };
    // first thread: remember job v as it is before this step changes it
    auto remember = [&](uint32_t v) {
        if (A.stamp[v] == sh_epoch) return;
        A.stamp[v] = sh_epoch;
        A.keep_gi[v] = A.st.gi[v]; A.keep_ci[v] = A.st.ci[v];
        A.keep_ds[2 * v] = A.ds_g[v]; A.keep_ds[2 * v + 1] = A.ds_c[v];
        A.touched[sh_touched++] = v;
    };
    auto put_jobs_back = [&]() {
        for (uint32_t i = 0; i < sh_touched; ++i) {
            const uint32_t v = A.touched[i];
            A.st.gi[v] = A.keep_gi[v]; A.st.ci[v] = A.keep_ci[v];
            A.ds_g[v] = A.keep_ds[2 * v]; A.ds_c[v] = A.keep_ds[2 * v + 1];
        }
        sh_undone += sh_touched ? 1u : 0u;
    };

    auto refresh = [&](uint32_t v) { nd_refresh_wave(A, v, A.st.gi[v], A.st.ci[v], lane); };
    // ScheduleJob(j); the same code path for all threads
    auto schedule_job = [&](uint32_t j) {
        for (;;) {                                           // ---- GPUs
            if (tid == 0) {
                const RsStep up = nd_cached_step(A, j, 0);
                sh_step = up;
                sh_lack = (uint32_t)up.dg; sh_lost = 0.f; sh_ok = 1u; sh_touched = 0u; sh_epoch += 1u;
            }
            __syncthreads();
            const RsStep st = sh_step;
            if (!st.any) { __syncthreads(); break; }
            const bool below_min = rs_fl_s(A, j) >= 0 && A.st.gi[j] < rs_fl_s(A, j);
            const uint32_t per_gpu = nd_cpl(A, st.lvl);
            keep_nodes();
            __syncthreads();
            if (A.st.gi[j] >= 0 && st.lvl != A.st.ci[j]) {   // its parts go to the step's level: their CPUs must be free
                const uint32_t more = per_gpu - nd_cpl(A, A.st.ci[j]);
                for (uint32_t n = tid; n < N; n += ND_THREADS) {
                    const uint32_t k = nd_part(A, n, j);
                    if (!k) continue;
                    if (A.free_c[n] < more * k) atomicAnd(&sh_ok, 0u);
                    else A.free_c[n] -= more * k;
                }
                __syncthreads();
            }
            uint32_t n0 = 0;
            bool walking = sh_ok && sh_lack > 0;             // (read here, written again only behind the next barrier)
            __syncthreads();
            while (walking && n0 < N) {                      // the walk over the nodes, a node per thread at a time
                const uint32_t lack = sh_lack;
                const uint32_t n = n0 + tid;
                const bool in = n < N;
                uint32_t offer = 0;
                bool ask = false;                            // somebody here may be shrunk
                if (in) {
                    const uint32_t by_cpu = A.free_c[n] / per_gpu;
                    offer = A.free_g[n] < by_cpu ? A.free_g[n] : by_cpu;
                    uint32_t who;
                    const float low = nd_lowest_on(A, n, j, A.ds_g, who);
                    ask = who != ND_NONE && (below_min || st.slope > low);
                }
                if (tid == 0) { sh_done = ND_THREADS; sh_ask = ND_THREADS; }
                uint32_t all;
                const uint32_t before = block_scan(offer, all);          // (its barriers order the two lines around it)
                if (in && before + offer >= lack) atomicMin(&sh_done, tid);
                if (in && ask && before + offer < lack) atomicMin(&sh_ask, tid);
                __syncthreads();
                const uint32_t done_t = sh_done, ask_t = sh_ask;
                const uint32_t last = done_t < ask_t ? done_t : ask_t;   // the nodes up to here give what they offer
                if (in && tid <= last && offer) nd_add(A, n, j, offer < lack - before ? offer : lack - before, per_gpu);
                if (tid == (last < ND_THREADS ? last : 0u)) {
                    const uint32_t upto = last < ND_THREADS ? before + offer : all;
                    sh_lack = lack - (upto < lack ? upto : lack);
                    sh_vnode = ask_t < done_t ? n0 + ask_t : ND_NONE;
                    sh_next = ask_t < done_t ? n0 + ask_t + 1u : n0 + ND_THREADS;
                }
                __syncthreads();
                const uint32_t f = sh_vnode;
                if (f != ND_NONE) {                          // node f: the job still lacks GPUs and somebody may be shrunk
                    for (;;) {
                        if (wave == 0) {                     // the first wavefront: a resident of node f per lane
                            const uint32_t c = A.cnt[f];
                            const size_t base = (size_t)f * A.gpn;
                            if (c > 64u) {                       // more residents than lanes: the first lane asks them one by one
                                if (lane == 0) {
                                    uint32_t who;
                                    const float low = nd_lowest_on(A, f, j, A.ds_g, who);
                                    if (who == ND_NONE || !(below_min || st.slope > low)) {
                                        sh_v = ND_NONE;
                                    } else {
                                        const RsGive gv = rs_down_gpu(A, who);
                                        remember(who);
                                        const uint32_t per_v = nd_cpl(A, A.st.ci[who]);
                                        const uint32_t here_has = nd_part(A, f, who);
                                        const uint32_t here = (uint32_t)gv.dg < here_has ? (uint32_t)gv.dg : here_has;
                                        nd_drop(A, f, who, here, per_v);
                                        sh_rest = (uint32_t)gv.dg - here; sh_per_v = per_v; sh_v = who;
                                        sh_lost = sh_lost + gv.loss;
                                        A.st.gi[who] = gv.tgt; if (gv.tgt < 0) A.st.ci[who] = 0u;
                                        rs_refresh_give(A, who);
                                        sh_shrinks += 1u;
                                    }
                                }
                            } else {
                                // the node's list and what it has free, asked for together; then the residents' slopes
                                const uint32_t free_g = A.free_g[f], free_c = A.free_c[f];
                                const uint32_t word = lane < c ? A.res[base + lane] : j << 16;
                                const uint32_t rv = word >> 16;
                                const float sl = rv != j ? A.ds_g[rv] : INF;
                                unsigned long long key = ~0ull;      // (slope as a word that orders like it, job): lower job among equals
                                if (sl < INF) key = ((unsigned long long)rs_ordered(sl) << 32) | rv;
                                key = wave_min_u64_rows(key);
                                const uint32_t who = (uint32_t)key;
                                const float low = rs_unordered((uint32_t)(key >> 32));
                                if (key == ~0ull || !(below_min || st.slope > low)) {
                                    if (lane == 0) sh_v = ND_NONE;
                                } else {
                                    // the job's state and what remembering it reads, together
                                    const int32_t gi0 = A.st.gi[who];
                                    const uint32_t ci0 = A.st.ci[who];
                                    const uint32_t so = A.X.tb.seg_off[who], ns = A.X.tb.seg_off[who + 1] - so;
                                    const uint32_t stamp = A.stamp[who];
                                    const float ds_c0 = A.ds_c[who];
                                    const uint32_t slot = (uint32_t)__ffsll((long long)__ballot(lane < c && rv == who)) - 1u;
                                    const uint32_t here_has = wave_lane_u32(word, slot) & 0xFFFFu;
                                    const float ds_g0 = __uint_as_float(wave_lane_u32(__float_as_uint(sl), slot));
                                    const uint32_t last = wave_lane_u32(word, c - 1u);
                                    const RsShrunk sk = rs_shrink_wave(A, who, so, ns, 0, gi0, ci0, lane);
                                    if (lane == 0) {
                                        if (stamp != sh_epoch) {     // (remember)
                                            A.stamp[who] = sh_epoch;
                                            A.keep_gi[who] = gi0; A.keep_ci[who] = ci0;
                                            A.keep_ds[2 * who] = ds_g0; A.keep_ds[2 * who + 1] = ds_c0;
                                            A.touched[sh_touched++] = who;
                                        }
                                        const uint32_t per_v = nd_cpl(A, ci0);
                                        const uint32_t here = (uint32_t)sk.gv.dg < here_has ? (uint32_t)sk.gv.dg : here_has;
                                        A.free_g[f] = free_g + here; A.free_c[f] = free_c + here * per_v;      // (nd_drop)
                                        if (here_has - here) A.res[base + slot] = (who << 16) | (here_has - here);
                                        else { A.res[base + slot] = last; A.cnt[f] = c - 1u; }
                                        sh_rest = (uint32_t)sk.gv.dg - here; sh_per_v = per_v; sh_v = who;
                                        sh_lost = sh_lost + sk.gv.loss;
                                        A.st.gi[who] = sk.gi; A.st.ci[who] = sk.ci;
                                        A.ds_g[who] = sk.ds_g; A.ds_c[who] = sk.ds_c;
                                        sh_shrinks += 1u;
                                    }
                                }
                            }
                        }
                        __syncthreads();
                        const uint32_t v = sh_v, rest = sh_rest, per_v = sh_per_v;
                        if (v == ND_NONE) break;
                        if (rest > 0) {                      // the rest from its other parts, the last one first
                            uint32_t k[ND_PER], local = 0;
#pragma unroll
                            for (uint32_t i = 0; i < ND_PER; ++i) {
                                const uint32_t r = tid * per_thread + i;     // position from the last node
                                k[i] = (i < per_thread && r < N && N - 1u - r != f) ? nd_part(A, N - 1u - r, v) : 0u;
                                local += k[i];
                            }
                            uint32_t all;
                            uint32_t running = block_scan(local, all);
#pragma unroll
                            for (uint32_t i = 0; i < ND_PER; ++i) {
                                if (k[i] && rest > running) {
                                    const uint32_t give = k[i] < rest - running ? k[i] : rest - running;
                                    nd_drop(A, N - 1u - (tid * per_thread + i), v, give, per_v);
                                }
                                running += k[i];
                            }
                            __syncthreads();
                        }
                        if (tid == 0) {
                            const uint32_t by_cpu = A.free_c[f] / per_gpu;
                            const uint32_t offer = A.free_g[f] < by_cpu ? A.free_g[f] : by_cpu;
                            const uint32_t t = offer < sh_lack ? offer : sh_lack;
                            if (t) nd_add(A, f, j, t, per_gpu);
                            sh_lack -= t;
                        }
                        __syncthreads();
                        if (sh_lack == 0) break;
                    }
                }
                n0 = sh_next;
                walking = sh_lack > 0;
                __syncthreads();
            }
            if (tid == 0) {
                bool ok = sh_ok != 0u && sh_lack == 0u;
                if (ok && !below_min && !(st.gain > sh_lost)) ok = false;
                if (!ok) put_jobs_back();
                else { A.st.gi[j] = st.tgt; A.st.ci[j] = st.lvl; sh_moves += 1u; }
                sh_go = ok ? 1u : 0u;
            }
            __syncthreads();
            const uint32_t go = sh_go;
            if (go) {
                const uint32_t n_changed = sh_touched + 1u;      // a wavefront per job whose state changed
                for (uint32_t i = wave; i < n_changed; i += ND_WAVES) refresh(i < sh_touched ? A.touched[i] : j);
            } else {
                restore_nodes();
            }
            __syncthreads();
            if (!go) break;
        }
        for (;;) {                                           // ---- CPUs: on every node the job is on
            if (tid == 0) { sh_step = nd_cached_step(A, j, 1); sh_lost = 0.f; sh_ok = 1u; sh_touched = 0u; sh_epoch += 1u; }
            __syncthreads();
            const RsStep st = sh_step;
            if (!st.any) { __syncthreads(); break; }
            const uint32_t more = nd_cpl(A, st.lvl) - nd_cpl(A, A.st.ci[j]);
            keep_nodes();
            {                                                // its parts, in node order
                uint32_t k[ND_PER], local = 0;
#pragma unroll
                for (uint32_t i = 0; i < ND_PER; ++i) {
                    const uint32_t n = tid * per_thread + i;
                    k[i] = (i < per_thread && n < N) ? nd_part(A, n, j) : 0u;
                    local += k[i] ? 1u : 0u;
                }
                uint32_t all;
                uint32_t at = block_scan(local, all);
#pragma unroll
                for (uint32_t i = 0; i < ND_PER; ++i)
                    if (k[i]) { A.plist[2 * at] = tid * per_thread + i; A.plist[2 * at + 1] = k[i]; ++at; }
                if (tid == 0) sh_np = all;
                __syncthreads();
            }
            const uint32_t np = sh_np;
            bool found = true;                               // every part so far has its CPUs
            for (uint32_t p = 0; p < np && found; ++p) {
                const uint32_t n = A.plist[2 * p], need = more * A.plist[2 * p + 1];
                for (;;) {
                    if (wave == 0) {                         // the first wavefront: its lanes share the job's step down
                        const uint32_t free_here = A.free_c[n];
                        if (free_here >= need) { if (lane == 0) { A.free_c[n] = free_here - need; sh_flag = 0u; } }
                        else {
                            uint32_t who;
                            const float low = nd_lowest_on_wave(A, n, j, A.ds_c, who, lane);
                            if (who == ND_NONE || !(st.slope > low)) { if (lane == 0) { sh_ok = 0u; sh_flag = 0u; } }
                            else {
                                const int32_t gi0 = A.st.gi[who];
                                const uint32_t ci0 = A.st.ci[who];
                                const uint32_t so = A.X.tb.seg_off[who], ns = A.X.tb.seg_off[who + 1] - so;
                                const RsShrunk sk = rs_shrink_wave(A, who, so, ns, 1, gi0, ci0, lane);
                                if (lane == 0) {
                                    remember(who);
                                    sh_per_v = nd_cpl(A, ci0) - nd_cpl(A, ci0 - 1u);
                                    sh_v = who; sh_flag = 1u;
                                    sh_lost = sh_lost + sk.gv.loss;
                                    A.st.ci[who] = sk.ci;
                                    A.ds_g[who] = sk.ds_g; A.ds_c[who] = sk.ds_c;
                                    sh_shrinks += 1u;
                                }
                            }
                        }
                    }
                    __syncthreads();
                    const uint32_t flag = sh_flag, v = sh_v, less = sh_per_v;
                    found = sh_ok != 0u;
                    if (flag)                                 // the job that gives a level gives it on all its nodes
                        for (uint32_t m = tid; m < N; m += ND_THREADS) A.free_c[m] += less * nd_part(A, m, v);
                    __syncthreads();
                    if (!flag) break;
                }
            }
            if (tid == 0) {
                bool ok = sh_ok != 0u;
                if (ok && !(st.gain > sh_lost)) ok = false;
                if (!ok) put_jobs_back();
                else { A.st.ci[j] = st.lvl; sh_moves += 1u; }
                sh_go = ok ? 1u : 0u;
            }
            __syncthreads();
            const uint32_t go = sh_go;
            if (go) {
                const uint32_t n_changed = sh_touched + 1u;      // a wavefront per job whose state changed
                for (uint32_t i = wave; i < n_changed; i += ND_WAVES) refresh(i < sh_touched ? A.touched[i] : j);
            } else {
                restore_nodes();
            }
            __syncthreads();
            if (!go) break;
        }
    };

    // ---- privileged jobs (below their floor) come first, in job order: their list (tmp_off serves as the list)
    uint32_t n_first = 0;
    for (uint32_t base = 0; base < J; base += ND_THREADS) {
        const uint32_t j = base + tid;
        const bool is = j < J && A.first[j] != 0u;
        uint32_t all;
        const uint32_t at = block_scan(is ? 1u : 0u, all);
        if (is) A.tmp_off[n_first + at] = j;
        n_first += all;
    }
    __syncthreads();
    // ---- then the others: their order is fixed once (when the privileged jobs are through), by GPU slope, then CPU
    // slope (both descending), then index.
    // Most jobs find nothing to do when their turn comes, and whether that is so follows from values that change
    // only when a step is committed.  A GPU step does nothing when there is none, or when what the nodes can give
    // a job at its level (GPUs with their CPUs) is less than the step needs and no job anywhere has a slope below
    // this job's (then nobody on any node may be shrunk).  A CPU step does nothing when there is none, or when no
    // job anywhere has a lower CPU slope and all free CPUs together are fewer than the step needs.  Passing over
    // such a job changes nothing, so the jobs are not sorted: all threads look for the first job in the order, after
    // the one served last, that is not of that kind; it is served in full and the search starts again.
    auto comes_before = [&](float ga, float ca, uint32_t a, float gb, float cb, uint32_t b) {
        return ga > gb || (ga == gb && (ca > cb || (ca == cb && a < b)));
    };
    float last_g = INF, last_c = INF;
    uint32_t last_j = 0u, moves_seen = ND_NONE, k_first = 0;
    bool others = false;
    for (;;) {                                               // one job per turn; ScheduleJob appears once in the code
        if (k_first < n_first) {
            schedule_job(A.tmp_off[k_first++]);
            continue;
        }
        if (!others) {
            for (uint32_t j = tid; j < J; j += ND_THREADS) {
                const bool in = rs_part(A, j) && !A.first[j];
                A.sg[j] = in ? A.ug[j] : -1.f;               // the cached slopes are current; -1: not in the list
                A.sc[j] = in ? A.uc[j] : -1.f;
            }
            others = true;
        }
        __syncthreads();
        const bool fresh = sh_moves != moves_seen;          // a step was committed since the last look (or this is the first)
        moves_seen = sh_moves;
        __syncthreads();
        if (fresh) {
            if (tid < RK_MAX_CPU_LEVELS) sh_take[tid] = 0ull;
            if (tid == 0) sh_free_c = 0ull;
            {
                RsMin two[2];
                rs_two_lowest<ND_WAVES, ND_THREADS>(sh_ds, J, tid, lane, wave, sh_two_k, sh_two_s, two);
                if (tid == 0) { sh_min[0] = two[0]; sh_min[1] = two[1]; }
            }
            {                                                    // what the nodes can give at every CPU level
                unsigned long long fc = 0;
                for (uint32_t n = tid; n < N; n += ND_THREADS) fc += A.free_c[n];
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) fc += __shfl_xor(fc, off, 64);
                if (lane == 0 && fc) atomicAdd(&sh_free_c, fc);
                for (uint32_t l = 0; l < A.X.grid.n_cpu; ++l) {
                    const uint32_t per_gpu = nd_cpl(A, l);
                    unsigned long long t = 0;
                    for (uint32_t n = tid; n < N; n += ND_THREADS) {
                        const uint32_t by_cpu = A.free_c[n] / per_gpu;
                        t += A.free_g[n] < by_cpu ? A.free_g[n] : by_cpu;
                    }
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
                    if (lane == 0 && t) atomicAdd(&sh_take[l], t);
                }
            }
        }
        __syncthreads();
        const RsMin mg = sh_min[0], mc = sh_min[1];
        const unsigned long long free_c = sh_free_c;
        float best_g = -1.f, best_c = -1.f;
        uint32_t best_j = ND_NONE;
        for (uint32_t j0 = tid; j0 < J; j0 += 4 * ND_THREADS) {          // four jobs' values in flight
            float kg[4], kc[4], ug[4], uc[4];
            uint32_t dg[4], lv[4];
            unsigned long long dc[4];
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const uint32_t j = j0 + k * ND_THREADS;
                const bool in = j < J;
                kg[k] = in ? A.sg[j] : -1.f; kc[k] = in ? A.sc[j] : -1.f;
                ug[k] = in ? A.ug[j] : 0.f; uc[k] = in ? A.uc[j] : 0.f;
                dg[k] = in ? A.udg[j] : 0u; lv[k] = in ? A.st.ci[j] : 0u; dc[k] = in ? A.udc_c[j] : 0ull;
            }
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const uint32_t j = j0 + k * ND_THREADS;
                if (kg[k] < 0.f || !comes_before(last_g, last_c, last_j, kg[k], kc[k], j)) continue;
                const float lowest_g = j == mg.i1 ? mg.m2 : mg.m1, lowest_c = j == mc.i1 ? mc.m2 : mc.m1;
                const bool gpu_idle = !(ug[k] > 0.f) || (sh_take[lv[k]] < dg[k] && !(ug[k] > lowest_g));
                const bool cpu_idle = !(uc[k] > 0.f) || (free_c < dc[k] && !(uc[k] > lowest_c));
                if (gpu_idle && cpu_idle) continue;
                if (best_j == ND_NONE || comes_before(kg[k], kc[k], j, best_g, best_c, best_j)) { best_g = kg[k]; best_c = kc[k]; best_j = j; }
            }
        }
        {                                                    // the first of the threads' candidates in the order
            const RsPick pick = rs_pick_first<ND_WAVES>(best_g, best_c, best_j, lane, wave, sh_pick_key, sh_pick_j);
            best_g = pick.g; best_c = pick.c; best_j = pick.j;
        }
        if (best_j == ND_NONE) break;
        if (tid == 0) sh_full += 1u;
        schedule_job(best_j);
        last_g = best_g; last_c = best_c; last_j = best_j;
    }
    __syncthreads();

    // ---- memory, then the records
    nd_finish<ND_THREADS>(A, A.np, A.tmp_off, A.tmp_parts, A.touched, A.res, sh_mem, sh_scan);
    if (tid == 0 && A.stats) { A.stats[0] = sh_moves; A.stats[1] = sh_full; A.stats[2] = sh_shrinks; A.stats[3] = sh_undone; A.stats[4] = 0u; }
}

}  // namespace

extern "C" int32_t rk_reschedule_nodes(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                       const rk_alloc_grid *grid, const rk_nodes *nodes, const float *best_thr,
                                       const uint32_t *best_plan, const float *curve_thr,
                                       const rk_job_state *jobs_state, const uint32_t *prev_off,
                                       const rk_place_entry *prev_entries, uint64_t n_prev_entries,
                                       rk_assign *assign, uint32_t *place_off,
                                       rk_place_entry *entries, uint64_t cap_entries, float *total, uint32_t *stats) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if ((rc = rk_check_table(ctx, table, 0, table ? table->n_jobs : 0))) return rc;
    if ((rc = rk_check_grid(ctx, grid))) return rc;
    if (!nodes || !total || !jobs_state || !place_off) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    const uint32_t J = table->n_jobs;
    if (J > 0 && (!ref_thr || !assign || !jobs_state->cur_seg || !jobs_state->cur_c ||
                  (table->n_segs > 0 && (!best_thr || !best_plan || !curve_thr))))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if ((prev_off == nullptr) != (prev_entries == nullptr))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "the earlier placement needs both its offsets and its entries");
    if (nodes->n_nodes == 0 || nodes->n_nodes > RK_MAX_NODES || nodes->gpus_per_node == 0 ||
        nodes->gpus_per_node > 65535u || nodes->cpus_per_node > 65535u || !(nodes->mem_per_node_gb >= 0.f))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "nodes: 1..%u nodes of 1..65535 GPUs, at most 65535 CPUs, memory >= 0", RK_MAX_NODES);
    if (grid->cpu_mode != 1u)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "the search over nodes needs CPU levels per GPU (cpu_mode 1)");
    const uint64_t gpus = (uint64_t)nodes->n_nodes * nodes->gpus_per_node;
    if (gpus > ND_MAX_GPUS) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%llu GPUs, the search over nodes takes up to %u", (unsigned long long)gpus, ND_MAX_GPUS);
    if (table->max_segs_per_job > 32767u) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 32767 segments per job");
    if (J > RK_MAX_JOBS_PER_ROUND)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u jobs, the allocation kernels take up to %u", J, RK_MAX_JOBS_PER_ROUND);
    if (cap_entries < gpus && J > 0) return rk_fail(ctx, RK_ERR_CAPACITY, "entries: %llu records, %llu may be needed", (unsigned long long)cap_entries, (unsigned long long)gpus);
    if (J > 0 && !entries) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    RK_HIP(ctx, hipSetDevice(ctx->device));
    return rk_launch_reschedule_nodes(ctx, ref_thr, table, grid, nodes, best_thr, best_plan, curve_thr, jobs_state, prev_off,
                                      prev_entries, n_prev_entries, assign, place_off, entries, total, stats);
}

// The kernels' argument, with the working memory it points to; *words: of the node tables.
static int32_t nd_kernel_args(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table, const rk_alloc_grid *grid,
                              const rk_nodes *nodes, const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                              const rk_job_state *jobs_state, const uint32_t *prev_off, const rk_place_entry *prev_entries,
                              uint64_t n_prev_entries, rk_assign *assign, uint32_t *place_off, rk_place_entry *entries,
                              float *total, uint32_t *stats, NdKernArgs &K) {
    const uint32_t J = table->n_jobs;
    const uint64_t gpus = (uint64_t)nodes->n_nodes * nodes->gpus_per_node;
    int32_t rc;
    const size_t n = J ? J : 1, N = nodes->n_nodes;
    const size_t nodes_words = nd_nodes_words(N, (size_t)gpus);
    uint32_t *w_nodes, *w_jobs;
    float *f_jobs;
    unsigned long long *u64;
    RsGives *gives;
    if ((rc = rk_scratch(ctx, SL_ND_GIVES, n * sizeof(RsGives), (void **)&gives))) return rc;
    if ((rc = rk_scratch(ctx, SL_ND_NODES, (2 * nodes_words + 2 * N + (size_t)gpus) * sizeof(uint32_t), (void **)&w_nodes))) return rc;
    if ((rc = rk_scratch(ctx, SL_ND_U32, (14 * n + 1) * sizeof(uint32_t), (void **)&w_jobs))) return rc;
    if ((rc = rk_scratch(ctx, SL_ND_F32, 10 * n * sizeof(float), (void **)&f_jobs))) return rc;
    if ((rc = rk_scratch(ctx, SL_ND_U64, 2 * n * sizeof(unsigned long long), (void **)&u64))) return rc;
    NdBody &A = K.b;
    K.X.ref_thr = ref_thr; K.X.tb = table_dev(table); K.X.grid = grid_dev(grid);
    K.X.best_thr = best_thr; K.X.best_plan = best_plan; K.X.curve_thr = curve_thr;
    A.G = gpus;
    A.n_jobs = J; A.n_nodes = nodes->n_nodes; A.gpn = nodes->gpus_per_node; A.cpn = nodes->cpus_per_node;
    A.mem_gb = nodes->mem_per_node_gb;
    A.state = jobs_state->state; A.cur_seg = jobs_state->cur_seg; A.cur_c = jobs_state->cur_c;
    A.floor_seg = jobs_state->floor_seg; A.floor_c = jobs_state->floor_c;
    A.prev_off = prev_off; A.prev_entries = prev_entries; A.n_prev = n_prev_entries;
    A.free_g = w_nodes; A.free_c = w_nodes + N; A.cnt = w_nodes + 2 * N; A.res = w_nodes + ((3 * N + 3) & ~(size_t)3);
    A.keep_nodes = w_nodes + nodes_words; A.nodes_words = (uint32_t)nodes_words;
    A.plist = w_nodes + 2 * nodes_words; A.tmp_parts = A.plist + 2 * N;
    A.st.gi = reinterpret_cast<int32_t *>(w_jobs); A.st.ci = w_jobs + n; A.udg = w_jobs + 2 * n; A.touched = w_jobs + 3 * n;
    A.stamp = w_jobs + 4 * n; A.first = w_jobs + 5 * n; A.keep_ci = w_jobs + 6 * n;
    A.keep_gi = reinterpret_cast<int32_t *>(w_jobs + 7 * n); A.np = w_jobs + 8 * n;
    A.tmp_off = w_jobs + 10 * n;                             // n + 1 words
    A.seg_off = table->seg_off;
    uint32_t *more = w_jobs + 11 * n + 1;
    A.tgt_g = reinterpret_cast<int32_t *>(more); A.lvl_g = more + n; A.lvl_c = more + 2 * n;
    A.ds_g = f_jobs; A.ds_c = f_jobs + n; A.ug = f_jobs + 2 * n; A.uc = f_jobs + 3 * n; A.sg = f_jobs + 4 * n;
    A.sc = f_jobs + 5 * n; A.keep_ds = f_jobs + 6 * n; A.gain_g = f_jobs + 8 * n; A.gain_c = f_jobs + 9 * n;
    A.udc_c = u64; A.okey = u64 + n;
    A.gives = gives; A.give = nullptr; A.give_c = nullptr;
    A.assign = assign; A.place_off = place_off; A.entries = entries; A.total = total; A.stats = stats;
    return RK_OK;
}

// Dynamic LDS of k_nodes_lds and k_sim_nodes may be all of it: once per context.
static int32_t nd_raise_lds(rk_ctx *ctx) {
    if (ctx->nodes_lds_raised) return RK_OK;
    const auto most = hipFuncAttributeMaxDynamicSharedMemorySize;
    const void *const fs[] = {reinterpret_cast<const void *>(k_nodes_lds<ND_SMALL_THREADS, true>), reinterpret_cast<const void *>(k_nodes_lds<ND_FEW_THREADS, true>),
                              reinterpret_cast<const void *>(k_nodes_lds<ND_THREADS, false>), reinterpret_cast<const void *>(k_sim_nodes<ND_SMALL_THREADS, false, 0u>),
                              reinterpret_cast<const void *>(k_sim_nodes<ND_FEW_THREADS, false, 0u>), reinterpret_cast<const void *>(k_sim_nodes<ND_THREADS, true, 0u>),
                              reinterpret_cast<const void *>(k_sim_nodes<ND_SMALL_THREADS, true, 0u>), reinterpret_cast<const void *>(k_sim_nodes<ND_FEW_THREADS, true, 0u>),
                              reinterpret_cast<const void *>(k_sim_nodes<ND_THREADS, true, 8u>), reinterpret_cast<const void *>(k_sim_nodes<ND_SMALL_THREADS, true, 8u>),
                              reinterpret_cast<const void *>(k_sim_nodes<ND_FEW_THREADS, true, 8u>)};
    for (const void *f : fs) RK_HIP(ctx, hipFuncSetAttribute(f, most, (int)ND_LDS_MOST));
    RK_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(k_reschedule_nodes), most, 2 * RK_MAX_JOBS_PER_ROUND * sizeof(float)));
    ctx->nodes_lds_raised = true;
    return RK_OK;
}

int32_t rk_launch_reschedule_nodes(rk_ctx *ctx, const float *ref_thr, const rk_plan_table *table,
                                   const rk_alloc_grid *grid, const rk_nodes *nodes, const float *best_thr,
                                   const uint32_t *best_plan, const float *curve_thr, const rk_job_state *jobs_state,
                                   const uint32_t *prev_off, const rk_place_entry *prev_entries, uint64_t n_prev_entries,
                                   rk_assign *assign, uint32_t *place_off, rk_place_entry *entries, float *total,
                                   uint32_t *stats) {
    NdKernArgs K;
    NdBody &A = K.b;
    int32_t rc;
    if ((rc = nd_kernel_args(ctx, ref_thr, table, grid, nodes, best_thr, best_plan, curve_thr, jobs_state, prev_off, prev_entries,
                             n_prev_entries, assign, place_off, entries, total, stats, K))) return rc;
    if ((rc = nd_raise_lds(ctx))) return rc;
    const size_t J = A.n_jobs, n = J ? J : 1, N = A.n_nodes, nodes_words = A.nodes_words;
    // Where the nodes and their copy fit a CU's LDS beside the cached slopes (512 nodes of 8 GPUs and 10,000 jobs do), the
    // loop runs on them there.
    const size_t lds_lj = nd_lds_words(J, N, nodes_words, true) * sizeof(uint32_t), lds_l = nd_lds_words(J, N, nodes_words, false) * sizeof(uint32_t);
    const bool in_lds = A.gpn <= 64u && lds_l <= ND_LDS_MOST, jobs_too = in_lds && lds_lj <= ND_LDS_MOST;
    A.book = !in_lds;
    if (A.book) {
        k_nd_init<<<(uint32_t)((N + 255) / 256), 256, 0, ctx->stream>>>(K);
        RK_CHECK_LAUNCH(ctx, "k_nd_init");
    }
    if (J > 0) {
        k_nd_prepare<<<(uint32_t)((J + 3) / 4), 256, 0, ctx->stream>>>(K);
        RK_CHECK_LAUNCH(ctx, "k_nd_prepare");
    }
    if (jobs_too && J <= ND_FEW_THREADS) k_nodes_lds<ND_FEW_THREADS, true><<<1, ND_FEW_THREADS, lds_lj, ctx->stream>>>(K);
    else if (jobs_too) k_nodes_lds<ND_SMALL_THREADS, true><<<1, ND_SMALL_THREADS, lds_lj, ctx->stream>>>(K);
    else if (in_lds) k_nodes_lds<ND_THREADS, false><<<1, ND_THREADS, lds_l, ctx->stream>>>(K);
    else k_reschedule_nodes<<<1, ND_THREADS, (size_t)2 * n * sizeof(float), ctx->stream>>>(K);           // at most 96 KiB
    RK_CHECK_LAUNCH(ctx, "k_nodes_lds");
    return RK_OK;
}

// Ticks of a simulation whose rounds search node by node, from the one that *A.tick says (k_sim_init and k_sim_step have
// opened it): enough launches on the context's stream for all of them, a launch past the last tick returns at once.
constexpr uint32_t SIM_NODES_ROUNDS = 64;        // rounds of a launch
constexpr uint64_t ND_STATES_MOST = 1u << 19;    // states of all jobs that are found beforehand (80 bytes each)
constexpr uint32_t ND_STATES_PER_TICK = 65536;   // ... that a tick pays for
constexpr uint32_t ND_STATES_NODES_WORDS = 5632; // ... words of the nodes' tables that one wavefront copies no slower than all

bool rk_sim_nodes_fit(uint32_t n_jobs, const rk_nodes *nodes) {
    const size_t N = nodes->n_nodes, gpus = N * nodes->gpus_per_node;
    return n_jobs > 0 && nodes->gpus_per_node <= 64u &&
           nd_lds_words(n_jobs, N, nd_nodes_words(N, gpus), true, true) * sizeof(uint32_t) <= ND_LDS_MOST;
}

int32_t rk_launch_sim_nodes(rk_ctx *ctx, const SimArgs &S, const float *ref_thr, const rk_plan_table *table, const rk_alloc_grid *grid,
                            const rk_nodes *nodes, const float *best_thr, const uint32_t *best_plan, const float *curve_thr,
                            uint64_t cap_parts, rk_assign *assign) {
    NdSimArgs K;
    int32_t rc;
    const rk_job_state held = {S.F.state, S.S.seg, S.S.lvl, nullptr, nullptr};
    if ((rc = nd_kernel_args(ctx, ref_thr, table, grid, nodes, best_thr, best_plan, curve_thr, &held, S.at_off, S.at_ent, cap_parts,
                             assign, S.now_off, S.now_ent, S.tick_total, nullptr, K))) return rc;
    if ((rc = nd_raise_lds(ctx))) return rc;
    K.S = S;
    K.rounds = SIM_NODES_ROUNDS;
    K.b.book = false;
    const uint32_t J = K.b.n_jobs;
    const size_t N = K.b.n_nodes, gpus = N * K.b.gpn;
    size_t lds = nd_lds_words(J, N, K.b.nodes_words, true, true) * sizeof(uint32_t);
    const NdKernArgs prepare = K;
    // With a job per thread, all states of the jobs are found beforehand where they are not too many for memory and for the
    // ticks: 0.4 us per 1,000 states, and a round is at least 25 us shorter (a simulation of one tick may have nothing to do: 42
    // and 55 us; two ticks of 300 jobs on 64 GPUs 214 and 131, of 900 on 1,024 GPUs, 207,000 states, 5.86 and 4.40 ms).
    // One wavefront copies the nodes' tables and looks through the residents, which costs it more the more of them there are:
    // 24 ticks of 100, 300 and 500 jobs on 256 nodes of 8 GPUs 5.8 and 4.7, 19.3 and 14.9, 25.9 and 20.0 ms, on 512 (5,632 words) 8.2 and
    // 7.7, 22.3 and 19.7, 36.2 and 31.9; 12 ticks of 60 and 250 jobs on 256 nodes of 16 (4,864) 2.87 and 2.74, 8.31 and 8.03, on 1,024 of 2
    // (5,120) 5.67 and 5.62, 12.5 and 12.0, on 768 of 5 (6,144) 4.90 and 5.08, 13.6 and 13.7, on 1,024 of 4 (7,168) 4.59 and 4.92, 12.8
    // and 13.0, on 2,048 of 1 (8,192) 13.8 and 13.6, 22.2 and 22.5, of 500 jobs there 21.8 and 22.8.
    const uint64_t per_job = ((uint64_t)table->max_segs_per_job + 1u) * grid->n_cpu, states = J * per_job;
    const uint32_t threads = J <= ND_FEW_THREADS ? ND_FEW_THREADS : J <= ND_SMALL_THREADS ? ND_SMALL_THREADS : ND_THREADS;
    const size_t lds_tab = nd_tab_words(threads, N, gpus, K.b.nodes_words) * sizeof(uint32_t);
    const bool tab = J <= ND_THREADS && K.b.nodes_words <= ND_STATES_NODES_WORDS && lds_tab <= ND_LDS_MOST && states <= ND_STATES_MOST && S.n_ticks > 1u && states <= (uint64_t)ND_STATES_PER_TICK * S.n_ticks;
    const bool eight = K.b.gpn == 8u;
    if (tab) {
        lds = lds_tab;
        char *mem;
        if ((rc = rk_scratch(ctx, SL_ND_STATES, states * (ND_STATE_WORDS * sizeof(uint32_t) + sizeof(uint4)), (void **)&mem))) return rc;
        K.states.words = reinterpret_cast<uint32_t *>(mem);
        K.states.best = reinterpret_cast<uint4 *>(mem + states * ND_STATE_WORDS * sizeof(uint32_t));
        K.states.per_job = (uint32_t)per_job;
        K.shares = nd_share_words(N, gpus) ? 1u : 0u;
        NdKernArgs all = prepare;
        all.b.state = nullptr;                               // (as if everybody took part)
        k_nd_states<<<dim3(J, grid->n_cpu), 256, 0, ctx->stream>>>(all, K.states);
        RK_CHECK_LAUNCH(ctx, "k_nd_states");
    }
    for (uint32_t t = 0; t < S.n_ticks; t = S.n_ticks - t > SIM_NODES_ROUNDS ? t + SIM_NODES_ROUNDS : S.n_ticks) {
        k_nd_prepare<<<(J + 3) / 4, 256, 0, ctx->stream>>>(prepare);
        RK_CHECK_LAUNCH(ctx, "k_nd_prepare");
        if (tab && threads == ND_THREADS) { if (eight) k_sim_nodes<ND_THREADS, true, 8u><<<1, ND_THREADS, lds, ctx->stream>>>(K); else k_sim_nodes<ND_THREADS, true, 0u><<<1, ND_THREADS, lds, ctx->stream>>>(K); }
        else if (tab && threads == ND_SMALL_THREADS) { if (eight) k_sim_nodes<ND_SMALL_THREADS, true, 8u><<<1, ND_SMALL_THREADS, lds, ctx->stream>>>(K); else k_sim_nodes<ND_SMALL_THREADS, true, 0u><<<1, ND_SMALL_THREADS, lds, ctx->stream>>>(K); }
        else if (tab) { if (eight) k_sim_nodes<ND_FEW_THREADS, true, 8u><<<1, ND_FEW_THREADS, lds, ctx->stream>>>(K); else k_sim_nodes<ND_FEW_THREADS, true, 0u><<<1, ND_FEW_THREADS, lds, ctx->stream>>>(K); }
        else if (J <= ND_FEW_THREADS) k_sim_nodes<ND_FEW_THREADS, false, 0u><<<1, ND_FEW_THREADS, lds, ctx->stream>>>(K);
        else k_sim_nodes<ND_SMALL_THREADS, false, 0u><<<1, ND_SMALL_THREADS, lds, ctx->stream>>>(K);
        RK_CHECK_LAUNCH(ctx, "k_sim_nodes");
    }
    return RK_OK;
}
