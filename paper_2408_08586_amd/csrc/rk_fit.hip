// Model fitting (paper Sec. 4, "Continuous model fitting"): the seven
// fittable parameters of every model type are chosen to minimise the root mean
// squared logarithmic error between Eq. 1 and measured runs.
//
// The work is a set of descents: one from every starting point of every model,
// then those that move an exponent off its bound.  A wavefront holds 64/W
// descents at a time (W = 16..64, the smallest power of two that holds a
// model's runs), a group of W lanes each.  One iteration evaluates a run's
// residual and its seven derivatives (analytic) per lane, sums the normal
// equations over the group, and solves the 7x7 system with a matrix row per
// lane.  A descent that ends is replaced at once by the next one of the
// wavefront's models, so no lane waits for the slowest descent of its
// wavefront.  float64 throughout.
#include <utility>

#include "rk_internal.h"
#include "rk_model.h"

namespace {

constexpr int FIT_THREADS = 256;
constexpr int NP = RK_FIT_PARAMS;
enum { TH_BWD, TH_SYNC, TH_OPT, TH_OPT_OFF, TH_OFF, TH_SWAP, TH_CONST };

struct FitArgs {
    JobDev jobs;
    rk_env env;
    uint32_t n_fits;
    const uint32_t *sample_off, *triple, *option, *cpus;
    const float *thr;
    uint32_t max_iter, n_starts;
    uint32_t most_runs;          // a model with more runs than this is left alone
    double refit_threshold;
    double offsets[RK_FIT_MAX_STARTS][NP];
    rk_fit_result out;
    uint32_t *next_model;        // the next model nobody has taken yet (starts at 0)
};

// Overlap of two stages (Sec. 4.3), (x^k + y^k)^(1/k) as M*(1 + r^k)^(1/k) with
// r = min/max, with its derivatives by the first argument and by k.
__device__ __forceinline__ void overlap(double k, double x, double y, double &f, double &fx, double &fk) {
    const double M = fmax(x, y), m = fmin(x, y);
    if (!(m > 0.0)) { f = M; fx = x >= y ? 1.0 : 0.0; fk = 0.0; return; }
    const double r = m / M, lr = log(r);
    const double rk = exp(k * lr);
    const double L = log1p(rk);
    f = M * exp(L / k);
    const double g = exp(L * (1.0 / k - 1.0));            // derivative by the larger argument
    fx = x >= y ? g : g * rk / r;
    fk = f * (rk * lr / ((1.0 + rk) * k) - L / (k * k));
}

// What a run contributes that does not depend on the parameters.
struct Run {
    double Tfwd, gc, aTfwd, am1, Tdp, Tconst, opt_scale, Toff, logy, b;
    bool off, valid;
};

__device__ Run load_run(const FitArgs &A, uint32_t j, uint32_t i) {
    Run R = {};
    const uint32_t packed = A.triple[i], o = A.option[i], c = A.cpus[i];
    const double d = RK_TRIPLE_D(packed), t = RK_TRIPLE_T(packed), p = RK_TRIPLE_P(packed);
    const uint32_t di = RK_TRIPLE_D(packed), ti = RK_TRIPLE_T(packed), pi = RK_TRIPLE_P(packed);
    const uint32_t z = o >> 2, gc = (o >> 1) & 1u, off = o & 1u;
    const uint32_t layers = A.jobs.layers[j], gb = A.jobs.gbatch[j], mu = A.jobs.mbatch[j] << RK_TRIPLE_V(packed);
    R.logy = log1p((double)A.thr[i]);
    R.valid = di > 0 && pi > 0 && o < 16u && mu > 0 && gb % (di * mu) == 0 && layers % pi == 0 && !(off && z < 2) &&
              !(off && c == 0);
    if (!R.valid) return R;
    const double P = A.jobs.P_bytes[j], s = A.jobs.seq[j], h = A.jobs.hidden[j], eb = A.jobs.elem_bytes[j];
    const double tfs = A.jobs.t_fwd_sample[j], b = gb, l = layers;
    const double n = (double)(gb / (di * mu));
    const bool pp = pi > 1;
    const double m = pp ? n : 1.0, a = pp ? 1.0 : n;
    R.b = b;
    R.Tfwd = tfs * mu / (t * p) * (m + p - 1.0);
    R.gc = gc;
    R.aTfwd = a * R.Tfwd;
    R.am1 = pp ? 0.0 : a - 1.0;
    const uint32_t N = A.env.gpus_per_node;
    const double bi = A.env.B_intra, bx = A.env.B_inter;
    double Bdp = bi, Btp = bi, Bpp = bi;
    if ((unsigned long long)di * ti * pi > N) {
        Btp = (N % ti == 0) ? bi : bx;
        Bdp = (N % ((unsigned long long)ti * di) == 0) ? bi : bx;
        Bpp = bx;
    }
    const double Vdp = di > 1 ? P * 2.0 * (d - 1.0) / (d * t * p) : 0.0;
    const double Vtp = ti > 1 ? eb * 4.0 * 2.0 * (t - 1.0) * b * s * h * l / (d * t) : 0.0;
    const double Vpp = pp ? eb * 2.0 * p * b * s * h / (d * t) : 0.0;
    R.Tdp = Vdp / Bdp;
    R.Tconst = Vtp / Btp + (pp ? Vpp / Bpp : 0.0);
    const double Psi = P / (t * p);
    R.off = off != 0;
    R.opt_scale = off ? Psi / (d * (double)c) : Psi / (z >= 1 ? d : 1.0);
    R.Toff = Psi / (d * (double)A.env.B_pcie);
    return R;
}

// One overlap of a run: of the backward pass with the synchronisation (every run), or, of an offloaded run, of the
// synchronisation with the offload or of the optimizer with the swapping.  The first argument is x[var]*a + b, the second
// y, the exponent 1/x[exp].
struct Task { double a, b, y; uint32_t var, exp; };
struct Overlap { double f, fx, fk, k; };

// The sums over a group of W lanes.  Partners inside a row of 16 lanes are reached by data-parallel-primitive moves
// (neighbour, neighbour pair, mirrored halves of 8, mirrored halves of 16), beyond it by shuffles; all 64 lanes must be
// active.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    const uint32_t l2 = (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, CTRL, 0xF, 0xF, false);
    const uint32_t h2 = (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, CTRL, 0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)h2 << 32) | l2));
}

// Normal equations of a group: the products of (J, r) with itself summed over the runs, a symmetric 8x8 matrix in LDS
// (J^T J in rows and columns 0..6, J^T r in row and column 7, r^T r in the corner), so that the lane that holds row i
// of the system reads its eight values in a piece.
constexpr int NR = NP + 1, N_SUM = NR * (NR + 1) / 2;

// One halving of N values over the pairs of lanes that CTRL exchanges: the lane whose `upper` is set keeps the sums of
// the upper values, its partner those of the lower.
template <int CTRL, int N>
__device__ __forceinline__ void halve(double (&v)[N_SUM], bool upper) {
    constexpr int H = (N + 1) / 2;
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double lo = v[i], hi = H + i < N ? v[H + i] : 0.0;
        v[i] = (upper ? hi : lo) + dpp_f64<CTRL>(upper ? lo : hi);
    }
}

// Sums the N_SUM products of every lane over its group of W lanes; a lane ends with up to three sums.  Every halving
// adds the same pairs as a sum of all values in all lanes would (both partners of such a step add the same two numbers),
// with 35 additions per lane instead of 36 for each of the log2 W steps; which half a lane keeps is chosen so that the
// mirrored partners of the later steps hold the same values.
template <int W>
__device__ __forceinline__ void group_sums(double (&v)[N_SUM], uint32_t lane) {
    const uint32_t b0 = lane & 1u, b1 = (lane >> 1) & 1u, b2 = (lane >> 2) & 1u, b3 = (lane >> 3) & 1u;
    halve<0xB1, 36>(v, b0 != b2);                           // quad_perm [1,0,3,2]
    halve<0x4E, 18>(v, b1 != b2);                           // quad_perm [2,3,0,1]
    halve<0x141, 9>(v, b2 != b3);                           // row_half_mirror
    halve<0x140, 5>(v, b3 != 0u);                           // row_mirror
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int off = 16; off < W; off <<= 1) v[i] += __shfl_xor(v[i], off, 64);
}

// where in the 8x8 matrix the lane's sum i = 0..2 belongs (row*8 + column | column*8 + row << 8), 0xFFFF: it has none
__device__ __forceinline__ uint32_t sum_place(uint32_t lane, uint32_t i) {
    const uint32_t b0 = lane & 1u, b1 = (lane >> 1) & 1u, b2 = (lane >> 2) & 1u, b3 = (lane >> 3) & 1u;
    const uint32_t k = (b3 ? 3u : 0u) + i;                  // among the four or five after the third halving
    if (k >= (b2 != b3 ? 4u : 5u)) return 0xFFFFu;
    uint32_t at = (b0 != b2 ? 18u : 0u) + (b1 != b2 ? 9u : 0u) + (b2 != b3 ? 5u : 0u) + k, r = 0;
    for (; at >= NR - r; ++r) at -= NR - r;                 // row r of the upper triangle has NR - r entries
    const uint32_t c = r + at;
    return (r * NR + c) | (c * NR + r) << 8;
}

// a value of lane N of every row of 16 lanes, in all lanes of the row
template <int N>
__device__ __forceinline__ double row_value(double v) { return dpp_f64<0x150 + N>(v); }   // row_newbcast

template <int... I, class F>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void for_each_index(F f) { unrolled(std::make_integer_sequence<int, N>{}, f); }

// Cholesky factorisation of the 7x7 system and its solution, by the lanes of a row of 16: lane i = 0..6 holds row i of
// the matrix in M (entries above the diagonal are ignored), lane 7 the right-hand side, which the factorisation turns
// into the forward solution; lanes 8..15 repeat lanes 0..7.  Every entry sees the operations of the row-by-row
// definition in their order.  delta is the same in all lanes; false when the matrix is not positive definite.
__device__ __forceinline__ bool solve_rows(double (&M)[NP], double (&delta)[NP]) {
    bool ok = true;
    double piv[NP];
    for_each_index<NP>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const double s = row_value<j>(M[j]);
        ok = ok && s > 0.0 && isfinite(s);
        piv[j] = sqrt(s > 0.0 ? s : 1.0);
        M[j] = M[j] / piv[j];
        for_each_index<NP - 1 - j>([&](auto cc) {
            constexpr int c = j + 1 + decltype(cc)::value;
            M[c] -= M[j] * row_value<c>(M[j]);
        });
    });
    for_each_index<NP>([&](auto ic) {                      // backward
        constexpr int i = NP - 1 - decltype(ic)::value;
        double v = row_value<NP>(M[i]);
        for_each_index<NP - 1 - i>([&](auto kc) {
            constexpr int k = i + 1 + decltype(kc)::value;
            v -= row_value<k>(M[i]) * delta[k];
        });
        delta[i] = v / piv[i];
    });
#pragma unroll
    for (int i = 0; i < NP; ++i) ok = ok && isfinite(delta[i]);
    return ok;
}

// The kernel's arguments for code that runs rarely: read where they are needed (the compiler would otherwise keep all of
// them in scalar registers from the start, more than there are).
__device__ __forceinline__ const FitArgs &cold_args() {
    auto p = (const FitArgs __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const FitArgs *)p;
}

// An exponent's kick is known by the version of the best point it starts from: what it ends with is kept, and the kicks
// of a model are gone through in order with what is known.
struct Rec {
    double x[NR], F, F0;                                  // the best point, its error; the error of the model's parameters
    double kick_x[3][NR], kick_F[3];                      // per exponent: where its last kick ended,
    uint32_t kick_iters[3], kick_of[3];                   // after how many iterations, from which version of the best point
    uint32_t model, start, iters, done;                   // `start`: the start the best point is from; `done`: starts that have ended
    uint32_t phase, version;                              // PHASE_STARTS, the kick that decides next (0..5), PHASE_DONE; of x, from 1
    uint32_t running, bound;                              // exponents whose kick from this version is under way; those on a bound
    uint32_t improved;
};
enum : uint32_t { PHASE_STARTS = 0xFFFFFFFEu, PHASE_DONE = 0xFFFFFFFFu };

// What a slot's next evaluation is for.
enum { SLOT_IDLE, SLOT_CURRENT, SLOT_START, SLOT_TRIAL };   // nothing; the current parameters; a descent's first point; a step

// A wavefront has 64/W slots with a descent under way in each.  A model's descents from its starting points are items of
// their own (the slots take them in order); the slot that finishes a model's last one goes on with its kicks, which build
// on one another.  When no model is left, slots without an item make kicks ahead from the best point there is; they count
// if that point is still the best one when their turn comes.  What belongs to a slot as a whole is held by all lanes of its
// group alike; lane i = 0..6 of every row of 16 (and lane 8 + i) also has component i of the vectors.  Nothing is shared
// between wavefronts but the number of the next model.
//
// Bound: the dependent float64 instructions of an iteration (about 2,700 for a wavefront of four slots, 7 us), first in
// number, then, when the models run out, in the longest chain of descents.  10,000 models x 16 runs, 5 starting points:
// 26.0 ms with a group per model whose 16 lanes all solved the same 7x7 system and which waited, descent by descent, for
// the slowest of the four models of its wavefront (850 iterations where a model needs 361 on average); 12.7 ms with the
// solutions taken by one wavefront for all slots of a workgroup, a lane each, between two barriers; 9.6 ms with the
// matrix rows spread over the group's lanes and no barrier at all; 9.0 ms with the overlaps dealt out to the lanes.
// 20 models: 8.1 -> 3.4 ms.  Kicks that would repeat an earlier one are not made again: 9.1 -> 8.5 ms; kicks made ahead
// by slots that have nothing else left: 8.3 ms, 20 models (other ones) 4.3 -> 3.1 ms.  Limiting the registers to three
// wavefronts per SIMD spills: 12.1 ms.
template <int W>
__global__ __launch_bounds__(FIT_THREADS, 2) void k_fit(FitArgs A) {
    constexpr double GTOL = 1e-14, XTOL = 1e-13, KICK_TO = 0.3;
    constexpr uint32_t WAVES = FIT_THREADS / 64, SLOTS = 64 / W, RECS = SLOTS + 1, NONE = 0xFFFFFFFFu;
    // per slot: the sums where the descent is and at the point evaluated, and that point; [64] takes what has no place
    __shared__ __align__(16) double sh_sums[WAVES][SLOTS][2][NR * NR + 2];
    __shared__ __align__(16) double sh_point[WAVES][SLOTS][NR];
    // per slot: the overlaps of the model's runs (at most three each), and the results of those of the offload
    __shared__ __align__(16) Task sh_task[WAVES][SLOTS][3 * W];
    __shared__ __align__(16) Overlap sh_over[WAVES][SLOTS][2 * W];
    // models under way: the best end point among the starting points, then among the kicks
    __shared__ Rec sh_rec[WAVES][RECS];

    const uint32_t wave = threadIdx.x >> 6, wlane = threadIdx.x & 63u, slot = wlane / W, lane = wlane % W;
    const uint32_t own = wlane & 7u;                      // the component (7: the right-hand side) this lane has
    const uint32_t row0 = wlane & ~15u;                   // first lane of this lane's row of 16
    double(*sums)[NR * NR + 2] = sh_sums[wave][slot];
    double *point = sh_point[wave][slot];
    Task *task = sh_task[wave][slot];
    Overlap *over = sh_over[wave][slot];
    uint32_t place[3];
#pragma unroll
    for (uint32_t i = 0; i < 3; ++i) {
        const uint32_t p = sum_place(wlane, i);
        place[i] = p == 0xFFFFu ? (uint32_t)(NR * NR) | (uint32_t)(NR * NR) << 8 : p;
    }
    const bool exponent = own == TH_SYNC || own == TH_OFF || own == TH_SWAP;
    const double lower = exponent ? 1.0 / RK_FIT_K_MAX : 0.0, upper = exponent ? 1.0 : __builtin_huge_val();

    Run R = {};
    bool has_run = false;
    uint32_t n_runs = 0, n_tasks = 0, off_rank = 0;       // of the slot's model; which of its offloaded runs the lane's is
    uint32_t state = SLOT_IDLE, model = NONE, start = 0, rec = 0, it = 0, iters = 0, into = 0;
    uint32_t kick = NONE, version = 0;                    // NONE: a descent from a starting point; 0..2: the kick of that exponent, from that version
    double lam = 0.0, nu = 0.0, pred = 0.0, F = 0.0, F0 = 0.0;
    bool ok = false, refit = false, want_item = true, opening = true;
    double x = 0.0, xn = 0.0, D = 0.0;                    // component `own` of the point, the point evaluated, the scaling
    // where the next items come from, the same in all lanes: a model, its next starting point, its record
    uint32_t src_model = NONE, src_start = NONE, src_rec = 0, free_recs = (1u << RECS) - 1u;
    bool src_dry = false;
    if (wlane < RECS) sh_rec[wave][wlane].phase = PHASE_DONE;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

    // the lane's component of the model's current parameters on the feasible set, and as a search point (exponents as 1/k)
    auto current = [&](const FitArgs &C, uint32_t m, double &th, double &sx) {
        const float *const src[NP] = {C.jobs.k_bwd, C.jobs.k_sync, C.jobs.k_opt, C.jobs.k_opt_off, C.jobs.k_off, C.jobs.k_swap, C.jobs.k_const};
        const float *from = src[0];
#pragma unroll
        for (int i = 1; i < NP; ++i) from = own == (uint32_t)i ? src[i] : from;
        const double v = from[m];
        th = exponent ? fmin(fmax(v, 1.0), RK_FIT_K_MAX) : fmax(v, 0.0);
        if (!(th == th)) th = exponent ? 1.0 : 0.0;       // NaN in the descriptor
        sx = exponent ? 1.0 / th : th;
    };
    auto clipped = [&](double v) { return fmin(fmax(v, lower), upper); };

    for (;;) {
        bool ended = false, step = false;                 // the descent has come to its end; it takes a step
        if (!opening && state != SLOT_IDLE) {
            const double F_t = sums[into][NR * NR - 1];
            bool first = state == SLOT_START;             // a descent's first point has been evaluated
            if (state == SLOT_CURRENT) {
                const FitArgs &C = cold_args();
                const uint32_t S = C.sample_off[model + 1] - C.sample_off[model];
                F0 = F_t;
                F = F0;
                refit = S > 0 && S <= C.most_runs && sqrt(F0 * (S ? 1.0 / (double)S : 0.0)) > C.refit_threshold;
                if (!refit) {
                    ended = true;
                } else if (start == 0) {
                    first = true;                         // the first descent begins where the parameters are
                } else {
                    xn = clipped(xn * exp(C.offsets[start - 1][own < NP ? own : 0]));
                    state = SLOT_START;
                }
            }
            if (first) {
                F = F_t;
                into ^= 1u;                               // the sums just made are those of the descent's point
                x = xn;
                D = sums[into ^ 1u][own * NR + own];
                lam = 1e-3;
                nu = 2.0;
                it = 0;
                step = A.max_iter > 0;
                ended = !step;
            } else if (state == SLOT_TRIAL) {
                bool active = true;
                if (ok && F_t < F && pred > 0.0) {
                    const double rho = (F - F_t) / pred, q = 2.0 * rho - 1.0;
                    lam = fmax(lam * fmax(1.0 / 3.0, 1.0 - q * q * q), 1e-15);
                    nu = 2.0;
                    x = xn;
                    F = F_t;
                    into ^= 1u;
                } else {
                    lam *= nu;
                    nu *= 2.0;
                    if (lam > 1e20) active = false;
                }
                ++it;
                step = active && it < A.max_iter;
                ended = !step;
            }
        }
        if (step) {
            ++iters;
            const double *cur = sums[into ^ 1u];
            double row[NR], M[NP], delta[NP];
#pragma unroll
            for (int j = 0; j < NR; ++j) row[j] = cur[own * NR + j];
            D = fmax(D, cur[own * NR + own]);
            const double g = row[NP], root = sqrt(fmax(D, 0.0)), scale = fmax(sqrt(F), 1e-300);
            const bool part = own < (uint32_t)NP;         // a component, not the right-hand side
            const bool fixed = part && ((x <= lower && g > 0.0) || (x >= upper && g < 0.0) || !(D > 0.0));
            const uint32_t fixed_all = (uint32_t)(__ballot(fixed) >> row0) & 0x7Fu;
            // converged: no free component's |g| / sqrt(D) is above the tolerance
            const bool converged = ((__ballot(part && !fixed && fabs(g) / root > GTOL * scale) >> row0) & 0x7Full) == 0ull;
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const bool on = own == (uint32_t)j;
                M[j] = (fixed || (fixed_all >> j & 1u)) ? (on ? 1.0 : 0.0) : !part ? -row[j] : on ? row[j] + lam * D : row[j];
            }
            ok = solve_rows(M, delta);
            double mine = delta[0];
#pragma unroll
            for (int i = 1; i < NP; ++i) mine = own == (uint32_t)i ? delta[i] : mine;
            xn = ok && part ? clipped(x + mine) : x;
            const double de = xn - x;
            const bool small = ok && ((__ballot(part && fabs(de) * root > XTOL * scale) >> row0) & 0x7Full) == 0ull;
            // what the quadratic model says the step gains
            double Ad = 0.0;
            for_each_index<NP>([&](auto jc) { Ad += row[decltype(jc)::value] * row_value<decltype(jc)::value>(de); });
            const double term = de * (2.0 * g + Ad);
            pred = 0.0;
            for_each_index<NP>([&](auto ic) { pred -= row_value<decltype(ic)::value>(term); });
            ended = converged || small;
            state = SLOT_TRIAL;
        }
        // without further models a kick whose model's best point has moved meanwhile is given up at once
        if (src_dry && kick != NONE && state != SLOT_IDLE) ended = ended || version != sh_rec[wave][rec].version;
        // Descents that have ended.  From a starting point: the model's best so far (the lowest error, the earlier start on
        // ties).  The slot that ends the last of them, or a kick, goes through the kicks as far as they are known.
        uint32_t freed = NONE;                            // the record of a model that is finished
        const unsigned long long any_ended = __ballot(ended);
        for (unsigned long long todo = any_ended; todo;) {
            const uint32_t who = ((uint32_t)__ffsll((long long)todo) - 1u) / W;
            if (slot == who) {
                Rec &m = sh_rec[wave][rec];
                bool decide = false;
                want_item = true;
                if (kick != NONE) {
                    decide = version == m.version;
                    if (decide) {
                        m.kick_x[kick][own] = x;
                        m.kick_F[kick] = F;
                        m.kick_iters[kick] = iters;
                        m.kick_of[kick] = version;
                    }
                } else {
                    if (refit) {
                        if (F < m.F || (F == m.F && start < m.start)) {
                            m.x[own] = x;
                            m.F = F;
                            m.start = start;
                        }
                        m.iters += iters;                 // (all lanes of the group add the same number to the same word)
                    }
                    const uint32_t done = m.done;
                    m.done = done + 1u;
                    decide = done == A.n_starts;
                    if (decide) {                         // every start has been tried
                        double th, x0;
                        current(cold_args(), model, th, x0);
                        const bool better = refit && m.F < F0;
                        if (!better) m.x[own] = x0;
                        m.F = better ? m.F : F0;
                        m.F0 = F0;
                        m.improved = better ? 1u : 0u;
                        m.iters = refit ? m.iters : 0u;
                        m.phase = 0u;
                        m.version = 1u;
                        m.running = 0u;
#pragma unroll
                        for (int i = 0; i < 3; ++i) m.kick_of[i] = 0u;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (decide) {
                    // An overlap exponent that ended on a bound sits on a plateau (at k = 32 the overlap function no longer
                    // feels k): try again from the best point with that exponent moved back inside, twice over the three
                    // exponents.  A kick from the point from which that exponent was last kicked ends as that one did.
                    double best = m.x[own], best_F = m.F;
                    uint32_t next = m.phase, v = m.version, sum = m.iters, running = m.running, improved = m.improved;
                    auto on_bound = [&]() {
                        const uint32_t b = (uint32_t)(__ballot(refit && exponent && (best <= lower * (1.0 + 1e-9) || best >= 1.0 - 1e-9)) >> row0);
                        return (b >> TH_SYNC & 1u) | (b >> TH_OFF & 1u) << 1 | (b >> TH_SWAP & 1u) << 2;
                    };
                    uint32_t bound = on_bound();
                    for (; next < 6u; ++next) {
                        const uint32_t e = next % 3u;
                        if (!(bound >> e & 1u)) continue;
                        if (m.kick_of[e] != v) break;
                        sum += m.kick_iters[e];
                        if (m.kick_F[e] < best_F) {
                            best_F = m.kick_F[e];
                            best = m.kick_x[e][own];
                            improved = 1u;
                            ++v;
                            running = 0u;
                            bound = on_bound();
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    const uint32_t e = next % 3u;
                    if (next < 6u) {
                        if (!(running >> e & 1u)) {       // (otherwise another slot is at it and goes on from there)
                            running |= 1u << e;
                            want_item = false;
                            kick = e;
                            version = v;
                            iters = 0;
                            xn = own == (e == 0u ? TH_SYNC : e == 1u ? TH_OFF : TH_SWAP) ? KICK_TO : best;
                            state = SLOT_START;
                        }
                    } else {
                        const FitArgs &C = cold_args();
                        const uint32_t S = C.sample_off[model + 1] - C.sample_off[model];
                        const double inv_S = S ? 1.0 / (double)S : 0.0, before = m.F0;
                        double th, x0;
                        current(C, model, th, x0);
                        if (improved) th = exponent ? 1.0 / best : best;
                        const rk_fit_result &o = C.out;
                        float *const dst[NP] = {o.k_bwd, o.k_sync, o.k_opt, o.k_opt_off, o.k_off, o.k_swap, o.k_const};
                        float *to = dst[0];
#pragma unroll
                        for (int i = 1; i < NP; ++i) to = own == (uint32_t)i ? dst[i] : to;
                        if (lane < (uint32_t)NP) {
                            if (to) to[model] = (float)th;
                            if (o.theta) o.theta[(size_t)model * NP + own] = th;
                        } else if (lane == (uint32_t)NP) {
                            if (o.rmsle_before) o.rmsle_before[model] = (float)sqrt(before * inv_S);
                            if (o.rmsle_after) o.rmsle_after[model] = (float)sqrt(best_F * inv_S);
                            // (more runs than the caller announced: left alone, flagged)
                            if (o.iters) o.iters[model] = S > C.most_runs ? 0xFFFFFFFFu : sum;
                        }
                        next = PHASE_DONE;
                        v = 0u;                           // (a kick of it that still runs ahead is of no use)
                        freed = rec;
                    }
                    m.x[own] = best;
                    m.F = best_F;
                    m.phase = next;
                    m.version = v;
                    m.iters = sum;
                    m.running = running;
                    m.bound = bound;
                    m.improved = improved;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // the next slot may work on the same record
            todo &= ~((W == 64 ? ~0ull : ((1ull << (W & 63)) - 1ull)) << (who * W));
        }
        // the next items: the current model's remaining starts, then another model, then kicks that may be needed
        if ((opening || any_ended) && __ballot(want_item)) {
            const FitArgs &C = cold_args();
            for (uint32_t who = 0; who < SLOTS; ++who) {
                const uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)freed, (int)(who * W));
                if (r != NONE) free_recs |= 1u << r;
            }
            for (uint32_t who = 0; who < SLOTS; ++who) {
                if (!__builtin_amdgcn_readlane(want_item ? 1 : 0, (int)(who * W))) continue;
                if (!src_dry && (src_start == NONE || src_start > A.n_starts)) {
                    uint32_t m = 0;
                    if (wlane == 0) m = atomicAdd(C.next_model, 1u);
                    m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
                    if (m >= C.n_fits) {
                        src_dry = true;
                    } else {
                        src_model = m;
                        src_start = 0;
                        src_rec = (uint32_t)__ffs((int)free_recs) - 1u;
                        free_recs &= free_recs - 1u;
                        Rec &q = sh_rec[wave][src_rec];
                        q.F = __builtin_huge_val();
                        q.model = m;
                        q.start = NONE;
                        q.iters = 0u;
                        q.done = 0u;
                        q.phase = PHASE_STARTS;
                    }
                }
                // With no model left, a kick that the one under way may make necessary: of an exponent on a bound that has
                // not been kicked from the best point and comes up again.  (Whole wavefront: the records are the same to all.)
                uint32_t ahead = NONE, ahead_rec = 0;
                if (src_dry) {
                    for (uint32_t r = 0; r < RECS && ahead == NONE; ++r) {
                        const Rec &m = sh_rec[wave][r];
                        for (uint32_t k = m.phase; k < 6u && k < m.phase + 3u; ++k) {
                            const uint32_t e = k % 3u;
                            if (ahead == NONE && (m.bound >> e & 1u) && !(m.running >> e & 1u) && m.kick_of[e] != m.version) {
                                ahead = e;
                                ahead_rec = r;
                            }
                        }
                    }
                    if (ahead != NONE) {
                        const uint32_t running = sh_rec[wave][ahead_rec].running | 1u << ahead;
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        sh_rec[wave][ahead_rec].running = running;
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    }
                }
                if (slot == who) {
                    want_item = false;
                    kick = ahead;
                    iters = 0;
                    if (src_dry && ahead == NONE) {
                        state = SLOT_IDLE;
                        want_item = true;                 // a kick may come up for it
                    } else {
                        const uint32_t take = src_dry ? sh_rec[wave][ahead_rec].model : src_model;
                        if (take != model) {              // the lane's run and the group's overlaps
                            const uint32_t s0 = C.sample_off[take];
                            n_runs = C.sample_off[take + 1] - s0;
                            if (n_runs > C.most_runs) n_runs = C.most_runs;
                            has_run = lane < n_runs;      // a lane without a run contributes nothing at all
                            R = Run{};
                            if (has_run) R = load_run(C, take, s0 + lane);
                            const unsigned long long off = (__ballot(R.off) >> (slot * W)) & (W == 64 ? ~0ull : ((1ull << (W & 63)) - 1ull));
                            off_rank = (uint32_t)__popcll(off & ((1ull << lane) - 1ull));
                            n_tasks = n_runs + 2u * (uint32_t)__popcll(off);
                            if (has_run) task[lane] = Task{R.Tfwd, R.gc * R.Tfwd, R.Tdp, TH_BWD, TH_SYNC};
                            if (R.off) {
                                task[n_runs + 2u * off_rank] = Task{0.0, R.Tdp, R.Toff, TH_CONST, TH_OFF};
                                task[n_runs + 2u * off_rank + 1u] = Task{R.opt_scale, 0.0, R.Toff, TH_OPT_OFF, TH_SWAP};
                            }
                        }
                        model = take;
                        if (src_dry) {
                            const Rec &m = sh_rec[wave][ahead_rec];
                            rec = ahead_rec;
                            version = m.version;
                            refit = true;                 // (only a refitted model has exponents to kick)
                            xn = own == (ahead == 0u ? TH_SYNC : ahead == 1u ? TH_OFF : TH_SWAP) ? KICK_TO : m.x[own];
                            state = SLOT_START;
                        } else {
                            state = SLOT_CURRENT;
                            start = src_start;
                            rec = src_rec;
                            double th;
                            current(C, model, th, xn);
                        }
                    }
                }
                if (!src_dry) ++src_start;
            }
            if (!__ballot(state != SLOT_IDLE)) break;
        }
        opening = false;
        // The evaluation.  First the overlaps of all runs, an overlap per lane and round: 16 runs of which 5 are offloaded
        // take two rounds, where a lane that computed all overlaps of its own run would take three.
        point[own] = xn;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        Overlap sync = {};
        double Tb = 0.0;
        const uint32_t tasks = state != SLOT_IDLE ? n_tasks : 0u;
        for (uint32_t t = lane; __ballot(t < tasks); t += W) {
            Task q = {};
            if (t < tasks) q = task[t];
            Overlap o;
            o.k = 1.0 / point[q.exp];
            const double first = point[q.var] * q.a + q.b;
            overlap(o.k, first, q.y, o.f, o.fx, o.fk);
            if (t < (uint32_t)W) { sync = o; Tb = first; }
            if (t >= n_runs && t < tasks) over[t - n_runs] = o;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        // then the residual ln(1+pred) - ln(1+y) of the lane's run and its derivatives by the search variables
        // (k = 1/v, dk/dv = -k^2); an invalid run predicts 0
        {
            double J[NR], v[N_SUM];
            const Overlap o1 = over[R.off ? 2u * off_rank : 0u], o2 = over[R.off ? 2u * off_rank + 1u : 0u];
            double T = R.aTfwd + R.am1 * Tb + sync.f + R.Tconst + point[TH_CONST];
            T += R.off ? o1.f + o2.f : point[TH_OPT] * R.opt_scale;
            const double pr = R.b / T;
            const bool use = has_run && R.valid;
            const double w = use ? -(pr / (T * (1.0 + pr))) : 0.0;
            J[TH_BWD] = use ? w * (R.Tfwd * (R.am1 + sync.fx)) : 0.0;
            J[TH_SYNC] = use ? w * sync.fk * (-sync.k * sync.k) : 0.0;
            J[TH_OPT] = use && !R.off ? w * R.opt_scale : 0.0;
            J[TH_OPT_OFF] = use && R.off ? w * (o2.fx * R.opt_scale) : 0.0;
            J[TH_OFF] = use && R.off ? w * o1.fk * (-o1.k * o1.k) : 0.0;
            J[TH_SWAP] = use && R.off ? w * o2.fk * (-o2.k * o2.k) : 0.0;
            J[TH_CONST] = w;
            J[NP] = use ? log1p(pr) - R.logy : has_run ? -R.logy : 0.0;
            int n = 0;
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int j = i; j < NR; ++j) v[n++] = J[i] * J[j];
            group_sums<W>(v, wlane);
            double *to = sums[into];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                to[place[i] & 0xFFu] = v[i];
                to[place[i] >> 8] = v[i];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

__global__ void k_fit_begin(uint32_t *next_model) { *next_model = 0u; }

template <int W>
void launch_fit(const FitArgs &A, uint32_t max_blocks, hipStream_t s) {
    constexpr uint64_t SLOTS = FIT_THREADS / W;          // of a workgroup
    const uint64_t items = (uint64_t)A.n_fits * (A.n_starts + 1u), want = (items + SLOTS - 1) / SLOTS;
    k_fit<W><<<(uint32_t)(want < max_blocks ? want : max_blocks), FIT_THREADS, 0, s>>>(A);
}

}  // namespace

extern "C" int32_t rk_fit_models(rk_ctx *ctx, const rk_jobs *jobs, const rk_env *env, const rk_samples *samples,
                                 const rk_fit_options *options, const rk_fit_result *result) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if (!jobs || !samples || !options || !result) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if ((rc = rk_check_env(ctx, env))) return rc;
    if (jobs->n_jobs == 0) return RK_OK;
    if (!samples->sample_off || !samples->triple || !samples->option || !samples->cpus || !samples->thr)
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "samples: null array");
    if (!jobs->P_bytes || !jobs->seq || !jobs->hidden || !jobs->elem_bytes || !jobs->t_fwd_sample || !jobs->k_bwd ||
        !jobs->k_sync || !jobs->k_opt || !jobs->k_opt_off || !jobs->k_off || !jobs->k_swap || !jobs->k_const ||
        !jobs->layers || !jobs->gbatch || !jobs->mbatch)
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "jobs: null array");
    if (samples->max_samples > RK_FIT_MAX_SAMPLES)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u runs per model, at most %u", samples->max_samples, RK_FIT_MAX_SAMPLES);
    if (options->n_starts > RK_FIT_MAX_STARTS)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "%u extra starting points, at most %u", options->n_starts, RK_FIT_MAX_STARTS);
    if (options->n_starts > 0 && !options->start_offsets) return rk_fail(ctx, RK_ERR_INVALID_ARG, "start_offsets is null");
    if (!(options->refit_threshold >= 0.f)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "refit_threshold negative or NaN");
    RK_HIP(ctx, hipSetDevice(ctx->device));
    FitArgs A;
    A.jobs = job_dev(jobs);
    A.env = *env;
    A.n_fits = jobs->n_jobs;
    A.sample_off = samples->sample_off; A.triple = samples->triple; A.option = samples->option;
    A.cpus = samples->cpus; A.thr = samples->thr;
    A.max_iter = options->max_iter; A.n_starts = options->n_starts;
    A.refit_threshold = (double)options->refit_threshold;
    for (uint32_t s = 0; s < RK_FIT_MAX_STARTS; ++s)
        for (int i = 0; i < NP; ++i) {
            const double v = s < options->n_starts ? options->start_offsets[(size_t)s * NP + i] : 0.0;
            if (!(v == v) || v > 700.0 || v < -700.0) return rk_fail(ctx, RK_ERR_INVALID_ARG, "start offset out of range");
            A.offsets[s][i] = v;
        }
    A.out = *result;
    if ((rc = rk_scratch(ctx, SL_FIT_NEXT, 4, (void **)&A.next_model))) return rc;
    k_fit_begin<<<1, 1, 0, ctx->stream>>>(A.next_model);
    RK_CHECK_LAUNCH(ctx, "k_fit_begin");
    const uint32_t ms = samples->max_samples;
    A.most_runs = ms <= 8 ? 8u : ms <= 16 ? 16u : ms <= 32 ? 32u : 64u;
    // Workgroups: one or two wavefronts per SIMD of the 256 compute units.  The second makes every iteration of the
    // first slower and pays only when there is enough to do for both beyond the longest descents of the last models:
    // 16 runs, 5 starting points, one against two: 3,000 models 5.7 against 6.5 ms, 6,000 7.4 against 7.3, 8,500 9.2
    // against 8.2, 10,000 9.6 against 9.1.  Wider groups have fewer models to a wavefront, and the line is drawn at the same
    // number of lanes; it could lie lower: 24 runs, 2,500 models 6.9 against 6.9, 3,500 7.8 against 7.5, 4,200 8.8 against
    // 7.8; 48 runs, 1,500 models 6.9 against 6.4, 2,100 7.0 against 6.8, 3,000 8.5 against 7.4.
    const uint32_t width = A.most_runs < 16u ? 16u : A.most_runs;
    const uint32_t blocks = (uint64_t)A.n_fits * width > 8192ull * 16ull ? 512u : 256u;
    if (width == 16u) launch_fit<16>(A, blocks, ctx->stream);
    else if (width == 32u) launch_fit<32>(A, blocks, ctx->stream);
    else launch_fit<64>(A, blocks, ctx->stream);
    RK_CHECK_LAUNCH(ctx, "k_fit");
    return RK_OK;
}
