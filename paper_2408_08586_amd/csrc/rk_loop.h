// What Algorithm 1's Schedule loop asks of a job's curves (paper Sec. 5.2, the paragraphs on slopes and on shrinking):
// a job's next step up in GPUs and in CPU levels, and what it gives when it steps down.  Shared by the loop over
// the cluster's totals and the loop over its nodes; `Args` is the kernel's argument struct with
//   X.tb, X.grid, X.ref_thr, X.best_thr, X.curve_thr   plan table, grid and the curves (segment layout, all jobs)
//   st.gi, st.ci                                       what every job holds: index of its GPU count (-1: nothing), CPU level
//   G                                                  GPUs of the cluster (no step goes beyond)
//   state, floor_seg, floor_c                          per job, each may be null
//   ds_g, ds_c                                         per job, for the cached slopes (rs_refresh_give)
//   next, gives                                        per job, for what is kept of it between its steps (rs_keep)
#pragma once
#include <type_traits>

#include "rk_internal.h"
#include "rk_model.h"

template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v) {
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    const uint32_t l2 = (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, CTRL, 0xF, 0xF, false);
    const uint32_t h2 = (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, CTRL, 0xF, 0xF, false);
    return ((unsigned long long)h2 << 32) | l2;
}

// Maximum over the wavefront, in every lane; all 64 lanes must be active.
// Within each row of 16 lanes by data-parallel-primitive moves (neighbour,
// neighbour pair, mirrored halves of 8, mirrored halves of 16), then the four
// rows through scalar registers.
__device__ __forceinline__ unsigned long long wave_max_u64_rows(unsigned long long v) {
    unsigned long long o;
    o = dpp_u64<0xB1>(v);  v = o > v ? o : v;                   // quad_perm [1,0,3,2]
    o = dpp_u64<0x4E>(v);  v = o > v ? o : v;                   // quad_perm [2,3,0,1]
    o = dpp_u64<0x141>(v); v = o > v ? o : v;                   // row_half_mirror
    o = dpp_u64<0x140>(v); v = o > v ? o : v;                   // row_mirror
    unsigned long long m = 0;
#pragma unroll
    for (int r = 0; r < 64; r += 16) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, r);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), r);
        const unsigned long long row = ((unsigned long long)hi << 32) | lo;
        m = row > m ? row : m;
    }
    return m;
}

// The minimum likewise.
__device__ __forceinline__ unsigned long long wave_min_u64_rows(unsigned long long v) { return ~wave_max_u64_rows(~v); }

// Minimum and maximum of a word over the wavefront, in every lane; all 64 lanes must be active.  Within each row of 16
// lanes as above, then every row's result into the rows behind it: an instruction per move, where a pair of words takes
// five, so what is ordered by several words is reduced word by word.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t rs_dpp_u32(uint32_t none, uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t rs_min_u32(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t rs_max_u32(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t row_min_u32(uint32_t v) {                        // within the rows of 16 lanes
    v = rs_min_u32(v, rs_dpp_u32<0xB1, 0xF>(0xFFFFFFFFu, v));                        // quad_perm [1,0,3,2]
    v = rs_min_u32(v, rs_dpp_u32<0x4E, 0xF>(0xFFFFFFFFu, v));                        // quad_perm [2,3,0,1]
    v = rs_min_u32(v, rs_dpp_u32<0x141, 0xF>(0xFFFFFFFFu, v));                       // row_half_mirror
    return rs_min_u32(v, rs_dpp_u32<0x140, 0xF>(0xFFFFFFFFu, v));                    // row_mirror
}
__device__ __forceinline__ uint32_t wave_min_u32_rows(uint32_t v) {
    v = row_min_u32(v);
    v = rs_min_u32(v, rs_dpp_u32<0x142, 0xA>(0xFFFFFFFFu, v));                       // row_bcast:15 into rows 1 and 3
    v = rs_min_u32(v, rs_dpp_u32<0x143, 0xC>(0xFFFFFFFFu, v));                       // row_bcast:31 into rows 2 and 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ uint32_t row_max_u32(uint32_t v) {
    v = rs_max_u32(v, rs_dpp_u32<0xB1, 0xF>(0u, v));
    v = rs_max_u32(v, rs_dpp_u32<0x4E, 0xF>(0u, v));
    v = rs_max_u32(v, rs_dpp_u32<0x141, 0xF>(0u, v));
    return rs_max_u32(v, rs_dpp_u32<0x140, 0xF>(0u, v));
}
__device__ __forceinline__ uint32_t row_sum_u32(uint32_t v) {                        // row_ror:8, 4, 2, 1
    v += rs_dpp_u32<0x128, 0xF>(0u, v);
    v += rs_dpp_u32<0x124, 0xF>(0u, v);
    v += rs_dpp_u32<0x122, 0xF>(0u, v);
    return v + rs_dpp_u32<0x121, 0xF>(0u, v);
}
__device__ __forceinline__ uint32_t wave_max_u32_rows(uint32_t v) {
    v = row_max_u32(v);
    v = rs_max_u32(v, rs_dpp_u32<0x142, 0xA>(0u, v));
    v = rs_max_u32(v, rs_dpp_u32<0x143, 0xC>(0u, v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Sums over the wavefront, in every lane; all 64 lanes must be active.  The additions are those of six exchanges with the lane
// 32, 16, 8, 4, 2 and 1 away, in that order: the halves and the pairs of rows change places by lane swaps, and within a row
// lanes that have the same value by then stand in for each other, so that rotations do (0.9 us less than exchanges through LDS).
__device__ __forceinline__ double wave_sum_f64(double v) {
    const auto two = [](double x, auto swap) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(x);
        const auto lo = swap((uint32_t)b), hi = swap((uint32_t)(b >> 32));
        return __longlong_as_double((long long)(((unsigned long long)hi[0] << 32) | lo[0])) +
               __longlong_as_double((long long)(((unsigned long long)hi[1] << 32) | lo[1]));
    };
    v = two(v, [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
    v = two(v, [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
    const auto turned = [](auto ctrl, double x) { return __longlong_as_double((long long)dpp_u64<decltype(ctrl)::value>((unsigned long long)__double_as_longlong(x))); };
    v += turned(std::integral_constant<int, 0x128>{}, v);       // row_ror:8, 4, 2, 1
    v += turned(std::integral_constant<int, 0x124>{}, v);
    v += turned(std::integral_constant<int, 0x122>{}, v);
    v += turned(std::integral_constant<int, 0x121>{}, v);
    return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
    const auto a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = a[0] + a[1];
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return row_sum_u32(b[0] + b[1]);
}

// Lane s of a value whose index is the same in all lanes (through a scalar register).
__device__ __forceinline__ uint32_t wave_lane_u32(uint32_t x, uint32_t s) {
    return (uint32_t)__builtin_amdgcn_readlane((int)x, __builtin_amdgcn_readfirstlane((int)s));
}

__device__ __forceinline__ unsigned long long cpu_cost(const GridDev &G, uint32_t ci, uint32_t g) {
    return G.cpu_mode ? (unsigned long long)G.cpu_levels[ci] * g : (unsigned long long)G.cpu_levels[ci];
}

struct RsStep { uint32_t any; int32_t tgt; uint32_t lvl; float slope, gain; unsigned long long dg, dc; };
struct RsGive { uint32_t any; int32_t tgt; float loss, slope; unsigned long long dg, dc; };

template <class Args>
__device__ __forceinline__ uint32_t rs_ns(const Args &A, uint32_t j) { return A.X.tb.seg_off[j + 1] - A.X.tb.seg_off[j]; }
template <class Args>
__device__ __forceinline__ unsigned long long rs_g(const Args &A, uint32_t j, int32_t s) {
    return s < 0 ? 0ull : A.X.tb.seg_g[A.X.tb.seg_off[j] + (uint32_t)s];
}
template <class Args>
__device__ __forceinline__ unsigned long long rs_c(const Args &A, uint32_t j, uint32_t c, int32_t s) {
    return s < 0 ? 0ull : cpu_cost(A.X.grid, c, (uint32_t)rs_g(A, j, s));
}
// value of job j at CPU level c, top memory tier, segment s (0 below the first segment)
template <class Args>
__device__ __forceinline__ float rs_at(const Args &A, const float *arr, uint32_t j, uint32_t c, int32_t s) {
    if (s < 0) return 0.f;
    const uint32_t n_mem = A.X.grid.n_mem, ns = rs_ns(A, j);
    return arr[(uint64_t)A.X.grid.n_cpu * n_mem * A.X.tb.seg_off[j] + ((uint64_t)c * n_mem + (n_mem - 1)) * ns + (uint32_t)s];
}
template <class Args>
__device__ __forceinline__ bool rs_part(const Args &A, uint32_t j) { return !A.state || A.state[j] == 0; }
// state 2: the job keeps exactly what it holds (it takes no step and gives nothing); any other non-zero state: it takes
// no part and holds nothing
template <class Args>
__device__ __forceinline__ bool rs_holds(const Args &A, uint32_t j) { return !A.state || A.state[j] == 0 || A.state[j] == 2; }
// the job's floor: segment (-1: none; a segment the job does not have counts as none) and CPU level (clamped)
template <class Args>
__device__ __forceinline__ int32_t rs_fl_s(const Args &A, uint32_t j) {
    if (!A.floor_seg) return -1;
    const int32_t f = A.floor_seg[j];
    return (f >= 0 && (uint32_t)f < rs_ns(A, j)) ? f : -1;
}
template <class Args>
__device__ __forceinline__ uint32_t rs_fl_c(const Args &A, uint32_t j) {
    if (rs_fl_s(A, j) < 0 || !A.floor_c) return 0u;
    const uint32_t c = A.floor_c[j];
    return c < A.X.grid.n_cpu ? c : A.X.grid.n_cpu - 1u;
}

// Next GPU step of job j, which holds (gi, ci).  `lanes` threads share the candidates (1: the calling thread alone; 64: a wavefront, all
// lanes get the result).  Highest slope, the smaller amount among equal slopes.
template <class Args>
__device__ RsStep rs_up_gpu(const Args &A, uint32_t j, int32_t gi, uint32_t ci, uint32_t lane, uint32_t lanes) {
    RsStep st = {0u, -1, ci, 0.f, 0.f, 0ull, 0ull};
    const float ref = A.X.ref_thr[j];
    const float cur = rs_at(A, A.X.curve_thr, j, ci, gi);
    const int32_t fl = rs_fl_s(A, j);
    if (fl >= 0 && gi < fl) {
        const uint32_t lvl = ci > rs_fl_c(A, j) ? ci : rs_fl_c(A, j);
        const float v = rs_at(A, A.X.curve_thr, j, lvl, fl);
        st.any = 1u; st.tgt = fl; st.lvl = lvl;
        st.dg = rs_g(A, j, fl) - rs_g(A, j, gi);
        st.dc = rs_c(A, j, lvl, fl) - rs_c(A, j, ci, gi);
        st.gain = (v - cur) / ref;
        st.slope = st.gain / (float)st.dg;
        return st;
    }
    const int32_t ns = (int32_t)rs_ns(A, j);
    unsigned long long key = 0;                            // slope bits, then the inverted segment index
    for (int32_t s = gi + 1 + (int32_t)lane; s < ns; s += (int32_t)lanes) {
        if (rs_g(A, j, s) > A.G) break;
        const float v = rs_at(A, A.X.curve_thr, j, ci, s);
        if (!(v > cur)) continue;
        const unsigned long long dg = rs_g(A, j, s) - rs_g(A, j, gi);
        const float gain = (v - cur) / ref;
        const float sl = gain / (float)dg;
        if (!(sl > 0.f)) continue;
        const unsigned long long k = ((unsigned long long)__float_as_uint(sl) << 32) | (0xFFFFFFFFu - (uint32_t)s);
        key = k > key ? k : key;
    }
    if (lanes > 1) key = wave_max_u64_rows(key);
    if (key) {
        const int32_t s = (int32_t)(0xFFFFFFFFu - (uint32_t)key);
        const float v = rs_at(A, A.X.curve_thr, j, ci, s);
        st.any = 1u; st.tgt = s;
        st.dg = rs_g(A, j, s) - rs_g(A, j, gi);
        st.dc = rs_c(A, j, ci, s) - rs_c(A, j, ci, gi);
        st.gain = (v - cur) / ref;
        st.slope = st.gain / (float)st.dg;
    }
    return st;
}

template <class Args>
__device__ RsStep rs_up_cpu(const Args &A, uint32_t j, int32_t gi, uint32_t ci, uint32_t lane, uint32_t lanes) {
    RsStep st = {0u, gi, ci, 0.f, 0.f, 0ull, 0ull};
    if (gi < 0) return st;
    const float ref = A.X.ref_thr[j];
    const float cur = rs_at(A, A.X.best_thr, j, ci, gi);
    unsigned long long key = 0;
    for (uint32_t c = ci + 1 + lane; c < A.X.grid.n_cpu; c += lanes) {
        const float v = rs_at(A, A.X.best_thr, j, c, gi);
        if (!(v > cur)) continue;
        const unsigned long long dc = rs_c(A, j, c, gi) - rs_c(A, j, ci, gi);
        const float gain = (v - cur) / ref;
        const float sl = gain / (float)dc;
        if (!(sl > 0.f)) continue;
        const unsigned long long k = ((unsigned long long)__float_as_uint(sl) << 32) | (0xFFFFFFFFu - c);
        key = k > key ? k : key;
    }
    if (lanes > 1) key = wave_max_u64_rows(key);
    if (key) {
        const uint32_t c = 0xFFFFFFFFu - (uint32_t)key;
        const float v = rs_at(A, A.X.best_thr, j, c, gi);
        st.any = 1u; st.lvl = c;
        st.dc = rs_c(A, j, c, gi) - rs_c(A, j, ci, gi);
        st.gain = (v - cur) / ref;
        st.slope = st.gain / (float)st.dc;
    }
    return st;
}

// What job v gives when it steps down in GPUs from (gi, ci): to where the curve's value just below its amount begins
// (the largest amount with a lower throughput, or the smallest with the same one when it holds more than it uses), not
// below its floor.  The curve does not fall along a row, so that place, the first amount whose value reaches the one
// just below, is found by bisection (lanes == 1) or by the 64 lanes of a wavefront looking at 64 amounts at a time
// (all lanes get the result).
template <class Args>
__device__ RsGive rs_down_gpu_at(const Args &A, uint32_t v, int32_t gi, uint32_t ci, uint32_t lane, uint32_t lanes) {
    RsGive gv = {0u, -1, 0.f, 0.f, 0ull, 0ull};
    const int32_t fl = rs_fl_s(A, v);
    if (!rs_part(A, v) || gi < 0 || (fl >= 0 && gi <= fl)) return gv;
    const float V = rs_at(A, A.X.curve_thr, v, ci, gi);
    const float want = rs_at(A, A.X.curve_thr, v, ci, gi - 1);
    int32_t t = -1;
    if (want > 0.f) {
        if (lanes > 1) {
            t = gi - 1;                                    // the amount just below reaches its own value
            for (int32_t base = 0; base < gi - 1; base += 64) {
                const int32_t s = base + (int32_t)lane;
                const bool reaches = s < gi - 1 && rs_at(A, A.X.curve_thr, v, ci, s) >= want;
                const unsigned long long m = __ballot(reaches);
                if (m) { t = base + (int32_t)__ffsll((long long)m) - 1; break; }
            }
        } else {
            int32_t lo = 0, hi = gi - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi) >> 1;
                if (rs_at(A, A.X.curve_thr, v, ci, mid) >= want) hi = mid; else lo = mid + 1;
            }
            t = lo;
        }
    }
    if (fl >= 0 && t < fl) t = fl;
    gv.any = 1u; gv.tgt = t;
    gv.loss = (V - rs_at(A, A.X.curve_thr, v, ci, t)) / A.X.ref_thr[v];
    gv.dg = rs_g(A, v, gi) - rs_g(A, v, t);
    gv.dc = rs_c(A, v, ci, gi) - rs_c(A, v, ci, t);
    gv.slope = gv.loss / (float)gv.dg;
    return gv;
}
template <class Args>
__device__ __forceinline__ RsGive rs_down_gpu(const Args &A, uint32_t v, uint32_t lane = 0, uint32_t lanes = 1) {
    return rs_down_gpu_at(A, v, A.st.gi[v], A.st.ci[v], lane, lanes);
}

// ... and when it steps down one CPU level from (gi, ci), not below its floor's level
template <class Args>
__device__ RsGive rs_down_cpu_at(const Args &A, uint32_t v, int32_t gi, uint32_t ci) {
    RsGive gv = {0u, gi, 0.f, 0.f, 0ull, 0ull};
    const uint32_t lowest = rs_fl_s(A, v) >= 0 ? rs_fl_c(A, v) : 0u;
    if (!rs_part(A, v) || gi < 0 || ci == 0 || ci <= lowest) return gv;
    gv.any = 1u;
    gv.loss = (rs_at(A, A.X.best_thr, v, ci, gi) - rs_at(A, A.X.best_thr, v, ci - 1, gi)) / A.X.ref_thr[v];
    gv.dc = rs_c(A, v, ci, gi) - rs_c(A, v, ci - 1, gi);
    gv.slope = gv.loss / (float)gv.dc;
    return gv;
}
template <class Args>
__device__ __forceinline__ RsGive rs_down_cpu(const Args &A, uint32_t v) { return rs_down_cpu_at(A, v, A.st.gi[v], A.st.ci[v]); }

// the cached slopes of job v after its state changed to (gi, ci): what it loses per unit it gives
template <class Args>
__device__ __forceinline__ void rs_refresh_give(const Args &A, uint32_t v) {
    const RsGive a = rs_down_gpu(A, v), b = rs_down_cpu(A, v);
    A.ds_g[v] = a.any ? a.slope : __int_as_float(0x7F800000);
    A.ds_c[v] = b.any ? b.slope : __int_as_float(0x7F800000);
}

// ---- the same steps for a wavefront that holds the job's rows in its registers
// The searches above follow one load with the next.  A job of at most 64 amounts fits a wavefront, an amount per lane:
// the rows its steps from (gi, ci) read are loaded at once (the curve and the best plans at CPU level ci and at the
// level below, the GPUs of every amount, and, a CPU level per lane, the best plans of amount gi), and every step is
// found from the registers, with the arithmetic of the functions above.
struct RsRows {
    uint32_t ns; float ref; int32_t fl; uint32_t fl_c; bool part;         // the same in all lanes
    float curve, curve_lo, best, best_lo;   // lane s: curve_thr and best_thr of amount s at level ci, and at level ci - 1 (0 without)
    uint32_t g;                             // lane s: GPUs of amount s
    float col;                              // lane c: best_thr of amount gi at level c (0 without)
};
__device__ __forceinline__ float rs_lane_f(float x, int32_t s) { return s < 0 ? 0.f : __uint_as_float(wave_lane_u32(__float_as_uint(x), (uint32_t)s)); }
__device__ __forceinline__ uint32_t rs_lane_u(uint32_t x, int32_t s) { return s < 0 ? 0u : wave_lane_u32(x, (uint32_t)s); }

// (so, ns: where the job's amounts begin in the plan table and how many they are, rs_ns)
template <class Args>
__device__ __forceinline__ RsRows rs_rows(const Args &A, uint32_t v, uint32_t so, uint32_t ns, int32_t gi, uint32_t ci, uint32_t lane) {
    RsRows R = {};
    const uint32_t n_mem = A.X.grid.n_mem, n_cpu = A.X.grid.n_cpu;
    R.ns = ns;
    R.ref = A.X.ref_thr[v];
    R.fl = rs_fl_s(A, v); R.fl_c = rs_fl_c(A, v); R.part = rs_part(A, v);
    const uint64_t job = (uint64_t)n_cpu * n_mem * so + (uint64_t)(n_mem - 1) * R.ns;    // level 0, top tier, amount 0
    const uint64_t level = (uint64_t)n_mem * R.ns;
    if (lane < R.ns) {
        R.curve = A.X.curve_thr[job + ci * level + lane];
        R.best = A.X.best_thr[job + ci * level + lane];
        if (ci > 0) {
            R.curve_lo = A.X.curve_thr[job + (ci - 1) * level + lane];
            R.best_lo = A.X.best_thr[job + (ci - 1) * level + lane];
        }
        R.g = A.X.tb.seg_g[so + lane];
    }
    if (gi >= 0 && lane < n_cpu) R.col = A.X.best_thr[job + lane * level + (uint32_t)gi];
    return R;
}

// rs_down_gpu_at on the row `curve` (lane s: the curve of amount s at level ci)
template <class Args>
__device__ __forceinline__ RsGive rs_down_gpu_rows(const Args &A, const RsRows &R, float curve, int32_t gi, uint32_t ci, uint32_t lane) {
    RsGive gv = {0u, -1, 0.f, 0.f, 0ull, 0ull};
    if (!R.part || gi < 0 || (R.fl >= 0 && gi <= R.fl)) return gv;
    const float V = rs_lane_f(curve, gi), want = rs_lane_f(curve, gi - 1);
    int32_t t = -1;
    if (want > 0.f) {
        const unsigned long long m = __ballot((int32_t)lane < gi - 1 && curve >= want);
        t = m ? (int32_t)__ffsll((long long)m) - 1 : gi - 1;
    }
    if (R.fl >= 0 && t < R.fl) t = R.fl;
    const uint32_t g_gi = rs_lane_u(R.g, gi), g_t = rs_lane_u(R.g, t);
    gv.any = 1u; gv.tgt = t;
    gv.loss = (V - rs_lane_f(curve, t)) / R.ref;
    gv.dg = (unsigned long long)g_gi - g_t;
    gv.dc = cpu_cost(A.X.grid, ci, g_gi) - (t < 0 ? 0ull : cpu_cost(A.X.grid, ci, g_t));
    gv.slope = gv.loss / (float)gv.dg;
    return gv;
}
// rs_down_cpu_at; hi and lo are the best plans' values of amount gi at levels ci and ci - 1
template <class Args>
__device__ __forceinline__ RsGive rs_down_cpu_rows(const Args &A, const RsRows &R, int32_t gi, uint32_t ci, float hi, float lo) {
    RsGive gv = {0u, gi, 0.f, 0.f, 0ull, 0ull};
    const uint32_t lowest = R.fl >= 0 ? R.fl_c : 0u;
    if (!R.part || gi < 0 || ci == 0 || ci <= lowest) return gv;
    const uint32_t g = rs_lane_u(R.g, gi);
    gv.any = 1u;
    gv.loss = (hi - lo) / R.ref;
    gv.dc = cpu_cost(A.X.grid, ci, g) - cpu_cost(A.X.grid, ci - 1, g);
    gv.slope = gv.loss / (float)gv.dc;
    return gv;
}
// rs_up_gpu for a job that is not below its floor
template <class Args>
__device__ __forceinline__ RsStep rs_up_gpu_rows(const Args &A, const RsRows &R, int32_t gi, uint32_t ci, uint32_t lane) {
    RsStep st = {0u, -1, ci, 0.f, 0.f, 0ull, 0ull};
    const float cur = rs_lane_f(R.curve, gi);
    const uint32_t g_cur = rs_lane_u(R.g, gi);
    uint32_t key = 0;                                      // slope bits; the smallest amount among equal slopes
    if ((int32_t)lane > gi && lane < R.ns && (unsigned long long)R.g <= A.G && R.curve > cur) {   // amounts ascend in GPUs
        const float sl = ((R.curve - cur) / R.ref) / (float)(R.g - g_cur);
        if (sl > 0.f) key = __float_as_uint(sl);
    }
    const uint32_t top = wave_max_u32_rows(key);
    if (top) {
        const int32_t s = (int32_t)__ffsll((long long)__ballot(key == top)) - 1;
        const uint32_t g_s = rs_lane_u(R.g, s);
        st.any = 1u; st.tgt = s;
        st.dg = (unsigned long long)g_s - g_cur;
        st.dc = cpu_cost(A.X.grid, ci, g_s) - (gi < 0 ? 0ull : cpu_cost(A.X.grid, ci, g_cur));
        st.gain = (rs_lane_f(R.curve, s) - cur) / R.ref;
        st.slope = st.gain / (float)st.dg;
    }
    return st;
}
// rs_up_cpu
template <class Args>
__device__ __forceinline__ RsStep rs_up_cpu_rows(const Args &A, const RsRows &R, int32_t gi, uint32_t ci, uint32_t lane) {
    RsStep st = {0u, gi, ci, 0.f, 0.f, 0ull, 0ull};
    if (gi < 0) return st;
    const float cur = rs_lane_f(R.best, gi);
    const uint32_t g = rs_lane_u(R.g, gi);
    const unsigned long long here = cpu_cost(A.X.grid, ci, g);
    uint32_t key = 0;                                      // likewise, the lowest level among equal slopes
    if (lane > ci && lane < A.X.grid.n_cpu && R.col > cur) {
        const float sl = ((R.col - cur) / R.ref) / (float)(cpu_cost(A.X.grid, lane, g) - here);
        if (sl > 0.f) key = __float_as_uint(sl);
    }
    const uint32_t top = wave_max_u32_rows(key);
    if (top) {
        const uint32_t c = (uint32_t)__ffsll((long long)__ballot(key == top)) - 1u;
        st.any = 1u; st.lvl = c;
        st.dc = cpu_cost(A.X.grid, c, g) - here;
        st.gain = (rs_lane_f(R.col, (int32_t)c) - cur) / R.ref;
        st.slope = st.gain / (float)st.dc;
    }
    return st;
}

// Job v, which holds (gi, ci), steps down in GPUs (res 0) or one CPU level (res 1): what it gives, what it holds then,
// and what it would lose per GPU / CPU given after that (infinite: nothing to give).
struct RsShrunk { RsGive gv; int32_t gi; uint32_t ci; float ds_g, ds_c; };
// ... after it gave gv, `lanes` threads sharing the searches (1, or the 64 of a wavefront)
template <class Args>
__device__ __forceinline__ RsShrunk rs_shrunk_at(const Args &A, uint32_t v, uint32_t res, int32_t gi, uint32_t ci, const RsGive &gv,
                                                 uint32_t lane, uint32_t lanes) {
    RsShrunk out;
    out.gv = gv;
    out.gi = res == 0 ? gv.tgt : gi;
    out.ci = res == 0 ? (gv.tgt < 0 ? 0u : ci) : ci - 1u;           // (with nothing left, every step down is none)
    const RsGive a = rs_down_gpu_at(A, v, out.gi, out.ci, lane, lanes), b = rs_down_cpu_at(A, v, out.gi, out.ci);
    out.ds_g = a.any ? a.slope : __int_as_float(0x7F800000);
    out.ds_c = b.any ? b.slope : __int_as_float(0x7F800000);
    return out;
}
// ... for a wavefront that has the job's rows
template <class Args>
__device__ __forceinline__ RsShrunk rs_shrunk_rows(const Args &A, const RsRows &R, uint32_t res, int32_t gi, uint32_t ci, const RsGive &gv,
                                                   uint32_t lane) {
    RsShrunk out;
    RsGive a, b;
    out.gv = gv;
    if (res == 0) {
        out.gi = gv.tgt;
        out.ci = gv.tgt < 0 ? 0u : ci;
        a = rs_down_gpu_rows(A, R, R.curve, out.gi, ci, lane);
        b = rs_down_cpu_rows(A, R, out.gi, out.ci, rs_lane_f(R.best, out.gi), rs_lane_f(R.best_lo, out.gi));
    } else {
        out.gi = gi;
        out.ci = ci - 1u;
        a = rs_down_gpu_rows(A, R, R.curve_lo, gi, out.ci, lane);
        b = rs_down_cpu_rows(A, R, gi, out.ci, rs_lane_f(R.col, (int32_t)out.ci), rs_lane_f(R.col, (int32_t)out.ci - 1));
    }
    out.ds_g = a.any ? a.slope : __int_as_float(0x7F800000);
    out.ds_c = b.any ? b.slope : __int_as_float(0x7F800000);
    return out;
}
// A whole wavefront calls; every lane gets the result.
template <class Args>
__device__ __forceinline__ RsShrunk rs_shrink_wave(const Args &A, uint32_t v, uint32_t so, uint32_t ns, uint32_t res, int32_t gi, uint32_t ci,
                                                   uint32_t lane) {
    if (ns > 64u) {
        const RsGive gv = res == 0 ? rs_down_gpu_at(A, v, gi, ci, lane, 64) : rs_down_cpu_at(A, v, gi, ci);
        return rs_shrunk_at(A, v, res, gi, ci, gv, lane, 64);
    }
    const RsRows R = rs_rows(A, v, so, ns, gi, ci, lane);
    const RsGive gv = res == 0 ? rs_down_gpu_rows(A, R, R.curve, gi, ci, lane)
                               : rs_down_cpu_rows(A, R, gi, ci, rs_lane_f(R.best, gi), rs_lane_f(R.best_lo, gi));
    return rs_shrunk_rows(A, R, res, gi, ci, gv, lane);
}

// What the loop over totals keeps of a job in the state a step finds it in, so that neither its own next steps nor the
// first step down that it is asked for wait for its rows: both steps up, and both steps down with the slopes after them.
// Whoever finds one of the four steps writes its two pieces, 16 bytes at a time.
struct __align__(16) RsNext {
    float ug; uint32_t dg; float gain_g; int32_t tgt_g;              // the GPU step (tgt_g -1: none)
    uint32_t lvl_g, below_ns; unsigned long long dcg;                // below_ns: its number of amounts, RS_BELOW when it is below its floor
    float uc, gain_c; uint32_t lvl_c; int32_t slot;                  // the CPU step (uc 0: none); the job's place in the list of holders, -1: none
    unsigned long long dcc; int32_t gi; uint32_t so;                 // the amount it holds; where its amounts begin in the plan table
};
struct __align__(16) RsGives {                                        // (of a job that holds something)
    uint32_t dg0; float loss0; uint32_t gis; float ds_g0;            // a step down in GPUs; gis: amounts before << 16 | after (0xFFFF: none)
    float ds_c0, ds_g; unsigned long long dc0;                       // ds_g, ds_c: the slopes in this state, ds_*0 and ds_*1 after the step
    float loss1, ds_g1, ds_c1, ds_c;                                 // a CPU level down
    unsigned long long dc1; uint32_t ci_ns, so;                      // the level before, its number of amounts << 8, where they begin
};
static_assert(sizeof(RsNext) == 64 && sizeof(RsGives) == 64, "four pieces each");
constexpr uint32_t RS_BELOW = 0x80000000u;
struct RsKept { float ds_g, ds_c, ug, uc; uint32_t dg, g; };

// The parts of it: steps up and down in GPUs and in CPUs, each found and stored by itself.
constexpr uint32_t RS_UP_G = 1u, RS_DOWN_G = 2u, RS_UP_C = 4u, RS_DOWN_C = 8u, RS_ALL_PARTS = 15u;

// Finds and stores the given parts for job v, which holds (gi, ci); LANES: the 64 of a wavefront, which has the rows
// of a job of at most 64 amounts at once, or 1.  so, ns: where the job's amounts begin and how many they are; gives: where
// the steps down go; also: where else the steps up go, or null.  (g, the GPUs it holds: with the step up in GPUs.)
template <uint32_t LANES, class Args>
__device__ __forceinline__ RsKept rs_keep(const Args &A, uint32_t v, uint32_t so, uint32_t ns, int32_t gi, uint32_t ci, int32_t slot, uint32_t lane,
                                          uint32_t parts, RsGives *gives, RsNext *also) {
    const float INF = __int_as_float(0x7F800000);
    const int32_t fl = rs_fl_s(A, v);
    const bool below = fl >= 0 && gi < fl, rows = LANES == 64u && ns <= 64u && !below;
    RsRows R = {};
    if (rows) R = rs_rows(A, v, so, ns, gi, ci, lane);
    RsKept k = {INF, INF, 0.f, 0.f, 0u, 0u};
    auto store = [](void *to, uint32_t a, uint32_t b, uint32_t c, uint32_t d) { *static_cast<uint4 *>(to) = uint4{a, b, c, d}; };
    if (parts & RS_UP_G) {
        const RsStep u = rows ? rs_up_gpu_rows(A, R, gi, ci, lane) : rs_up_gpu(A, v, gi, ci, lane, LANES);
        k.g = rows ? rs_lane_u(R.g, gi) : (uint32_t)rs_g(A, v, gi);
        k.ug = u.any ? u.slope : 0.f; k.dg = (uint32_t)u.dg;
        if (lane == 0) {
            auto up = [&](RsNext *to) {
                store(&to->ug, __float_as_uint(k.ug), k.dg, __float_as_uint(u.gain), u.any ? (uint32_t)u.tgt : 0xFFFFFFFFu);
                store(&to->lvl_g, u.lvl, ns | (below ? RS_BELOW : 0u), (uint32_t)u.dc, (uint32_t)(u.dc >> 32));
            };
            up(A.next + v);
            if (also) up(also);
        }
    }
    if (parts & RS_DOWN_G) {
        const RsGive a = rows ? rs_down_gpu_rows(A, R, R.curve, gi, ci, lane) : rs_down_gpu_at(A, v, gi, ci, lane, LANES);
        k.ds_g = a.any ? a.slope : INF;
        RsShrunk s = {a, -1, 0u, INF, INF};
        if (a.any) s = rows ? rs_shrunk_rows(A, R, 0, gi, ci, a, lane) : rs_shrunk_at(A, v, 0, gi, ci, a, lane, LANES);
        if (lane == 0 && gi >= 0) {
            store(&gives->dg0, (uint32_t)a.dg, __float_as_uint(a.loss), ((uint32_t)gi << 16) | ((uint32_t)s.gi & 0xFFFFu), __float_as_uint(s.ds_g));
            store(&gives->ds_c0, __float_as_uint(s.ds_c), __float_as_uint(k.ds_g), (uint32_t)a.dc, (uint32_t)(a.dc >> 32));
        }
    }
    if (parts & RS_UP_C) {
        const RsStep u = rows ? rs_up_cpu_rows(A, R, gi, ci, lane) : rs_up_cpu(A, v, gi, ci, lane, LANES);
        k.uc = u.any ? u.slope : 0.f;
        if (lane == 0) {
            auto up = [&](RsNext *to) {
                store(&to->uc, __float_as_uint(k.uc), __float_as_uint(u.gain), u.lvl, (uint32_t)slot);
                store(&to->dcc, (uint32_t)u.dc, (uint32_t)(u.dc >> 32), (uint32_t)gi, so);
            };
            up(A.next + v);
            if (also) up(also);
        }
    }
    if (parts & RS_DOWN_C) {
        const RsGive b = rows ? rs_down_cpu_rows(A, R, gi, ci, rs_lane_f(R.best, gi), rs_lane_f(R.best_lo, gi)) : rs_down_cpu_at(A, v, gi, ci);
        k.ds_c = b.any ? b.slope : INF;
        RsShrunk s = {b, -1, 0u, INF, INF};
        if (b.any) s = rows ? rs_shrunk_rows(A, R, 1, gi, ci, b, lane) : rs_shrunk_at(A, v, 1, gi, ci, b, lane, LANES);
        if (lane == 0 && gi >= 0) {
            store(&gives->loss1, __float_as_uint(b.loss), __float_as_uint(s.ds_g), __float_as_uint(s.ds_c), __float_as_uint(k.ds_c));
            store(&gives->dc1, (uint32_t)b.dc, (uint32_t)(b.dc >> 32), ci | (ns << 8), so);
        }
    }
    return k;
}

// What the lanes of a wavefront stored so far is seen by all its lanes from here on: the hardware keeps a wavefront's
// accesses in order, so only the compiler has to.
__device__ __forceinline__ void rs_wave_order() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// A workgroup barrier that orders LDS traffic only: every wavefront waits for its own LDS operations, not for its
// global loads and stores, which __syncthreads() would also drain.  Enough where what is exchanged is in LDS.
__device__ __forceinline__ void rs_lds_barrier() {
    asm volatile("" ::: "memory");               // the compiler keeps memory accesses on their side of the barrier
    __builtin_amdgcn_s_waitcnt(0xC07F);          // vmcnt 63, expcnt 7, lgkmcnt 0
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A float as an unsigned word that orders the same way (-0 as +0), and back.
__device__ __forceinline__ uint32_t rs_ordered(float x) {
    const uint32_t b = __float_as_uint(x + 0.f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float rs_unordered(uint32_t u) { return __uint_as_float((u & 0x80000000u) ? (u & 0x7FFFFFFFu) : ~u); }

// The job that comes first in the loops' order (GPU slope, then CPU slope, both descending, then the lower index)
// among the candidates of a workgroup's threads (j == 0xFFFFFFFF: a thread without one; slopes are not negative).
// All threads call and all get the result.  The slopes travel as one key of two words that order like them, the
// wavefronts reduce by DPP, the first one reduces their results; sh_key and sh_j hold WAVES + 1 entries.
struct RsPick { float g, c; uint32_t j; };
template <int WAVES>
__device__ __forceinline__ RsPick rs_pick_first(float g, float c, uint32_t j, uint32_t lane, uint32_t wave,
                                                unsigned long long *sh_key, uint32_t *sh_j) {
    const uint32_t NONE = 0xFFFFFFFFu;
    const uint32_t kg = j == NONE ? 0u : rs_ordered(g), kc = j == NONE ? 0u : rs_ordered(c);
    const uint32_t top_g = wave_max_u32_rows(kg), top_c = wave_max_u32_rows(kg == top_g ? kc : 0u);
    const uint32_t first = wave_min_u32_rows(j != NONE && kg == top_g && kc == top_c ? j : NONE);
    if (lane == 0) { sh_key[wave] = ((unsigned long long)top_g << 32) | top_c; sh_j[wave] = first; }
    rs_lds_barrier();
    if (wave == 0) {
        const unsigned long long k2 = lane < WAVES ? sh_key[lane] : 0ull;
        const uint32_t j2 = lane < WAVES ? sh_j[lane] : NONE;
        const uint32_t g2 = (uint32_t)(k2 >> 32), c2 = (uint32_t)k2;
        const uint32_t tg = wave_max_u32_rows(g2), tc = wave_max_u32_rows(g2 == tg ? c2 : 0u);
        const uint32_t f2 = wave_min_u32_rows(g2 == tg && c2 == tc ? j2 : NONE);
        if (lane == 0) { sh_key[WAVES] = ((unsigned long long)tg << 32) | tc; sh_j[WAVES] = f2; }
    }
    rs_lds_barrier();
    RsPick out;
    const unsigned long long t = sh_key[WAVES];
    out.j = sh_j[WAVES];
    out.g = rs_unordered((uint32_t)(t >> 32));
    out.c = rs_unordered((uint32_t)t);
    return out;
}

// The two lowest give-slopes over all jobs, per resource, and the job of the lowest (the lower index among equal
// values; none: 0xFFFFFFFF with both values infinite).  ds holds the slopes [2][n_jobs] (LDS).  All THREADS threads of
// the workgroup call and all get the result in out[0] (GPUs) and out[1] (CPUs).  Every thread keeps the two lowest
// of its own jobs; the lowest goes through DPP minima, first of the slope as a word that orders like it, then of the job,
// the second lowest is the minimum of what the threads hold once the lowest's owner puts its own second in.
// sh_k and sh_s hold 2 * (WAVES + 1) entries each.
struct RsMin { float m1, m2; uint32_t i1; };
template <int WAVES, int THREADS>
__device__ __forceinline__ void rs_two_lowest(const float *ds, uint32_t n_jobs, uint32_t tid, uint32_t lane, uint32_t wave,
                                              unsigned long long *sh_k, uint32_t *sh_s, RsMin (&out)[2]) {
    const float INF = __int_as_float(0x7F800000);
    const uint32_t NONE = 0xFFFFFFFFu;
    float a[2] = {INF, INF}, b[2] = {INF, INF};
    uint32_t ia[2] = {NONE, NONE};
    for (uint32_t v0 = tid; v0 < n_jobs; v0 += 4 * THREADS) {            // four loads per resource in flight
        float x[2][4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t v = v0 + k * THREADS;
            x[0][k] = v < n_jobs ? ds[v] : INF;
            x[1][k] = v < n_jobs ? ds[n_jobs + v] : INF;
        }
#pragma unroll
        for (uint32_t r = 0; r < 2; ++r)
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {                           // ascending jobs: the lower one stays among equals
                const float y = x[r][k];
                if (y < a[r]) { b[r] = a[r]; a[r] = y; ia[r] = v0 + k * THREADS; }
                else if (y < b[r]) b[r] = y;
            }
    }
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r) {
        const uint32_t low = ia[r] == NONE ? NONE : rs_ordered(a[r]), low_w = wave_min_u32_rows(low);
        const uint32_t who_w = wave_min_u32_rows(low == low_w ? ia[r] : NONE);
        if (lane == 0) sh_k[r * (WAVES + 1) + wave] = ((unsigned long long)low_w << 32) | who_w;
    }
    rs_lds_barrier();
    if (wave == 0) {
#pragma unroll
        for (uint32_t r = 0; r < 2; ++r) {
            const unsigned long long k = lane < WAVES ? sh_k[r * (WAVES + 1) + lane] : ~0ull;
            const uint32_t l2 = (uint32_t)(k >> 32), low = wave_min_u32_rows(l2);
            const uint32_t who = wave_min_u32_rows(l2 == low ? (uint32_t)k : NONE);
            if (lane == 0) sh_k[r * (WAVES + 1) + WAVES] = ((unsigned long long)low << 32) | who;
        }
    }
    rs_lds_barrier();
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r) {
        const unsigned long long low = sh_k[r * (WAVES + 1) + WAVES];
        out[r].i1 = low == ~0ull ? NONE : (uint32_t)low;
        out[r].m1 = low == ~0ull ? INF : rs_unordered((uint32_t)(low >> 32));
        // what this thread holds beside the lowest: its own lowest, or its second when the lowest is its own
        const float mine = (ia[r] != NONE && ia[r] == out[r].i1) ? b[r] : a[r];
        const uint32_t w = wave_min_u32_rows(rs_ordered(mine));
        if (lane == 0) sh_s[r * (WAVES + 1) + wave] = w;
    }
    rs_lds_barrier();
    if (wave == 0) {
#pragma unroll
        for (uint32_t r = 0; r < 2; ++r) {
            const uint32_t w = wave_min_u32_rows(lane < WAVES ? sh_s[r * (WAVES + 1) + lane] : rs_ordered(INF));
            if (lane == 0) sh_s[r * (WAVES + 1) + WAVES] = w;
        }
    }
    rs_lds_barrier();
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r) out[r].m2 = rs_unordered(sh_s[r * (WAVES + 1) + WAVES]);
}
