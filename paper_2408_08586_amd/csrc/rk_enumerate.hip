// Plan enumeration on the device (paper Sec. 3: 3D-parallel plans with
// d*t*p = g, Table 1; Fig. 6: only some GPU counts are valid).
//
// One workgroup per job.  Instead of testing every g it builds the divisor
// lists of b/mu (data-parallel sizes) and of the layer count (pipeline sizes),
// forms the products d*t*p <= g_max with t in {1,2,4,8} for every allowed
// micro-batch shift v (d must divide b/(mu*2^v)), and orders them by the key
// (g, t, p, v) in LDS.  Up to 256 keys, as most jobs have, find their places by
// counting the smaller ones, a thread per key.  More of them go by a bitmap of
// the GPU counts that occur: it gives every key its segment (rank of its g among
// the distinct counts = a population count), the keys are gathered by segment,
// and only the few keys of one segment are compared with each other.
// The counting pass also parks the triples it found, in the table's own words,
// in a scratch buffer (512 words per job at first, then the widest job's triples
// and a quarter more, at most 2,048).  After the exclusive scan of the counts the
// table's content is made from the parked words: by the fill pass (k_fill, a
// wavefront per job, which marks where a new GPU count begins), or in a scheduling
// round that is evaluated ahead by k_fused.  Either is launched while the counts are
// still on their way to the host: it checks on the device that the table is
// large enough and leaves it alone otherwise.  (The search is repeated only when
// the scratch buffer was too small.)
// Jobs whose searches would be identical (same layer count, same number of
// micro-batches per step) share one: a hash table names a leader for each such
// group, only leaders search, the others take the leader's counts and copy the
// leader's parked words.
//
// Small calls are bound by their launches, so up to ENUM_SELF_SCAN jobs are
// scanned by the workgroup that finishes its search last, which also writes
// the totals straight to pinned host memory (two launches instead of four and
// a copy); large ones by all workgroups of k_scan_tiles from the sums that
// k_spread_counts leaves (128,000 jobs: 73 us with one workgroup, 4 us).  The
// fill was 114 us for them while it decoded keys and counted segments in LDS
// again, 31 us as a copy (28 us with the segments parked as well, for half as
// much scratch again); 10,000 jobs: 14 -> 8 us and the scan 13 -> 4 us.
#include <cstring>

#include "rk_internal.h"

namespace {

constexpr int ENUM_THREADS = 256;
constexpr uint32_t MAX_T = RK_MAX_TRIPLES_PER_JOB;
constexpr uint32_t MAX_DIV = 1024;

enum { ERR_TOO_MANY_TRIPLES = 1, ERR_TOO_MANY_DIVISORS = 2, ERR_PARK_FULL = 4 };
enum { MODE_COUNT = 0, MODE_FILL_SEARCH = 1 };

// a job's word in cnt_t: its triples and the flags its search raised (so nothing has to be cleared between calls)
constexpr uint32_t CNT_MASK = 0xFFFFFFu, CNT_FLAGS = 24u;
static_assert(MAX_T <= CNT_MASK, "the count and the flags share a word");

// What the scan of the counts leaves: offsets in the table, totals for the fill pass, and both for the host.
struct ScanOut {
    uint32_t *off_t, *off_s;   // n_jobs + 1 each
    uint32_t *totals;
    uint32_t *back;            // [16 words of totals | n_jobs + 1 triple offsets | n_jobs + 1 segment offsets], one piece for the host
    uint32_t back_offsets;     // ... the offsets only when the host keeps mirrors of them
};

__device__ __forceinline__ void write_totals(const ScanOut &S, uint32_t n_jobs, uint64_t nt, uint64_t ns, uint32_t mt, uint32_t ms,
                                             uint32_t err) {
    S.off_t[n_jobs] = (uint32_t)nt; S.off_s[n_jobs] = (uint32_t)ns;
    for (uint32_t *to : {S.totals, S.back}) {
        to[TOT_NT_LO] = (uint32_t)nt; to[TOT_NT_HI] = (uint32_t)(nt >> 32);
        to[TOT_NS_LO] = (uint32_t)ns; to[TOT_NS_HI] = (uint32_t)(ns >> 32);
        to[TOT_MAX_T] = mt; to[TOT_MAX_S] = ms; to[TOT_ERR] = err;
    }
    if (S.back_offsets) { S.back[16 + n_jobs] = (uint32_t)nt; S.back[16 + 2 * n_jobs + 1] = (uint32_t)ns; }
}
__device__ __forceinline__ void write_offsets(const ScanOut &S, uint32_t n_jobs, uint32_t j, uint32_t t, uint32_t s) {
    S.off_t[j] = t; S.off_s[j] = s;
    if (S.back_offsets) { S.back[16 + j] = t; S.back[16 + n_jobs + 1 + j] = s; }
}

// exclusive prefix sum of one value per thread over the workgroup (all threads call it): inside the
// wavefronts by DPP (rows of 16, then each row's sum into the rows behind it), then the wavefronts' totals through
// LDS (lds: one word per wavefront)
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t *lds, uint32_t *total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t incl = v;
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x111, 0xF, 0xF, false);     // row_shr:1, 2, 4, 8
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x112, 0xF, 0xF, false);
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x114, 0xF, 0xF, false);
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x118, 0xF, 0xF, false);
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x142, 0xA, 0xF, false);     // row_bcast:15 into rows 1 and 3
    incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x143, 0xC, 0xF, false);     // row_bcast:31 into rows 2 and 3
    if (lane == 63u) lds[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (uint32_t w = 0; w < ENUM_THREADS / 64; ++w) {
        if (w < wave) before += lds[w];
        all += lds[w];
    }
    *total = all;
    __syncthreads();
    return before + incl - v;
}

// What the search of a job depends on (besides the bounds of the call): its layer count and b/mu; (0, 0) for a
// job that has no plan at all.
__device__ __forceinline__ void search_key(uint32_t l, uint32_t b, uint32_t mu, uint32_t &kl, uint32_t &kn) {
    const bool any = l > 0 && b > 0 && mu > 0 && (b % mu) == 0;
    kl = any ? l : 0u;
    kn = any ? b / mu : 0u;
}

__device__ __forceinline__ uint32_t search_hash(uint32_t kl, uint32_t kn) {
    uint32_t h = (kl * 0x9E3779B1u) ^ (kn * 0x85EBCA77u);
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    return h;
}

// leader[j] = the job whose search job j shares (itself for the leaders).  Open addressing with linear probing,
// an entry is a job index + 1 and never changes once set; the table has at least twice as many slots as there are
// jobs, so every probe sequence ends at an empty slot or at the job's own kind, and nobody waits for anybody.
// Equal jobs of a workgroup first elect one of them through a table in LDS; only that one goes to the global table.
constexpr int LEAD_THREADS = 256;
constexpr uint32_t SHARE_MIN_JOBS = 2048;                  // calls with fewer jobs do not look for equal ones
constexpr uint32_t SCAN_MOST_TILES = 4096;                 // beyond 2^20 jobs one workgroup scans (every tile reads all before it)
// A thread scans two neighbouring jobs.  Of more jobs the workgroups queue at the counter: a round of 500 jobs took 90.9 us
// with the scan in here and 95.0 with one of its own, one of 1,000 jobs 101.3 and 98.3, one of 2,000 139.6 and 128.8.
constexpr uint32_t ENUM_SELF_SCAN = 2 * ENUM_THREADS;
// Beyond this many jobs the leaders are listed and so many workgroups take them in turn.  With a workgroup per job, of which
// nearly all have nothing to do, 128,000 jobs of 45 kinds took 117 us, now 96, of 3,000 kinds 129 and 112, 60,000 of 45 kinds
// 76 and 67; where nearly all jobs are kinds of their own, which is not what jobs are like, the list costs more than it saves
// (128,000 of 100,000 kinds 280 and 303, with 2,048 workgroups 378: searches differ in length).  10,000 jobs: 48.9 and 50.9.
// (All of these with the offsets still copied to the host, which took another 15 us.)
constexpr uint32_t ENUM_TURNS = 16384;

__global__ __launch_bounds__(LEAD_THREADS) void k_enum_leaders(const uint32_t *__restrict__ layers,
                                                               const uint32_t *__restrict__ gbatch,
                                                               const uint32_t *__restrict__ mbatch, uint32_t n_jobs,
                                                               uint32_t *__restrict__ tab, uint32_t tab_mask,
                                                               uint32_t *__restrict__ leader, uint32_t *__restrict__ list, uint32_t *n_list) {
    __shared__ uint32_t ltab[2 * LEAD_THREADS], s_kl[LEAD_THREADS], s_kn[LEAD_THREADS], s_lead[LEAD_THREADS], s_n, s_at;
    const uint32_t tid = threadIdx.x, j = blockIdx.x * LEAD_THREADS + tid;
    const bool valid = j < n_jobs;
    uint32_t kl = 0, kn = 0;
    if (valid) search_key(layers[j], gbatch[j], mbatch[j], kl, kn);
    s_kl[tid] = kl;
    s_kn[tid] = kn;
    ltab[tid] = 0u;
    ltab[tid + LEAD_THREADS] = 0u;
    if (tid == 0) s_n = 0u;
    __syncthreads();
    const uint32_t h = search_hash(kl, kn);
    uint32_t rep = tid;                                     // the thread that speaks for this job's kind
    if (valid) {
        uint32_t slot = h & (2u * LEAD_THREADS - 1u);
        for (;;) {
            const uint32_t old = atomicCAS(&ltab[slot], 0u, tid + 1u);
            if (old == 0u) break;
            if (s_kl[old - 1u] == kl && s_kn[old - 1u] == kn) { rep = old - 1u; break; }
            slot = (slot + 1u) & (2u * LEAD_THREADS - 1u);
        }
    }
    uint32_t at = UINT32_MAX;                               // a leader's place among those of the workgroup
    if (valid && rep == tid) {
        uint32_t slot = h & tab_mask, lead = j;
        for (;;) {
            const uint32_t old = atomicCAS(&tab[slot], 0u, j + 1u);
            if (old == 0u) { if (list) at = atomicAdd(&s_n, 1u); break; }
            const uint32_t o = old - 1u;
            uint32_t ol, on;
            search_key(layers[o], gbatch[o], mbatch[o], ol, on);
            if (ol == kl && on == kn) { lead = o; break; }
            slot = (slot + 1u) & tab_mask;
        }
        s_lead[tid] = lead;
    }
    __syncthreads();
    if (valid) leader[j] = s_lead[rep];
    if (!list || s_n == 0u) return;
    if (tid == 0) s_at = atomicAdd(n_list, s_n);            // (one by one they took 40 us for 100,000 leaders)
    __syncthreads();
    if (at != UINT32_MAX) list[s_at + at] = j;
}

// the counts of a job that did not search are its leader's; sums and maxima of every workgroup's jobs for k_scan_tiles
struct TileSum { unsigned long long t, s; uint32_t mt, ms, err, pad; };

__global__ __launch_bounds__(LEAD_THREADS) void k_spread_counts(const uint32_t *__restrict__ leader, uint32_t n_jobs,
                                                                uint32_t *__restrict__ cnt_t, uint32_t *__restrict__ cnt_s,
                                                                TileSum *__restrict__ sums, uint32_t *__restrict__ tab, uint32_t tab_slots,
                                                                uint32_t *__restrict__ n_list) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_list = 0u;     // (all searches have been made)
    // the leaders' table has been read: zero for the next call (a launch of its own before it took 5 us)
    for (uint32_t i = blockIdx.x * LEAD_THREADS + threadIdx.x; i < tab_slots / 4u; i += gridDim.x * LEAD_THREADS)
        reinterpret_cast<uint4 *>(tab)[i] = uint4{0u, 0u, 0u, 0u};
    __shared__ uint32_t w_t[LEAD_THREADS / 64], w_s[LEAD_THREADS / 64], w_mt[LEAD_THREADS / 64], w_ms[LEAD_THREADS / 64], w_e[LEAD_THREADS / 64];
    const uint32_t j = blockIdx.x * LEAD_THREADS + threadIdx.x;
    uint32_t ct = 0, cs = 0;
    if (j < n_jobs) {
        const uint32_t l = leader[j];
        ct = cnt_t[l]; cs = cnt_s[l];
        if (l != j) { cnt_t[j] = ct; cnt_s[j] = cs; }
    }
    uint32_t err = ct >> CNT_FLAGS, st = ct & CNT_MASK, ss = cs, mt = st, ms = cs;   // (256 jobs of at most 2,048 triples)
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t a = __shfl_xor(mt, off, 64), b = __shfl_xor(ms, off, 64);
        mt = a > mt ? a : mt; ms = b > ms ? b : ms;
        st += __shfl_xor(st, off, 64); ss += __shfl_xor(ss, off, 64); err |= __shfl_xor(err, off, 64);
    }
    const uint32_t w = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0) { w_t[w] = st; w_s[w] = ss; w_mt[w] = mt; w_ms[w] = ms; w_e[w] = err; }
    __syncthreads();
    if (threadIdx.x == 0) {
        TileSum o = {0ull, 0ull, 0u, 0u, 0u, 0u};
        for (uint32_t k = 0; k < LEAD_THREADS / 64; ++k) {
            o.t += w_t[k]; o.s += w_s[k]; o.err |= w_e[k];
            o.mt = w_mt[k] > o.mt ? w_mt[k] : o.mt; o.ms = w_ms[k] > o.ms ? w_ms[k] : o.ms;
        }
        sums[blockIdx.x] = o;
    }
}

// Exclusive scan of the counts, a workgroup per LEAD_THREADS jobs: what lies before them is the sum over the workgroups
// before (a few loads per thread up to the 4,096 workgroups this is used for), the rest a scan of its own.
__global__ __launch_bounds__(LEAD_THREADS) void k_scan_tiles(const uint32_t *__restrict__ cnt_t, const uint32_t *__restrict__ cnt_s,
                                                             uint32_t n_jobs, const TileSum *__restrict__ sums, ScanOut S) {
    static_assert(LEAD_THREADS == ENUM_THREADS, "block_excl_scan");
    __shared__ uint32_t tmp[ENUM_THREADS / 64];
    __shared__ unsigned long long b_t[LEAD_THREADS / 64], b_s[LEAD_THREADS / 64];
    __shared__ uint32_t b_mt[LEAD_THREADS / 64], b_ms[LEAD_THREADS / 64], b_e[LEAD_THREADS / 64];
    const uint32_t tid = threadIdx.x, j = blockIdx.x * LEAD_THREADS + tid;
    const bool last = blockIdx.x == gridDim.x - 1;
    const uint32_t ct = j < n_jobs ? cnt_t[j] & CNT_MASK : 0u, cs = j < n_jobs ? cnt_s[j] : 0u;
    unsigned long long bt = 0, bs = 0;
    uint32_t mt = 0, ms = 0, err = 0;
    for (uint32_t k = tid; k < blockIdx.x + (last ? 1u : 0u); k += LEAD_THREADS) {   // (the last one also closes the totals)
        const TileSum o = sums[k];
        if (k < blockIdx.x) { bt += o.t; bs += o.s; }
        mt = o.mt > mt ? o.mt : mt; ms = o.ms > ms ? o.ms : ms; err |= o.err;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t a = __shfl_xor(mt, off, 64), b = __shfl_xor(ms, off, 64);
        mt = a > mt ? a : mt; ms = b > ms ? b : ms;
        bt += __shfl_xor(bt, off, 64); bs += __shfl_xor(bs, off, 64); err |= __shfl_xor(err, off, 64);
    }
    const uint32_t w = tid >> 6;
    if ((tid & 63u) == 0) { b_t[w] = bt; b_s[w] = bs; b_mt[w] = mt; b_ms[w] = ms; b_e[w] = err; }
    uint32_t all_t, all_s;
    const uint32_t et = block_excl_scan(ct, tmp, &all_t), es = block_excl_scan(cs, tmp, &all_s);   // (also the barrier after b_*)
    bt = 0; bs = 0; mt = 0; ms = 0; err = 0;
#pragma unroll
    for (uint32_t k = 0; k < LEAD_THREADS / 64; ++k) {
        bt += b_t[k]; bs += b_s[k]; err |= b_e[k];
        mt = b_mt[k] > mt ? b_mt[k] : mt; ms = b_ms[k] > ms ? b_ms[k] : ms;
    }
    if (j < n_jobs) write_offsets(S, n_jobs, j, (uint32_t)(bt + et), (uint32_t)(bs + es));
    if (last && tid == 0) write_totals(S, n_jobs, bt + all_t, bs + all_s, mt, ms, err);
}

// LISTED: the workgroups take the jobs in list, *n_list of them, in turn; else job blockIdx.x, if it is a leader.
// self_scan != 0: the workgroup that ends last also scans the counts (n_jobs <= ENUM_SELF_SCAN, no leaders).
// The counter of finished workgroups starts at zero and is left at zero by the one that ends last: what it has to be is
// known on the device alone, whatever became of the calls before (one that ended in an error, one that was only recorded).
template <int MODE, bool LISTED>
__global__ __launch_bounds__(ENUM_THREADS) void k_enumerate(
    const uint32_t *__restrict__ layers, const uint32_t *__restrict__ gbatch,
    const uint32_t *__restrict__ mbatch, rk_plan_bounds bounds, const uint32_t *__restrict__ leader,
    const uint32_t *__restrict__ list, const uint32_t *__restrict__ n_list, uint32_t *cnt_t, uint32_t *cnt_s, uint32_t *__restrict__ park, uint32_t park_stride,
    const uint32_t *__restrict__ triple_off, const uint32_t *__restrict__ seg_off,
    uint32_t *__restrict__ triples, uint32_t *__restrict__ seg_g, uint32_t *__restrict__ seg_first,
    uint32_t self_scan, ScanOut S) {
    extern __shared__ uint32_t gmap[];                      // counting and search modes: bitmap of the GPU counts, word prefixes
    // Two arrays serve everything (a third would cost occupancy): `lists` holds the two divisor lists and later
    // the keys gathered by segment; `keys` holds the keys as they are found, then (once every thread has its keys
    // in registers) the segments' sizes and starts, and at the end the keys in order.
    __shared__ uint32_t lists[2 * MAX_DIV];
    uint32_t *dlist = lists, *plist = lists + MAX_DIV;
    __shared__ __align__(16) uint32_t keys[MAX_T + 4];
    static_assert(TOT_WORDS <= 16, "the totals share a block with the leaders' table");
    static_assert(2 * MAX_DIV >= MAX_T, "the gathered keys reuse the divisor lists");
    __shared__ uint32_t scan_tmp[ENUM_THREADS];
    __shared__ uint32_t nd, np, nk;

    const uint32_t tid = threadIdx.x, n_search = LISTED ? *n_list : 0u;
    for (uint32_t turn = blockIdx.x; !LISTED || turn < n_search; turn += gridDim.x) {
    const uint32_t j = LISTED ? list[turn] : turn;
    if (MODE == MODE_COUNT && !LISTED && leader && leader[j] != j) return;   // (whole workgroup) the leader searches for this job
    if (LISTED && turn != blockIdx.x) __syncthreads();                    // (the turn before has read its arrays)
    uint32_t cnt, err = 0;
    const uint32_t *fin = keys;                                 // the keys in order
    {
        const uint32_t l = layers[j], b = gbatch[j], mu = mbatch[j];
        if (tid == 0) { nd = 0; np = 0; nk = 0; }
        __syncthreads();

        const bool any = l > 0 && b > 0 && mu > 0 && (b % mu) == 0;
        const uint32_t n = any ? b / mu : 0;
        // divisors of n (data-parallel sizes) and of l (pipeline sizes), unordered
        // (every divisor d with d*d <= n brings n/d along, so the search stops at the square root)
        const uint32_t dmax = n < bounds.g_max ? n : bounds.g_max;
        for (uint32_t d = tid + 1; (uint64_t)d * d <= n; d += ENUM_THREADS) {
            const uint32_t e = n / d;
            if (e * d == n) {
                if (d <= dmax) { uint32_t i = atomicAdd(&nd, 1u); if (i < MAX_DIV) dlist[i] = d; }
                if (e != d && e <= dmax) { uint32_t i = atomicAdd(&nd, 1u); if (i < MAX_DIV) dlist[i] = e; }
            }
        }
        uint32_t pmax = l < bounds.pp_max ? l : bounds.pp_max;
        pmax = pmax < bounds.g_max ? pmax : bounds.g_max;
        if (!any) pmax = 0;
        for (uint32_t p = tid + 1; p <= pmax; p += ENUM_THREADS)
            if (l % p == 0) { uint32_t i = atomicAdd(&np, 1u); if (i < MAX_DIV) plist[i] = p; }
        __syncthreads();
        if (nd > MAX_DIV || np > MAX_DIV) err |= ERR_TOO_MANY_DIVISORS;
        const uint32_t cd = nd < MAX_DIV ? nd : MAX_DIV, cp = np < MAX_DIV ? np : MAX_DIV;

        // products d * 2^lt * p <= g_max (at most 1024 * 1024 * 4 combinations: 32-bit arithmetic)
        uint32_t nlt = 0;                               // tensor-parallel sizes allowed: 2^0..2^(nlt-1)
        for (uint32_t t = 1; t <= 8 && t <= bounds.tp_max; t <<= 1) ++nlt;
        const uint32_t pairs = cd * cp;
        for (uint32_t c = tid; c < pairs; c += ENUM_THREADS) {
            const uint32_t p = plist[c % cp], d = dlist[c / cp];
            const uint64_t dp = (uint64_t)d * p;
            // micro-batch shifts this d works with: mu*2^v divides b and d divides b/(mu*2^v)
            uint32_t vmask = 0;
            for (uint32_t v = 0; v < 4; ++v)
                if (((bounds.mu_mask >> v) & 1u) && (n & ((1u << v) - 1u)) == 0 && ((n >> v) % d) == 0) vmask |= 1u << v;
            for (uint32_t lt = 0; lt < nlt; ++lt) {
                const uint64_t g = dp << lt;
                if (g <= bounds.g_max) {
                    for (uint32_t v = 0; v < 4; ++v) {
                        if (!((vmask >> v) & 1u)) continue;
                        const uint32_t i = atomicAdd(&nk, 1u);
                        if (i < MAX_T) keys[i] = ((uint32_t)g << 16) | (lt << 14) | (p << 2) | v;
                    }
                }
            }
        }
        __syncthreads();
        if (nk > MAX_T) err |= ERR_TOO_MANY_TRIPLES;
        cnt = nk < MAX_T ? nk : MAX_T;

        // Sort.  Keys are distinct.  A key per thread, at most: a key's place is the number of smaller ones, four of them per
        // read that goes to all lanes (8 jobs of 60 to 200 keys: 9.1 us for the kernel with the steps below and the caches written back for the counter, 6.8).
        if (cnt <= (uint32_t)ENUM_THREADS) {
            const uint32_t own = tid < cnt ? keys[tid] : 0xFFFFFFFFu, whole = cnt & ~3u;
            const uint4 *const k4 = reinterpret_cast<const uint4 *>(keys);
            uint32_t rank = 0;
            for (uint32_t q = 0; q < whole; q += 4u) {
                const uint4 k = k4[q / 4u];
                rank += (k.x < own ? 1u : 0u) + (k.y < own ? 1u : 0u) + (k.z < own ? 1u : 0u) + (k.w < own ? 1u : 0u);
            }
            for (uint32_t q = whole; q < cnt; ++q) rank += keys[q] < own ? 1u : 0u;
            if (tid < cnt) lists[rank] = own;                   // (the divisors have been read)
            fin = lists;
            __syncthreads();
        } else {
        // More of them: (1) bitmap of the GPU counts that occur; (2) population counts in front of
        // every bitmap word: a key's segment is the rank of its g among the distinct counts; (3) sizes of the
        // segments, every key takes a slot in its own; (4) starts of the segments; (5) keys gathered by segment;
        // (6) a key's final place = start of its segment + number of smaller keys inside it.
        constexpr uint32_t PER = MAX_T / ENUM_THREADS;          // keys per thread, at most
        const uint32_t n_words = (bounds.g_max >> 5) + 1u;
        uint32_t *bitmap = gmap, *before = gmap + n_words, *seg = keys, *gathered = lists;
        uint32_t mine[PER], slot[PER], place[PER];
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r) {
            const uint32_t i = tid + r * ENUM_THREADS;
            mine[r] = i < cnt ? keys[i] : 0u;
        }
        for (uint32_t w = tid; w < n_words; w += ENUM_THREADS) bitmap[w] = 0u;
        __syncthreads();                                        // every key is in a register: `keys` becomes the segment table
        for (uint32_t i = tid; i <= cnt; i += ENUM_THREADS) seg[i] = 0u;     // there are at most cnt segments
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r)
            if (tid + r * ENUM_THREADS < cnt) atomicOr(&bitmap[mine[r] >> 21], 1u << ((mine[r] >> 16) & 31u));
        __syncthreads();
        const uint32_t wpt = (n_words + ENUM_THREADS - 1) / ENUM_THREADS;
        const uint32_t w_lo = tid * wpt < n_words ? tid * wpt : n_words;
        const uint32_t w_hi = w_lo + wpt < n_words ? w_lo + wpt : n_words;
        uint32_t bits = 0;
        for (uint32_t w = w_lo; w < w_hi; ++w) bits += (uint32_t)__popc(bitmap[w]);
        uint32_t n_seg;
        uint32_t run = block_excl_scan(bits, scan_tmp, &n_seg);
        for (uint32_t w = w_lo; w < w_hi; ++w) { before[w] = run; run += (uint32_t)__popc(bitmap[w]); }
        __syncthreads();
        auto segment_of = [&](uint32_t key) -> uint32_t {
            const uint32_t g = key >> 16;
            return before[g >> 5] + (uint32_t)__popc(bitmap[g >> 5] & ((1u << (g & 31u)) - 1u));
        };
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r)
            if (tid + r * ENUM_THREADS < cnt) slot[r] = atomicAdd(&seg[segment_of(mine[r])], 1u);
        __syncthreads();
        const uint32_t spt = (n_seg + ENUM_THREADS - 1) / ENUM_THREADS;
        const uint32_t s_lo = tid * spt < n_seg ? tid * spt : n_seg;
        const uint32_t s_hi = s_lo + spt < n_seg ? s_lo + spt : n_seg;
        uint32_t sizes = 0, all;
        for (uint32_t q = s_lo; q < s_hi; ++q) sizes += seg[q];
        run = block_excl_scan(sizes, scan_tmp, &all);
        for (uint32_t q = s_lo; q < s_hi; ++q) { const uint32_t n = seg[q]; seg[q] = run; run += n; }
        if (tid == 0) seg[n_seg] = cnt;
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r)
            if (tid + r * ENUM_THREADS < cnt) gathered[seg[segment_of(mine[r])] + slot[r]] = mine[r];
        __syncthreads();
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r) {
            place[r] = 0;
            if (tid + r * ENUM_THREADS < cnt) {
                const uint32_t q = segment_of(mine[r]), a = seg[q], b = seg[q + 1];
                uint32_t rank = a;
                for (uint32_t x = a; x < b; ++x) rank += gathered[x] < mine[r] ? 1u : 0u;
                place[r] = rank;
            }
        }
        __syncthreads();                                        // the segment table has been read: `keys` takes the result
#pragma unroll
        for (uint32_t r = 0; r < PER; ++r)
            if (tid + r * ENUM_THREADS < cnt) keys[place[r]] = mine[r];
        __syncthreads();
        }
    }
    // segments: runs of equal g.  Each thread owns a contiguous chunk.
    const uint32_t chunk = (cnt + ENUM_THREADS - 1) / ENUM_THREADS;
    const uint32_t lo = tid * chunk < cnt ? tid * chunk : cnt;
    const uint32_t hi = lo + chunk < cnt ? lo + chunk : cnt;
    uint32_t starts = 0;
    for (uint32_t i = lo; i < hi; ++i)
        starts += (i == 0 || (fin[i] >> 16) != (fin[i - 1] >> 16)) ? 1u : 0u;
    uint32_t nseg;
    uint32_t sidx = block_excl_scan(starts, scan_tmp, &nseg);

    // the job's words go to its place in the table or, if they fit, to its slot of the parked words (k_fill finds the
    // segments again)
    const bool room = MODE != MODE_COUNT || cnt <= park_stride;
    const size_t at = MODE == MODE_COUNT ? (size_t)j * park_stride : triple_off[j];
    const uint32_t s0 = MODE == MODE_COUNT ? 0u : seg_off[j];
    for (uint32_t i = lo; i < hi && room; ++i) {
        const uint32_t k = fin[i];
        const uint32_t g = k >> 16, lt = (k >> 14) & 3u, p = (k >> 2) & 0xFFFu, v = k & 3u;
        const uint32_t d = g / (p << lt), word = d | (lt << 16) | (p << 18) | (v << 30);
        if (MODE == MODE_COUNT) { park[at + i] = word; continue; }
        triples[at + i] = word;
        if (i == 0 || g != (fin[i - 1] >> 16)) {
            seg_g[s0 + sidx] = g;
            seg_first[s0 + sidx] = i;
            ++sidx;
        }
    }
    if (MODE != MODE_COUNT) return;
    if (!room) err |= ERR_PARK_FULL;
    if (LISTED || !self_scan) {
        if (tid == 0) { cnt_t[j] = cnt | (err << CNT_FLAGS); cnt_s[j] = nseg; }
        if (LISTED) continue;
        return;
    }
    // Counts, then the counter, at the device's scope (the workgroups sit on several L2 caches).  A release at the counter would
    // write a whole L2 back for two words.  Instead this rests on what gfx950 does with atomic stores and loads at that scope,
    // not on the language's ordering of relaxed operations: a store is written through to where all of the device sees it and counts as done
    // only there, so when the wait before the counter is over the counts have arrived; the loads of the workgroup
    // that brings the counter to its end read from there too.  Nothing else is handed over here.
    __shared__ uint32_t ends;
    if (tid == 0) {
        __hip_atomic_store(&cnt_t[j], cnt | (err << CNT_FLAGS), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&cnt_s[j], nseg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        ends = __hip_atomic_fetch_add(&S.totals[TOT_DONE], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (ends != gridDim.x - 1u) return;
    if (tid == 0) S.totals[TOT_DONE] = 0u;                      // (for the next launch)
    constexpr uint32_t OWN = ENUM_SELF_SCAN / ENUM_THREADS;     // neighbouring jobs of a thread, at most
    const uint32_t own = (gridDim.x + ENUM_THREADS - 1u) / ENUM_THREADS, first = tid * own;
    uint32_t ct[OWN], cs[OWN], sum_t = 0, sum_s = 0, mt = 0, ms = 0, flags = 0, all_t, all_s;
#pragma unroll
    for (uint32_t i = 0; i < OWN; ++i) {
        const bool in = i < own && first + i < gridDim.x;
        ct[i] = in ? __hip_atomic_load(&cnt_t[first + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        cs[i] = in ? __hip_atomic_load(&cnt_s[first + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    }
#pragma unroll
    for (uint32_t i = 0; i < OWN; ++i) {
        flags |= ct[i] >> CNT_FLAGS;
        ct[i] &= CNT_MASK;
        sum_t += ct[i]; sum_s += cs[i];
        mt = ct[i] > mt ? ct[i] : mt; ms = cs[i] > ms ? cs[i] : ms;
    }
    uint32_t et = block_excl_scan(sum_t, scan_tmp, &all_t), es = block_excl_scan(sum_s, scan_tmp, &all_s);
#pragma unroll
    for (uint32_t i = 0; i < OWN; ++i) {
        if (i < own && first + i < gridDim.x) write_offsets(S, gridDim.x, first + i, et, es);
        et += ct[i]; es += cs[i];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t a = __shfl_xor(mt, off, 64), b = __shfl_xor(ms, off, 64);
        mt = a > mt ? a : mt; ms = b > ms ? b : ms;
        flags |= __shfl_xor(flags, off, 64);
    }
    if ((tid & 63u) == 0) { scan_tmp[tid >> 6] = mt; scan_tmp[4 + (tid >> 6)] = ms; scan_tmp[8 + (tid >> 6)] = flags; }
    __syncthreads();
    if (tid == 0) {
        for (uint32_t w = 1; w < ENUM_THREADS / 64; ++w) {
            mt = scan_tmp[w] > mt ? scan_tmp[w] : mt;
            ms = scan_tmp[4 + w] > ms ? scan_tmp[4 + w] : ms;
            flags |= scan_tmp[8 + w];
        }
        write_totals(S, gridDim.x, all_t, all_s, mt, ms, flags);
    }
    return;
    }
}

// The table from the parked words, a wavefront per job.  Launched before the host has seen the totals: nothing is
// written unless the counting pass raised no flag and the table takes everything (the same in all threads).
constexpr int FILL_THREADS = 256;
constexpr uint32_t FILL_AHEAD = 4;         // loads of a lane in flight: jobs mostly have fewer than 256 triples (with two 32 us where this takes 31)

__global__ __launch_bounds__(FILL_THREADS) void k_fill(uint32_t n_jobs, const uint32_t *__restrict__ leader,
                                                       const uint32_t *__restrict__ park, uint32_t park_stride,
                                                       const uint32_t *__restrict__ triple_off, const uint32_t *__restrict__ seg_off,
                                                       uint32_t *__restrict__ triples, uint32_t *__restrict__ seg_g,
                                                       uint32_t *__restrict__ seg_first, const uint32_t *__restrict__ totals,
                                                       uint64_t cap_triples, uint64_t cap_segs) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t j = blockIdx.x * (FILL_THREADS / 64) + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint64_t nt = ((uint64_t)totals[TOT_NT_HI] << 32) | totals[TOT_NT_LO];
    const uint64_t ns = ((uint64_t)totals[TOT_NS_HI] << 32) | totals[TOT_NS_LO];
    if (j >= n_jobs || totals[TOT_ERR] != 0u || nt > 0xFFFFFFFFull || nt > cap_triples || ns > cap_segs) return;
    const uint32_t t0 = triple_off[j], t_n = triple_off[j + 1] - t0, s0 = seg_off[j];
    const uint32_t *from = park + (size_t)(leader ? leader[j] : j) * park_stride;   // parked by the job that searched
    uint32_t *const to_t = triples + t0, *const to_g = seg_g + s0, *const to_f = seg_first + s0;
    uint32_t seg = 0, last = 0;                            // segments so far, GPUs of the word before (no word has 0)
    for (uint32_t base = 0; base < t_n; base += 64 * FILL_AHEAD) {
        uint32_t w[FILL_AHEAD];
#pragma unroll
        for (uint32_t u = 0; u < FILL_AHEAD; ++u) {
            const uint32_t i = base + 64 * u + lane;
            w[u] = i < t_n ? from[i] : 0u;
        }
#pragma unroll
        for (uint32_t u = 0; u < FILL_AHEAD; ++u) {
            if (base + 64 * u >= t_n) break;
            const uint32_t i = base + 64 * u + lane, g = word_gpus(w[u]);
            const uint32_t before = (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)g, 0x138, 0xF, 0xF, false);   // wave_shr:1
            const bool in = i < t_n, starts = in && g != before;
            const unsigned long long m = __ballot(starts);
            if (in) to_t[i] = w[u];
            if (starts) {
                const uint32_t s = seg + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                to_g[s] = g;
                to_f[s] = i;
            }
            seg += (uint32_t)__popcll(m);
            last = (uint32_t)__builtin_amdgcn_readlane((int)g, 63);
        }
    }
}

// exclusive scan of the per-job counts, totals and maxima: one workgroup walks
// the jobs in tiles of 8192, every thread taking eight neighbouring jobs with
// two 16-byte loads per array (the next tile is requested before the current
// one is scanned); a thread sums its eight, the sums are scanned inside the
// wavefronts by shuffles and across them through LDS, and the offsets leave
// through LDS so that the stores are coalesced too.
constexpr uint32_t SCAN_PER = 8, SCAN_TILE = 1024 * SCAN_PER;

struct Eight { uint32_t v[SCAN_PER]; };

// counts of jobs j0 .. j0+7 (0 beyond the end); cnt + j0 is 32-byte aligned
__device__ __forceinline__ Eight load_eight(const uint32_t *__restrict__ cnt, uint32_t j0, uint32_t n_jobs) {
    Eight e;
    if (j0 + SCAN_PER <= n_jobs) {
        const uint4 a = *reinterpret_cast<const uint4 *>(cnt + j0), b = *reinterpret_cast<const uint4 *>(cnt + j0 + 4);
        e.v[0] = a.x; e.v[1] = a.y; e.v[2] = a.z; e.v[3] = a.w;
        e.v[4] = b.x; e.v[5] = b.y; e.v[6] = b.z; e.v[7] = b.w;
    } else {
#pragma unroll
        for (uint32_t i = 0; i < SCAN_PER; ++i) e.v[i] = j0 + i < n_jobs ? cnt[j0 + i] : 0u;
    }
    return e;
}

__global__ __launch_bounds__(1024) void k_scan_counts(const uint32_t *__restrict__ cnt_t,
                                                      const uint32_t *__restrict__ cnt_s, uint32_t n_jobs, ScanOut S) {
    __shared__ __align__(16) uint32_t buf_t[SCAN_TILE], buf_s[SCAN_TILE];
    __shared__ unsigned long long wave_t[16], wave_s[16];
    __shared__ uint32_t wave_mt[16], wave_ms[16], wave_e[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    unsigned long long carry_t = 0, carry_s = 0;            // everything before the tile (same in every thread)
    uint32_t mt = 0, ms = 0, err = 0;                       // running maxima and flags of this thread's elements
    Eight nt_next = load_eight(cnt_t, tid * SCAN_PER, n_jobs), ns_next = load_eight(cnt_s, tid * SCAN_PER, n_jobs);
    for (uint32_t base = 0; base < n_jobs; base += SCAN_TILE) {
        Eight ct = nt_next;
        const Eight cs = ns_next;
        if (base + SCAN_TILE < n_jobs) {
            nt_next = load_eight(cnt_t, base + SCAN_TILE + tid * SCAN_PER, n_jobs);
            ns_next = load_eight(cnt_s, base + SCAN_TILE + tid * SCAN_PER, n_jobs);
        }
        unsigned long long sum_t = 0, sum_s = 0;
#pragma unroll
        for (uint32_t i = 0; i < SCAN_PER; ++i) {
            err |= ct.v[i] >> CNT_FLAGS;
            ct.v[i] &= CNT_MASK;
            sum_t += ct.v[i]; sum_s += cs.v[i];
            mt = ct.v[i] > mt ? ct.v[i] : mt;
            ms = cs.v[i] > ms ? cs.v[i] : ms;
        }
        unsigned long long it = sum_t, is = sum_s;          // inclusive scan of the threads' sums inside the wavefront
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const unsigned long long at = __shfl_up(it, off, 64), as = __shfl_up(is, off, 64);
            if ((int)lane >= off) { it += at; is += as; }
        }
        if (lane == 63u) { wave_t[wave] = it; wave_s[wave] = is; }
        __syncthreads();
        unsigned long long before_t = 0, before_s = 0, all_t = 0, all_s = 0;
#pragma unroll
        for (uint32_t w = 0; w < 16; ++w) {
            if (w < wave) { before_t += wave_t[w]; before_s += wave_s[w]; }
            all_t += wave_t[w]; all_s += wave_s[w];
        }
        uint32_t run_t = (uint32_t)(carry_t + before_t + it - sum_t), run_s = (uint32_t)(carry_s + before_s + is - sum_s);
        uint32_t ot[SCAN_PER], os[SCAN_PER];
#pragma unroll
        for (uint32_t i = 0; i < SCAN_PER; ++i) {
            ot[i] = run_t; os[i] = run_s;
            run_t += ct.v[i]; run_s += cs.v[i];
        }
        uint4 *dt = reinterpret_cast<uint4 *>(buf_t + tid * SCAN_PER), *ds = reinterpret_cast<uint4 *>(buf_s + tid * SCAN_PER);
        dt[0] = make_uint4(ot[0], ot[1], ot[2], ot[3]); dt[1] = make_uint4(ot[4], ot[5], ot[6], ot[7]);
        ds[0] = make_uint4(os[0], os[1], os[2], os[3]); ds[1] = make_uint4(os[4], os[5], os[6], os[7]);
        __syncthreads();
#pragma unroll
        for (uint32_t i = 0; i < SCAN_PER; ++i) {
            const uint32_t at = i * 1024 + tid, j = base + at;
            if (j < n_jobs) {
                write_offsets(S, n_jobs, j, buf_t[at], buf_s[at]);
            }
        }
        carry_t += all_t; carry_s += all_s;
        __syncthreads();                                    // LDS is read before the next tile overwrites it
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t a = __shfl_xor(mt, off, 64), b = __shfl_xor(ms, off, 64);
        mt = a > mt ? a : mt; ms = b > ms ? b : ms;
        err |= __shfl_xor(err, off, 64);
    }
    if (lane == 0) { wave_mt[wave] = mt; wave_ms[wave] = ms; wave_e[wave] = err; }
    __syncthreads();
    if (tid == 0) {
        for (uint32_t w = 0; w < 16; ++w) {
            mt = wave_mt[w] > mt ? wave_mt[w] : mt; ms = wave_ms[w] > ms ? wave_ms[w] : ms;
            err |= wave_e[w];
        }
        write_totals(S, n_jobs, carry_t, carry_s, mt, ms, err);
    }
}

__global__ void k_zero_words(uint32_t *p, uint32_t n) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

}  // namespace

static int32_t launch_fill(rk_ctx *ctx, const rk_plan_table *table, const EnumPending &P) {
    constexpr uint32_t PER = FILL_THREADS / 64;
    const uint32_t J = table->n_jobs;
    k_fill<<<(J + PER - 1) / PER, FILL_THREADS, 0, ctx->stream>>>(J, P.leader, P.park, P.park_stride, P.off_t, P.off_s, table->triples,
                                                                 table->seg_g, table->seg_first, P.totals, table->cap_triples, table->cap_segs);
    RK_CHECK_LAUNCH(ctx, "k_fill");
    return RK_OK;
}

int32_t rk_enumerate_begin(rk_ctx *ctx, const rk_jobs *jobs, const rk_plan_bounds *bounds, rk_plan_table *table, EnumPending &P, bool leave_content) {
    if (!jobs || !bounds || !table) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null argument");
    if (jobs->n_jobs > 0 && (!jobs->layers || !jobs->gbatch || !jobs->mbatch)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "job arrays are null");
    if (bounds->g_max < 1 || bounds->g_max > RK_MAX_G) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "g_max must be in 1..%u", RK_MAX_G);
    if (bounds->pp_max < 1 || bounds->pp_max > RK_MAX_PP) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "pp_max must be in 1..%u", RK_MAX_PP);
    if (bounds->tp_max < 1) return rk_fail(ctx, RK_ERR_INVALID_ARG, "tp_max below 1");
    if (bounds->zero_mask > 0xF || bounds->gc_mask > 3 || bounds->off_mask > 3 || bounds->mu_mask > 0xF)
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "option mask has unknown bits");
    if (bounds->mu_mask == 0) return rk_fail(ctx, RK_ERR_INVALID_ARG, "mu_mask allows no micro-batch size");
    RK_HIP(ctx, hipSetDevice(ctx->device));

    const uint32_t J = jobs->n_jobs;
    uint32_t opt = 0;
    for (uint32_t o = 0; o < 16; ++o) {
        const uint32_t z = o >> 2, gc = (o >> 1) & 1u, off = o & 1u;
        if (((bounds->zero_mask >> z) & 1u) && ((bounds->gc_mask >> gc) & 1u) && ((bounds->off_mask >> off) & 1u))
            opt |= 1u << o;
    }
    table->option_mask = opt;
    table->n_jobs = J;
    table->n_triples = table->n_segs = 0;
    table->max_triples_per_job = table->max_segs_per_job = 0;

    uint32_t *cnt_t, *cnt_s, *totals, *off_t, *off_s, *park;
    int32_t rc;
    if ((rc = rk_scratch(ctx, SL_CNT_T, (size_t)(2 * (size_t)J + 2) * 4, (void **)&cnt_t))) return rc;
    if ((rc = rk_scratch(ctx, SL_CNT_S, (size_t)(2 * (size_t)J + 2) * 4, (void **)&cnt_s))) return rc;
    // (a call with few jobs searches for each of them: two more launches would cost more than they save)
    const bool share = J >= SHARE_MIN_JOBS;
    uint64_t tab_slots = 64;                                  // leaders' hash table: a power of two, at least twice the jobs
    while (tab_slots < 2 * (uint64_t)J) tab_slots <<= 1;
    const uint32_t job_blocks = (J + LEAD_THREADS - 1) / LEAD_THREADS;
    const bool tiles = share && job_blocks <= SCAN_MOST_TILES;
    uint32_t *tab = nullptr, *leader = nullptr, *list = nullptr;
    TileSum *sums = nullptr;
    // The counter in the totals is zero where the last call came to its end (set below); otherwise it is cleared first.
    if ((rc = rk_scratch(ctx, SL_TOTALS, 16 * sizeof(uint32_t), (void **)&totals))) return rc;
    if (!ctx->enum_clear) {
        k_zero_words<<<1, 64, 0, ctx->stream>>>(totals, 16u);
        RK_CHECK_LAUNCH(ctx, "k_zero_words");
    }
    ctx->enum_clear = false;
    if (share) {
        const size_t had = ctx->scratch_bytes[SL_ENUM_TAB];
        if ((rc = rk_scratch(ctx, SL_ENUM_TAB, (size_t)tab_slots * 4, (void **)&tab))) return rc;
        if ((rc = rk_scratch(ctx, SL_ENUM_LEADER, ((J > ENUM_TURNS ? 2 : 1) * (size_t)J + 1) * 4, (void **)&leader))) return rc;
        if (J > ENUM_TURNS) list = leader + J;
        if ((rc = rk_scratch(ctx, SL_ENUM_SUMS, (size_t)job_blocks * sizeof(TileSum), (void **)&sums))) return rc;
        if (ctx->scratch_bytes[SL_ENUM_TAB] != had) ctx->enum_tab_clear = 0;         // new memory
    }
    // one slot per job for the parked words: as wide as the widest job seen so far, or a first guess
    if (ctx->park_stride == 0) ctx->park_stride = 512;
    const uint32_t park_stride = ctx->park_stride;
    if ((rc = rk_scratch(ctx, SL_PARK, ((size_t)J * park_stride + 1) * 4, (void **)&park))) return rc;
    const bool fill = table->triples != nullptr;              // otherwise a sizing call
    if (fill && (!table->triple_off || !table->seg_off || !table->seg_g || !table->seg_first))
        return rk_fail(ctx, RK_ERR_INVALID_ARG, "table buffer is null");
    off_t = fill ? table->triple_off : cnt_t + J;             // offsets go straight into the table
    off_s = fill ? table->seg_off : cnt_s + J;
    // what comes back in one piece: totals, then the two offset arrays (pinned host memory that the scan writes)
    const size_t words_back = 16 + 2 * ((size_t)J + 1);
    if (ctx->h_stage_words < words_back) {
        if (ctx->h_stage) RK_HIP(ctx, hipHostFree(ctx->h_stage));
        ctx->h_stage = nullptr; ctx->h_stage_words = 0;
        RK_HIP(ctx, hipHostMalloc((void **)&ctx->h_stage, (words_back + words_back / 4) * 4, hipHostMallocDefault));
        ctx->h_stage_words = words_back + words_back / 4;
    }
    uint32_t *h = ctx->h_stage;
    if (!ctx->counts_ev) RK_HIP(ctx, hipEventCreateWithFlags(&ctx->counts_ev, hipEventDisableTiming));

    const bool mirrors = fill && table->h_triple_off && table->h_seg_off;
    // All of them go straight to the host, a wavefront's words in one piece.  As a copy that the host sends for, behind the scan,
    // they cost an enumeration of 3,333 jobs 44 instead of 30 us, of 10,000 jobs 48 and 33, of 128,000 jobs 93 and 78.
    uint32_t *back;
    RK_HIP(ctx, hipHostGetDevicePointer((void **)&back, h, 0));
    const ScanOut S = {off_t, off_s, totals, back, mirrors ? 1u : 0u};

    const size_t gmap_bytes = (size_t)((bounds->g_max >> 5) + 1u) * 2 * sizeof(uint32_t);   // bitmap + word prefixes
    const bool self_scan = J > 0 && J <= ENUM_SELF_SCAN && !share;
    size_t tab_clear = 0;
    if (share) {
        // the table is zero where earlier calls came to their end; otherwise it is cleared first
        const size_t clear = ctx->enum_tab_clear;
        ctx->enum_tab_clear = 0;
        if (clear < tab_slots) {
            k_zero_words<<<(uint32_t)((tab_slots + 255) / 256), 256, 0, ctx->stream>>>(tab, (uint32_t)tab_slots);
            RK_CHECK_LAUNCH(ctx, "k_zero_words");
        }
        tab_clear = clear < tab_slots ? (size_t)tab_slots : clear;
        k_enum_leaders<<<job_blocks, LEAD_THREADS, 0, ctx->stream>>>(jobs->layers, jobs->gbatch, jobs->mbatch, J, tab,
                                                                    (uint32_t)(tab_slots - 1), leader, list, totals + TOT_LEADERS);
        RK_CHECK_LAUNCH(ctx, "k_enum_leaders");
    }
    if (J > 0) {
        const auto count = list ? k_enumerate<MODE_COUNT, true> : k_enumerate<MODE_COUNT, false>;
        count<<<list ? ENUM_TURNS : J, ENUM_THREADS, gmap_bytes, ctx->stream>>>(
            jobs->layers, jobs->gbatch, jobs->mbatch, *bounds, leader, list, totals + TOT_LEADERS, cnt_t, cnt_s, park, park_stride,
            nullptr, nullptr, nullptr, nullptr, nullptr, self_scan ? 1u : 0u, S);
        RK_CHECK_LAUNCH(ctx, "k_enumerate<count>");
    }
    if (share) {
        k_spread_counts<<<job_blocks, LEAD_THREADS, 0, ctx->stream>>>(leader, J, cnt_t, cnt_s, sums, tab, (uint32_t)tab_slots, totals + TOT_LEADERS);
        RK_CHECK_LAUNCH(ctx, "k_spread_counts");
    }
    if (tiles) k_scan_tiles<<<job_blocks, LEAD_THREADS, 0, ctx->stream>>>(cnt_t, cnt_s, J, sums, S);
    else if (!self_scan) k_scan_counts<<<1, 1024, 0, ctx->stream>>>(cnt_t, cnt_s, J, S);
    RK_CHECK_LAUNCH(ctx, "k_scan_counts");
    RK_HIP(ctx, hipEventRecord(ctx->counts_ev, ctx->stream));
    // The fill pass (or what the caller launches instead) goes out before the host knows the totals, so that the device does not
    // wait for the round trip: the kernel itself checks the flags and the table's capacity.
    P = EnumPending{jobs, *bounds, leader, cnt_t, cnt_s, park, off_t, off_s, totals, park_stride, gmap_bytes, tab_clear, fill, mirrors, share, false,
                    false, false, TableGuard{}};
    return fill && J > 0 && !leave_content ? launch_fill(ctx, table, P) : RK_OK;
}

int32_t rk_enumerate_end(rk_ctx *ctx, rk_plan_table *table, EnumPending &P) {
    const uint32_t J = table->n_jobs;
    const uint32_t *const h = ctx->h_stage;
    RK_HIP(ctx, hipEventSynchronize(ctx->counts_ev));
    ctx->enum_clear = true;                                   // the kernels before the event have run
    if (P.share) ctx->enum_tab_clear = P.tab_clear;

    if (h[TOT_ERR] & ERR_TOO_MANY_TRIPLES) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "a job has more than %u triples", MAX_T);
    if (h[TOT_ERR] & ERR_TOO_MANY_DIVISORS) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "a job has more than %u candidate d or p sizes", MAX_DIV);
    const uint64_t nt = ((uint64_t)h[TOT_NT_HI] << 32) | h[TOT_NT_LO];
    const uint64_t ns = ((uint64_t)h[TOT_NS_HI] << 32) | h[TOT_NS_LO];
    if (nt > 0xFFFFFFFFull) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 2^32-1 triples");
    table->n_triples = nt;
    table->n_segs = ns;
    table->max_triples_per_job = h[TOT_MAX_T];
    table->max_segs_per_job = h[TOT_MAX_S];
    ctx->seen_t[1] = ctx->seen_t[0]; ctx->seen_s[1] = ctx->seen_s[0];
    ctx->seen_t[0] = h[TOT_MAX_T]; ctx->seen_s[0] = h[TOT_MAX_S];
    ctx->seen_segs = ns; ctx->seen_jobs = J;
    const bool parked = !(h[TOT_ERR] & ERR_PARK_FULL);
    if (!parked) {                                            // next time the slots will be wide enough
        uint32_t want = h[TOT_MAX_T] + h[TOT_MAX_T] / 4;
        want = (want + 63u) & ~63u;
        ctx->park_stride = want > MAX_T ? MAX_T : want;
    }

    P.whole = h[TOT_ERR] == 0u;
    const TableGuard &G = P.guard;                            // (what table_usable asks)
    P.taken = P.ahead && P.whole && nt <= G.cap_triples && ns <= G.cap_segs && h[TOT_MAX_T] <= G.most_t && h[TOT_MAX_S] <= G.most_s;
    if (!P.fill) return RK_OK;
    if (table->cap_triples < nt || table->cap_segs < ns)
        return rk_fail(ctx, RK_ERR_CAPACITY, "table too small: need %llu triples and %llu segments",
                       (unsigned long long)nt, (unsigned long long)ns);
    if (P.mirrors) {
        memcpy(table->h_triple_off, h + 16, ((size_t)J + 1) * 4);
        memcpy(table->h_seg_off, h + 16 + J + 1, ((size_t)J + 1) * 4);
    }
    int32_t rc;
    if (J > 0 && P.ahead && !P.taken && parked && (rc = launch_fill(ctx, table, P))) return rc;
    if (J > 0 && !parked) {                                   // the parked keys were incomplete: search again
        const rk_jobs *const jobs = P.jobs;
        k_enumerate<MODE_FILL_SEARCH, false><<<J, ENUM_THREADS, P.gmap_bytes, ctx->stream>>>(
            jobs->layers, jobs->gbatch, jobs->mbatch, P.bounds, nullptr, nullptr, nullptr, P.cnt_t, P.cnt_s, P.park, P.park_stride,
            P.off_t, P.off_s, table->triples, table->seg_g, table->seg_first, 0u, ScanOut{});
        RK_CHECK_LAUNCH(ctx, "k_enumerate<fill>");
    }
    return RK_OK;
}

extern "C" int32_t rk_enumerate_plans(rk_ctx *ctx, const rk_jobs *jobs, const rk_plan_bounds *bounds,
                                      rk_plan_table *table) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    EnumPending P;
    const int32_t rc = rk_enumerate_begin(ctx, jobs, bounds, table, P);
    return rc ? rc : rk_enumerate_end(ctx, table, P);
}
