// Fused path: evaluation (paper Sec. 4), best plan per segment (GetBestPlan,
// Sec. 5.2) and curves (Sec. 5.2, Fig. 6) in one kernel, one workgroup per
// job, without writing the candidates to memory.
//
// It exploits the structure of the model: plans without offload do not depend
// on the CPUs or the memory tier, so their per-segment maximum is taken once;
// offload plans depend on the CPUs only through the swap term and on the tier
// only through feasibility (a plan that fits a tier fits every larger one, so
// its key goes to the first tier and the tiers take a running maximum).  All
// values come from the functions of rk_model.h, so the results are
// bit-identical to the materialising path.
//
// Bound by the vector ALUs' issue slots.  Phase 1 has a lane per triple and
// packs the triples with a usable offload plan, so that the lanes of phase 2
// (a lane per packed triple and up to six CPU levels) are all busy; quotients
// by the same divisor share its reciprocal.  Many jobs take a wavefront each
// (DIRECT), whose lanes go from phase 1 straight to the CPU levels.  In a round
// the kernel also makes the plan table's content from what the enumeration's
// searches left: under the arithmetic that costs nothing that can be measured,
// as a launch of its own 3 us for few jobs and 30 for 128,000.  The
// 128,000 jobs of 256 rounds took 808 us in the first form (a lane per triple
// and level, a key per tier), 10,000 jobs on the full grid of 20 rows 117 us;
// now 402 and 69 us.
#include "rk_internal.h"
#include "rk_model.h"

namespace {

// Every wavefront of a job loads it and works out the same indexes, so where the jobs fill the chip several times one
// wavefront per job (DIRECT) costs the least: 402 us for 128,000 jobs with five rows against 672 with four wavefronts, 69
// against 85 us for 10,000 jobs with twenty, 55 against 62 for 7,000, 41.6 against 43.4 for 4,500.  Below that it is the
// single job that counts, and four wavefronts finish it sooner: 29.7 us against 32.1 for 3,000 jobs, 13 against 20 for 1,000.
// The line is that of five and twenty rows.  With one row and eight it could lie lower (2,500 jobs 22 against 26 and 26
// against 28 us), with more rows higher: 32 rows of 97 triples 51 against 49 us for 4,096 jobs and 82 against 86 for 10,000;
// 64 rows 105 against 90 for 6,000, 136 against 127 for 10,000, 383 against 432 for 40,000.  One job's lanes wait longest
// for each other where the rows are many and have tiers: 64 levels of three tiers, 302 against 204 us for 10,000 jobs and
// 1,033 against 709 for 40,000, where four wavefronts would be the better form at every count.
constexpr int FEW_JOBS = 256;
constexpr uint32_t FUSED_MANY = 4096;
constexpr uint32_t FUSED_FILL = 512;      // workgroups that occupy the chip: two per CU

struct FusedLds {          // element counts of the dynamic LDS regions
    uint32_t max_nt, max_ns, rows_per_pass;
};

__host__ __device__ inline size_t fused_lds_bytes(const FusedLds &L, bool direct) {
    return 8 + (size_t)L.max_ns * 8 + (size_t)L.rows_per_pass * L.max_ns * 8 + (size_t)L.max_nt * (direct ? 2 : 4 * 5 + 2) + (size_t)L.max_ns * 4;
}

// info word of a packed triple: usable offload options, first memory tier that holds them, segment
static_assert(RK_MAX_MEM_LEVELS <= 16, "fields of the info word");
__device__ __forceinline__ uint32_t info_word(uint32_t ok, uint32_t tier, uint32_t seg) { return ok | (tier << 4) | (seg << 8); }

// one step of an inclusive maximum scan along the wavefront: v = max(v, the value CTRL brings) where `take`
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long scan_max_step(unsigned long long v, bool take) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xF, false);
    const unsigned long long o = ((unsigned long long)hi << 32) | lo;
    return take && o > v ? o : v;
}

// blockIdx.y: which c_per_block CPU levels
// DIRECT: one wavefront, all rows in one pass; a lane goes from its triple straight to the CPU levels, nothing of a
// triple is kept in LDS and no barrier is needed.
template <int THREADS, bool DIRECT>
__global__ __launch_bounds__(THREADS) void k_fused(JobDev jobs, TableDev tb, GridDev grid, rk_env env,
                                                         uint32_t jb, uint32_t option_mask, FusedLds L,
                                                         uint32_t c_per_block, uint32_t c_per_pass, uint32_t m_per_pass,
                                                         float *__restrict__ best_thr, uint32_t *__restrict__ best_plan,
                                                         float *__restrict__ curve_thr, uint32_t *__restrict__ curve_plan,
                                                         uint32_t *__restrict__ curve_g,
                                                    TableGuard guard, ParkedWords parked) {
    if (!table_usable(guard)) return;
    extern __shared__ unsigned long long lds64[];
    uint32_t &n_packed = *reinterpret_cast<uint32_t *>(lds64);               // triples packed so far
    unsigned long long *seg_plain = lds64 + 1;                               // [max_ns]
    unsigned long long *seg_best = seg_plain + L.max_ns;                     // [rows_per_pass][max_ns]
    // packed triples with a usable offload plan (before they are packed: t_info[tl] = segment of triple tl)
    float *t_base0 = reinterpret_cast<float *>(seg_best + (size_t)L.rows_per_pass * L.max_ns);
    float *t_base1 = t_base0 + L.max_nt;
    float *t_topt = t_base1 + L.max_nt;
    float *t_toff = t_topt + L.max_nt;
    uint32_t *t_info = reinterpret_cast<uint32_t *>(t_toff + L.max_nt);
    uint32_t *l_segg = DIRECT ? reinterpret_cast<uint32_t *>(t_base0) : t_info + L.max_nt;   // [max_ns] GPUs of the job's segments
    uint16_t *t_16 = reinterpret_cast<uint16_t *>(l_segg + L.max_ns);        // [max_nt] number of a packed triple; DIRECT: segment of a triple

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t j = jb + blockIdx.x;
    const uint32_t c_begin = blockIdx.y * c_per_block;
    const uint32_t c_end = c_begin + c_per_block < grid.n_cpu ? c_begin + c_per_block : grid.n_cpu;
    const uint32_t t0 = tb.triple_off[j], nt = tb.triple_off[j + 1] - t0;
    const uint32_t s0 = tb.seg_off[j], ns = tb.seg_off[j + 1] - s0;
    const uint32_t n_mem = grid.n_mem, n_rows = grid.n_cpu * n_mem;
    const uint64_t sbase = (uint64_t)n_rows * (s0 - tb.seg_off[jb]);
    const Job J = load_job(jobs, j);

    // per segment: nothing found yet, its GPU count, and its number in the info word of each of its triples
    if (tid == 0) n_packed = 0u;
    const uint32_t *words = tb.triples + t0;
    if (parked.words) {
        // The table's content is made here, from the words that the search left (k_fill): a segment begins where the GPUs
        // change.  Every wavefront counts through all words, 64 at a time, and takes every THREADS / 64-th time its share.
        words = parked.words + (size_t)(parked.leader ? parked.leader[j] : j) * parked.stride;
        const bool write = blockIdx.y == 0;
        uint32_t seg = 0, before = 0;                        // segments so far, GPUs of the last word (no word has 0)
        for (uint32_t base = 0; base < nt; base += 64u) {
            const uint32_t t = base + lane, w = t < nt ? words[t] : 0u, g = word_gpus(w);
            const uint32_t g_before = (uint32_t)__builtin_amdgcn_update_dpp((int)before, (int)g, 0x138, 0xF, 0xF, false);      // wave_shr:1
            const bool starts = t < nt && g != g_before;
            const unsigned long long m = __ballot(starts);
            if (THREADS == 64 || (base / 64u) % (THREADS / 64u) == tid / 64u) {
                const uint32_t s = seg + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                if (starts) {
                    seg_plain[s] = 0ull;
                    l_segg[s] = g;
                    if (write) parked.seg_g[s0 + s] = g;
                    if (write && parked.seg_first) parked.seg_first[s0 + s] = t;
                }
                if (t < nt) {
                    const uint32_t own = starts ? s : s - 1u;
                    if (DIRECT) t_16[t] = (uint16_t)own; else t_info[t] = own;
                    if (write && parked.triples) parked.triples[t0 + t] = w;
                }
            }
            seg += (uint32_t)__popcll(m);
            before = (uint32_t)__builtin_amdgcn_readlane((int)g, 63);
        }
    } else
    for (uint32_t s = tid; s < ns; s += THREADS) {
        seg_plain[s] = 0ull;
        l_segg[s] = tb.seg_g[s0 + s];
        const uint32_t first = tb.seg_first[s0 + s];
        const uint32_t last = s + 1 < ns ? tb.seg_first[s0 + s + 1] : nt;
        for (uint32_t t = first; t < last; ++t) {
            if (DIRECT) t_16[t] = (uint16_t)s; else t_info[t] = s;
        }
    }
    const float fb = (float)J.gbatch, inv_kswap = __builtin_amdgcn_rcpf(J.k_swap);
    // The key of an offload plan at `levels` neighbouring CPU levels from ci on, in the rows from `slot` on.  Options in
    // plan order: (z2,gc0) (z2,gc1) (z3,gc0) (z3,gc1); the stage does not change the value.
    auto over_levels = [&](const Offload &O, uint32_t ok, uint32_t plan, uint32_t g, uint32_t ci, uint32_t c_stop,
                           unsigned long long *slot, size_t stride) {
        Triple Tb; Tb.b = fb;
        const uint32_t plan0 = plan + (ok & 1u ? 9u : 13u), plan1 = plan + (ok & 2u ? 11u : 15u);
        for (; ci < c_stop; ++ci, slot += stride) {
            const float sw = swap_term(J, O, cpus_of(grid, ci, g));
            const unsigned long long k0 = ok & 5u ? make_key(thr_offload(Tb, O, 0, sw), plan0) : 0ull;
            const unsigned long long k1 = ok & 10u ? make_key(thr_offload(Tb, O, 1, sw), plan1) : 0ull;
            atomicMax(slot, k0 > k1 ? k0 : k1);
        }
    };
    if (DIRECT)
        for (uint32_t i = tid; i < (c_end - c_begin) * n_mem * L.max_ns; i += THREADS) seg_best[i] = 0ull;
    __syncthreads();

    // phase 1: one lane per triple; a workgroup's turn packs behind the turn before, so what it overwrites of the
    // segment numbers has been read
    for (uint32_t base = 0; base < nt; base += THREADS) {
        const uint32_t tl = base + tid;
        uint32_t ok = 0, info = 0;
        Offload O = {};
        if (tl < nt) {
            const Triple T = triple_terms(J, env, words[tl]);
            const uint32_t seg = DIRECT ? t_16[tl] : t_info[tl];
            // without offload: a stage above 0 does not change the throughput, so of those the lowest that fits
            unsigned long long k = 0;
#pragma unroll
            for (uint32_t gc = 0; gc < 2; ++gc) {
                bool fits[4];
#pragma unroll
                for (uint32_t z = 0; z < 4; ++z) fits[z] = ((option_mask >> (z * 4 + gc * 2)) & 1u) && gpu_mem_fits(J, env, T, z, gc, 0);
                if (fits[0]) {
                    const unsigned long long c = make_key(thr_plain(J, T, 0, gc), tl * 16 + gc * 2);
                    k = c > k ? c : k;
                }
                if (fits[1] || fits[2] || fits[3]) {
                    const uint32_t z = fits[1] ? 1u : fits[2] ? 2u : 3u;
                    const unsigned long long c = make_key(thr_plain(J, T, 1, gc), tl * 16 + z * 4 + gc * 2);
                    k = c > k ? c : k;
                }
            }
            if (k >> 32) atomicMax(&seg_plain[seg], k);
#pragma unroll
            for (uint32_t z = 2; z < 4; ++z)
#pragma unroll
                for (uint32_t gc = 0; gc < 2; ++gc) {
                    const uint32_t o = z * 4 + gc * 2 + 1;
                    if (((option_mask >> o) & 1u) && gpu_mem_fits(J, env, T, z, gc, 1)) ok |= 1u << ((z - 2) * 2 + gc);
                }
            if (ok) {
                const float need = host_bytes_needed(J, T);
                uint32_t tier = 0;                                // (tiers ascend)
                while (tier < n_mem && !(need <= tier_bytes(grid, tier, T.g))) ++tier;
                if (tier == n_mem) ok = 0;
                else {
                    O = offload_terms(J, env, T);
                    if (!DIRECT) info = info_word(ok, tier, seg);
                    else over_levels(O, ok, tl * 16u, T.g, c_begin, c_end, seg_best + (size_t)tier * L.max_ns + seg, (size_t)n_mem * L.max_ns);
                }
            }
        }
        if (DIRECT) continue;
        // the turn's triples are read before any of them is overwritten by a packed one (all turns of more than one
        // workgroup's width; the last barrier also closes the phase)
        const unsigned long long with = __ballot(ok != 0);
        uint32_t at = 0;
        if (lane == 0 && with) at = atomicAdd(&n_packed, (uint32_t)__popcll(with));
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(with & ((1ull << lane) - 1ull));
        __syncthreads();
        if (ok) {
            t_base0[at] = O.base[0]; t_base1[at] = O.base[1];
            t_topt[at] = O.topt_num; t_toff[at] = O.Toff;
            t_info[at] = info; t_16[at] = (uint16_t)tl;
            // T.b and 1/k_swap are the same for every triple of the job
        }
    }
    __syncthreads();
    const uint32_t np = n_packed;

    // A pass keeps the keys of some rows in LDS: several CPU levels with all their tiers, or, when the rows of one
    // level do not fit, some tiers of one level (m_per_pass < n_mem only together with c_per_pass == 1).  Either
    // way the rows of a pass are neighbours in the output, starting at row c_lo * n_mem + m_lo.
    const float inv_np = __builtin_amdgcn_rcpf((float)np), inv_ns = __builtin_amdgcn_rcpf((float)ns);
    const uint32_t q = small_quot(lane, inv_ns), s_lane = lane - q * ns;       // phase 3: the lane's row in a group and its segment
    const uint32_t r_group = ns <= 64u && ns > 0 ? small_quot(64u, inv_ns) : 1u;   // rows that 64 lanes hold whole
    for (uint32_t c_lo = c_begin; c_lo < c_end; c_lo += c_per_pass)
    for (uint32_t m_lo = 0; m_lo < n_mem; m_lo += m_per_pass) {
        const uint32_t c_hi = c_lo + c_per_pass < c_end ? c_lo + c_per_pass : c_end;
        const uint32_t m_hi = m_lo + m_per_pass < n_mem ? m_lo + m_per_pass : n_mem;
        const uint32_t m_cnt = m_hi - m_lo;
        const uint32_t pass_rows = (c_hi - c_lo) * m_cnt;
        const uint32_t row0 = c_lo * n_mem + m_lo;
        if (!DIRECT) {
            for (uint32_t i = tid; i < pass_rows * L.max_ns; i += THREADS) seg_best[i] = 0ull;
            __syncthreads();

            // phase 2: one item per packed triple and up to six neighbouring CPU levels, which share what is read and unpacked
            const uint32_t levels = c_hi - c_lo, parts = (levels + 5u) / 6u;
            const uint32_t per_part = parts > 1 ? small_quot(levels + parts - 1u, __builtin_amdgcn_rcpf((float)parts)) : levels;
            for (uint32_t i = tid; i < np * parts; i += THREADS) {
                const uint32_t part = parts > 1 ? small_quot(i, inv_np) : 0u, at = i - part * np;
                const uint32_t info = t_info[at], ok = info & 15u, tier = (info >> 4) & 15u, seg = info >> 8;
                const uint32_t plan = (uint32_t)t_16[at] * 16u;
                if (tier >= m_hi) continue;
                Offload O;
                O.base[0] = t_base0[at]; O.base[1] = t_base1[at];
                O.topt_num = t_topt[at]; O.Toff = t_toff[at]; O.inv_kswap = inv_kswap;
                const uint32_t ci = c_lo + part * per_part;
                over_levels(O, ok, plan, l_segg[seg], ci, ci + per_part < c_hi ? ci + per_part : c_hi,
                            seg_best + (size_t)((ci - c_lo) * m_cnt + (tier > m_lo ? tier - m_lo : 0u)) * L.max_ns + seg,
                            (size_t)m_cnt * L.max_ns);
            }
            __syncthreads();
        }
        if (m_cnt > 1) {                                          // what fits a tier fits the larger ones
            const uint32_t cols = (c_hi - c_lo) * ns;
            for (uint32_t i = tid; i < cols; i += THREADS) {
                const uint32_t c = small_quot(i, inv_ns);
                unsigned long long *col = seg_best + (size_t)c * m_cnt * L.max_ns + (i - c * ns), run = col[0];
                for (uint32_t m = 1; m < m_cnt; ++m) {
                    const unsigned long long k = col[(size_t)m * L.max_ns];
                    if (k >= run) run = k;
                    else col[(size_t)m * L.max_ns] = run;
                }
            }
            __syncthreads();
        }

        // phase 3: merge with the plans without offload, write, then the running maximum along each row.  A wavefront
        // takes as many whole rows as 64 lanes hold, or one row 64 entries at a time: the running maximum is
        // a segmented scan over packed keys (throughput bits, inverted segment index, GPUs of the segment: the lower
        // segment wins among equal throughputs), a row of more than 64 entries takes the last key of the 64 before
        // along, and the plan comes from the winning segment's merged key.
        constexpr uint32_t WAVES = THREADS / 64;
        const uint32_t l16 = lane & 15u;
        for (uint32_t r0 = (tid >> 6) * r_group; r0 < pass_rows; r0 += WAVES * r_group) {
            const uint32_t rl = ns <= 64u ? r0 + q : r0;
            unsigned long long carry = 0;
            for (uint32_t base = 0; base < ns; base += 64) {
                const uint32_t s = ns <= 64u ? s_lane : base + lane;
                const bool in = ns <= 64u ? q < r_group && rl < pass_rows : s < ns;
                const uint64_t out = sbase + (uint64_t)(row0 + rl) * ns + s;
                unsigned long long ck = 0;
                if (in) {
                    unsigned long long k = seg_best[(size_t)rl * L.max_ns + s];
                    const unsigned long long kp = seg_plain[s];
                    k = kp > k ? kp : k;
                    seg_best[(size_t)rl * L.max_ns + s] = k;
                    if (best_thr) {
                        best_thr[out] = key_thr(k);
                        best_plan[out] = key_plan(k);
                    }
                    if (k >> 32) ck = (k & 0xFFFFFFFF00000000ull) | ((0xFFFFu - s) << 16) | l_segg[s];
                }
                // from the lanes below that are in the same row: within 16 lanes, then the 16 and the 32 before
                ck = scan_max_step<0x111, 0xF>(ck, s >= 1u);               // row_shr:1
                ck = scan_max_step<0x112, 0xF>(ck, s >= 2u);               // row_shr:2
                ck = scan_max_step<0x114, 0xF>(ck, s >= 4u);               // row_shr:4
                ck = scan_max_step<0x118, 0xF>(ck, s >= 8u);               // row_shr:8
                ck = scan_max_step<0x142, 0xA>(ck, s > l16);               // row_bcast:15 into lanes 16..31 and 48..63
                ck = scan_max_step<0x143, 0xC>(ck, s > lane - 32u);        // row_bcast:31 into lanes 32..63
                if (ns > 64u) {
                    ck = carry > ck ? carry : ck;
                    carry = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(ck >> 32), 63) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ck, 63);
                }
                if (in) {
                    uint32_t plan = RK_NO_PLAN;
                    if (ck) plan = key_plan(seg_best[(size_t)rl * L.max_ns + (0xFFFFu - ((uint32_t)(ck >> 16) & 0xFFFFu))]);
                    curve_thr[out] = __uint_as_float((uint32_t)(ck >> 32));
                    curve_plan[out] = plan;
                    curve_g[out] = (uint32_t)ck & 0xFFFFu;
                }
            }
        }
        __syncthreads();
    }
}

}  // namespace

int32_t rk_launch_fused(rk_ctx *ctx, const rk_jobs *jobs, const rk_plan_table *table, const rk_alloc_grid *grid,
                        const rk_env *env, uint32_t jb, uint32_t je, float *best_thr, uint32_t *best_plan,
                        float *curve_thr, uint32_t *curve_plan, uint32_t *curve_g, const TableGuard *guard, const ParkedWords *parked) {
    if (je == jb) return RK_OK;
    FusedLds L;
    L.max_nt = table->max_triples_per_job ? table->max_triples_per_job : 1;
    L.max_ns = table->max_segs_per_job ? table->max_segs_per_job : 1;
    // rows per pass so that their segment keys stay within 48 KiB: whole CPU levels (all tiers of each) when a level
    // fits, otherwise one level at a time and as many of its tiers as fit (a row of 2,048 segments takes 16 KiB)
    const size_t one_row = (size_t)L.max_ns * 8, level_bytes = (size_t)grid->n_mem * one_row;
    uint32_t c_per_pass = 1, m_per_pass = grid->n_mem;
    if (level_bytes <= 48 * 1024) {
        c_per_pass = (uint32_t)((48 * 1024) / level_bytes);
        if (c_per_pass > grid->n_cpu) c_per_pass = grid->n_cpu;
    } else {
        m_per_pass = (uint32_t)((48 * 1024) / one_row);
        if (m_per_pass < 1) return rk_fail(ctx, RK_ERR_UNSUPPORTED, "more than 6144 segments per job");
    }
    L.rows_per_pass = c_per_pass * m_per_pass;
    const bool direct = je - jb >= FUSED_MANY && c_per_pass >= grid->n_cpu && m_per_pass >= grid->n_mem;
    const size_t lds = fused_lds_bytes(L, direct);
    if (fused_lds_bytes(L, false) > 160 * 1024)                 // (so a job's triples and segments number less than 2^16)
        return rk_fail(ctx, RK_ERR_UNSUPPORTED, "job too large for the fused kernel");
    if (lds > 64 * 1024 && !ctx->fused_lds_raised) {
        for (const void *f : {reinterpret_cast<const void *>(k_fused<FEW_JOBS, false>), reinterpret_cast<const void *>(k_fused<64, true>)})
            RK_HIP(ctx, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        ctx->fused_lds_raised = true;
    }
    // Few jobs leave most of the chip idle: their CPU levels are split over workgroups, down to four levels each (every
    // one repeats phase 1, which is worth about that many).
    uint32_t split = (je - jb) < FUSED_FILL ? FUSED_FILL / (je - jb) : 1u;
    if (split > (grid->n_cpu + 3u) / 4u) split = (grid->n_cpu + 3u) / 4u;
    const uint32_t c_per_block = (grid->n_cpu + split - 1u) / split;
    split = (grid->n_cpu + c_per_block - 1u) / c_per_block;
    if (c_per_pass > c_per_block) c_per_pass = c_per_block;
    const dim3 blocks(je - jb, split);
    auto *kernel = direct ? k_fused<64, true> : k_fused<FEW_JOBS, false>;
    kernel<<<blocks, direct ? 64 : FEW_JOBS, lds, ctx->stream>>>(job_dev(jobs), table_dev(table), grid_dev(grid), *env, jb,
                                                                     table->option_mask, L, c_per_block, c_per_pass, m_per_pass,
                                                                     best_thr, best_plan, curve_thr, curve_plan, curve_g, guard ? *guard : TableGuard{},
                                                                     parked ? *parked : ParkedWords{});
    RK_CHECK_LAUNCH(ctx, "k_fused");
    return RK_OK;
}

extern "C" int32_t rk_job_curves(rk_ctx *ctx, const rk_jobs *jobs, const rk_plan_table *table,
                                 const rk_alloc_grid *grid, const rk_env *env, uint32_t jb, uint32_t je,
                                 float *best_thr, uint32_t *best_plan, float *curve_thr, uint32_t *curve_plan,
                                 uint32_t *curve_g, uint64_t cap_segs) {
    if (!ctx) return RK_ERR_INVALID_ARG;
    int32_t rc;
    if (!jobs) return rk_fail(ctx, RK_ERR_INVALID_ARG, "jobs is null");
    if ((rc = rk_check_table(ctx, table, jb, je))) return rc;
    if (jobs->n_jobs != table->n_jobs) return rk_fail(ctx, RK_ERR_INVALID_ARG, "jobs and table disagree on n_jobs");
    if ((rc = rk_check_grid(ctx, grid))) return rc;
    if ((rc = rk_check_env(ctx, env))) return rc;
    RK_HIP(ctx, hipSetDevice(ctx->device));
    uint64_t nt, ns;
    if ((rc = rk_range_offsets(ctx, table, jb, je, &nt, &ns))) return rc;
    const uint64_t need = (uint64_t)grid->n_cpu * grid->n_mem * ns;
    if (need == 0) return RK_OK;
    if (!curve_thr || !curve_plan || !curve_g) return rk_fail(ctx, RK_ERR_INVALID_ARG, "null curve buffer");
    if ((best_thr == nullptr) != (best_plan == nullptr)) return rk_fail(ctx, RK_ERR_INVALID_ARG, "best_thr and best_plan must both be given or both be null");
    if (cap_segs < need) return rk_fail(ctx, RK_ERR_CAPACITY, "outputs hold %llu entries, %llu needed",
                                        (unsigned long long)cap_segs, (unsigned long long)need);
    return rk_launch_fused(ctx, jobs, table, grid, env, jb, je, best_thr, best_plan, curve_thr, curve_plan, curve_g);
}
