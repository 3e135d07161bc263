// Host-side launch wrappers of the liblap kernels (one per kernel family).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lap {

// candidate segment widths of the segment kernel: 2^PLAN_SEG_SHIFT0 .. 2^(PLAN_SEG_SHIFT0 + PLAN_SEG_CAND - 1) steps
constexpr uint32_t PLAN_SEG_SHIFT0 = 2, PLAN_SEG_CAND = 9;
// list entries of the segment kernel's pool per ordering and variable (the pool is shared: an
// ordering that needs more leaves fewer slots)
constexpr uint32_t PLAN_SEG_BUDGET = 27;

// Per-call facts about the trace, computed on the device before placement.
struct PlanHeader {
    unsigned long long or_sizes;   // bitwise OR of all sizes
    unsigned long long sum_sizes;  // sum of all sizes (bytes)
    uint32_t n_multi;              // variables that live for more than one step
    uint32_t shift;                // log2 of the offset granule: ctz(or_sizes)
    uint32_t fast;                 // 1: sum_sizes >> shift fits 32 bits -> packed 32-bit path
    uint32_t mode1;                // 1: per-step lists are in use (sum of lifetimes <= PLAN_CL * N, and not reg_before_lists)
    uint32_t part[2];              // placement workgroups that have started, per fit policy
    uint32_t progress[2];          // their progress, in units of 512 ranks, summed
    // segment lists (place_seg.hip), used when per-step lists are not and the pool has room
    uint32_t mode2;                // 1: the segment kernel places this trace; 2: the batches do, or have
    uint32_t seg_shift;            // log2 of the segment width in steps
    uint32_t seg_K;                // number of segments
    uint32_t seg_slots;            // orderings that have room in the list pool at once
    unsigned long long seg_need;   // list entries one ordering needs
    unsigned long long seg_tot[PLAN_SEG_CAND];   // per candidate width: blocks entered into lists, summed over the variables
    uint32_t seg_trial_rounds;     // trial run: search rounds of its multi-step variables, summed
    uint32_t seg_trial_vars;       // ... and how many those were
    uint32_t seg_next;             // next ordering to hand to a workgroup of the segment kernel
    uint32_t seg_pad;
};
constexpr uint32_t PLAN_CL = 6;

// Placed blocks in registers (place_reg.hip): whether they may be used: 128 rows of 256 entries, 16-bit
// steps ...
constexpr uint32_t PLAN_REG_MAX_VARS = 128 * 256;
inline bool reg_may_place(uint32_t n, uint32_t T) { return n <= PLAN_REG_MAX_VARS && T <= 0xFFFFu; }
// ... and whether they are, as far as the trace decides it: where per-step lists are not in use.  Up to 128 variables,
// and up to 768 where the second rule says so (the preparation asks it), these are not used although lifetimes are short
// enough for them.  A one-step variable costs the lists next to nothing and a multi-step one 3 to 5 us, while every
// variable costs the registers 0.25 us and more for each row it asks: up to three rows the registers win from a share
// of multi-step variables on that grows with the rows (times in registers over times with the lists, 16 best-fit
// orderings: 256 variables, one row, 1.16 at 2 % and 0.89 at 4 %; 512 variables 1.12 and 0.87 at 4 and 6 %; 768
// variables 1.09 and 0.90 at 6 and 8 %), and is that of one row less where orderings share the compute units (1024 of
// them: 256 variables 0.89 at 2 %, 512 variables 1.02 and 0.91 at 2 and 4 %, 768 variables 1.08 and 0.98 at 4 and 6 %).
// Larger traces always go to the lists (6000 variables, mostly one-step: 7.1 and 2.9 ms).  Up to 128 variables there is
// nothing in it (150 of them at 2 %: 0.97 to 1.09), the registers take all and the lists' launch is saved.
constexpr uint32_t PLAN_REG_ALWAYS_VARS = 128, PLAN_REG_FEW_VARS = 3 * 256;
__device__ __forceinline__ bool reg_places(const PlanHeader *hdr, uint32_t n, bool best_fit)
{
    if (!hdr->fast || (hdr->mode2 && !best_fit)) return false;
    return !hdr->mode1 || n <= PLAN_REG_ALWAYS_VARS;
}
__device__ __forceinline__ bool reg_before_lists(uint32_t n, uint32_t T, uint32_t n_multi, uint32_t B)
{
    return n <= PLAN_REG_FEW_VARS && T <= 0xFFFFu && n_multi * 40u >= n * ((n + 255) / 256 - (B > 512 ? 1u : 0u));
}

// Up to 64 variables placed at a time (place_batch.hip): whether that takes the place of the registers, and of the sweep.
// First-fit calls only: with best-fit orderings among them the registers place all in one launch.  What the trace has to do with
// it is batches_lose's.  ms in registers and in batches, of a residual chain, a pyramid of feature maps, and random lifetimes
// with six sizes:
//     256 orderings of   700   0.31 0.32 0.31 and 0.28 0.28 0.53      512 of   700   0.35 0.34 0.35 and 0.30 0.31 0.60
//                       1500   0.97 0.97      and 0.54 0.66                   1500   1.04 1.04      and 0.59 0.72
//                       3000   2.42 2.43 2.43 and 1.18 1.54 2.25              3000   2.95           and 1.34 1.74 2.64
//                     10 000             13.0 and           10.5            10 000             17.2 and           10.5
//                       9001   11.2           and 4.9                         9001   15.0           and 7.9
//     768            of 1500   1.02 1.02      and 0.99 1.09      1024 of      3000   2.86           and 2.69 2.89 3.44
//                       2500   2.20 2.20      and 1.81 1.96                   5000   11.5 11.6      and 4.8 5.3
//                       6400   13.8 14.2 13.7 and 6.9 7.5 7.0                 9001   29.3           and 14.4
// 2048 orderings of 3300: 4.38 and 5.25, of 5000 20.3 and 9.0.  Of a chain with the blocks in memory: 256 orderings of 13 400 20.4
// and 8.6, of 20 000 38.2 and 14.4, of 32 767 98 and 32; 1024 of 20 000 152 and 43; random lifetimes and six sizes: 100 of 15 000
// 23.4 and 19.7, 200 of 25 000 62.9 and 42.5.  More than 32 768 take the place of the sweep
// (40 000, random: 3.2 s by the sweep, 0.08 in batches).
constexpr uint32_t PLAN_BATCH_MAX_VARS = 1 << 17;
constexpr uint32_t PLAN_BATCH_LDS_VARS = 52 * 256 - 1;      // rows of 512 entries of 12 bytes in 160 KB, less 4 KB
inline bool batch_places(uint32_t n, uint32_t T, uint32_t B, bool any_best)
{
    return !any_best && n <= PLAN_BATCH_MAX_VARS && T <= 0xFFFFu && (n > 4096 || (n > 2048 && B <= 768) || (n > 1024 && B <= 512));
}

// Whether the registers are the faster ones all the same (where they may place: up to PLAN_REG_MAX_VARS).  A batch ends where a
// variable has been shown too few holes.  In a training iteration blocks are freed in the reverse order of their allocation and
// a hole takes many; where lifetimes cross, holes lie apart and are taken by one variable each, so that of equal sizes few
// go into a batch in an order that follows the trace (shuffled orderings place variables that are apart in time).
// meet, cross, equal: of 2048 pairs of variables that are listed close to each other, those that meet in time, those of them
// of which the one allocated first is freed first, and those of one size.  cross is at most 2 % of meet in the three families of
// training iterations and 15 % and more with lifetimes at random.  Times in registers over times in batches, lifetimes at
// random (18 shapes: short to long, some of one step, uniform and heavy-tailed), by the number of sizes:
//     orderings  variables      one       six        40         1000      shuffled only, 1 to 1000 sizes
//     16            1100     0.4        0.6  0.9                0.7 0.8   1.2  2.1
//                   1600                0.7  0.9                0.8 1.0   1.4  2.4
//                   2200                0.7  1.1                0.9 1.1   1.6  2.9
//                   3000     0.5  0.8   0.75 1.0   0.9  1.1     1.0
//                   9000     0.6  0.9   0.9  1.3   1.1  1.4     1.2
//                 14 000     0.5        0.75 1.1   0.9  1.2     1.15
//                 20 000     0.6        0.75 1.1   0.95 1.25    1.2
//                 30 000     0.65       0.95 1.3                1.4
//     512           1100     0.4        0.6                               0.8  1.4
//                   2200                                                  1.1  1.9
//                   3000     0.5  0.8   0.8  1.1   0.95 1.2               1.1  2.2
//                   9000     0.7  1.3   0.8  1.5   0.9  1.6               1.0  2.2
//           14 000, 20 000              1.2  1.8   1.5  1.9
//     1024          5000     1.0        1.3
//                   9000     0.8        0.85
//           13 000, 14 000   1.2        1.4
struct BatchTrial {
    bool first;                  // batches go before the segment lists where batches_before_segments says so
    bool look;                   // batches_lose decides about registers and batches (the second header is for the batches:
                                 // `fast` is not set there where the registers are to place)
    bool by_trace;               // there are other orderings than shuffles
};
__device__ __forceinline__ bool batches_lose(uint32_t n, uint32_t B, bool by_trace, uint32_t meet, uint32_t cross, uint32_t equal)
{
    if (cross * 8 < meet) return false;
    if (!by_trace) return n < 1536 && B > 256;
    if (equal * 3 > meet) return B <= 512 || n <= 10240;
    if (equal * 10 <= meet) return n < 2560;
    if (n > PLAN_BATCH_LDS_VARS) return n <= 24576 && B <= 256;
    return n < 4096 || (cross * 5 > meet * 2 && (B <= 512 || (n > 6143 && n <= 10240)));
}

// Whether they go before the segment lists.  All placed blocks are gone through for every batch, one ordering of 16 waves or two of
// 8 to a compute unit; the lists take a time that goes with their entries (and with how their searches converge, which this
// does not know), and from some 1000 orderings on with these as well.  ms with the lists and in batches, with the entries of a
// variable, of a residual chain, a pyramid of feature maps, and feature maps among one-step temporaries of random sizes:
//     orderings          16        256         600         1024        2048      4096
//     chain     33 000 (49)        427 32                  500 103               757 387
//               50 000 (63)        848 65                  764 215               1114 811
//               70 000 (79) 885 109 826 113    954 323     1011 413
//     pyramid   33 000 (20)        133 39                  176 121               552 452
//               50 000 (22) 183 68 209 71      255 200     282 256     514 493   908 955
//               70 000 (25) 253 125 296 133    364 375     405 480
//              100 000 (31) 734 251 857 261    921 737     991 951
//              131 072 (37) 922 407 1159 432   1278 1259   1337 1368
//     maps      33 000 (18)        172 46      177 95      183 125     280 241
//               50 000 (19)        364 95      374 203     381 268     423 511
//               70 000 (22)        465 177     484 381     489 509     604 952
// It is wrong by more than a tenth for the pyramid of 70 000 with 1024 orderings only.
__device__ __forceinline__ bool batches_before_segments(uint32_t n, uint32_t B, uint64_t need)
{
    const uint64_t rounds = (B + 255) / 256;
    return (uint64_t)n * n * rounds < need * (6700 + 1600 * rounds);
}

hipError_t launch_fill_u64(uint64_t *p, size_t n, uint64_t v, hipStream_t st);
// copies n_words 32-bit words of HOST memory to the device through kernel arguments (the host
// array is read before the call returns; nothing waits)
hipError_t launch_put_words(void *dst, const void *host_src, size_t n_words, hipStream_t st);
hipError_t launch_delta(uint32_t n, uint32_t T, const uint64_t *size, const uint32_t *alloc, const uint32_t *free_,
                        uint64_t *delta, hipStream_t st);
hipError_t launch_scan_peak(uint32_t T, uint64_t *delta, uint64_t *load, uint64_t *peak, uint32_t *t_peak,
                            hipStream_t st);
// The load profile in one launch by one workgroup.  The three launches (fill, scatter, scan) take 11.4 to 12.9 us whatever
// the number of variables up to 50 000; this one 6.4 us for 100 of them, 8 to 9 us for 8000, 9.6 to 11.7 us for 16 000
// and 13 to 17 us for 32 768 (20 to 2000 steps).  8191 steps: 8.8 to 11.6 us up to 16 000, and 17 us by three.  (By
// k_delta_line the three take 1 to 3 us less: whole calls of 16 384 variables 26 to 29 us, of 16 385 29 to 33.)
constexpr uint32_t LOAD_SMALL_VARS = 16384, LOAD_SMALL_STEPS = 8191;
hipError_t launch_load_small(uint32_t n, uint32_t T, const uint64_t *size, const uint32_t *alloc, const uint32_t *free_,
                             uint64_t *load, uint64_t *peak, uint32_t *t_peak, hipStream_t st);
hipError_t launch_validate(uint32_t n, uint32_t T, const uint64_t *size, const uint32_t *alloc, const uint32_t *free_,
                           const uint32_t *gap_lo, const uint32_t *gap_hi, const uint64_t *step_ns, uint64_t *out8,
                           hipStream_t st);

hipError_t launch_sort_perm(uint32_t n, uint32_t B, const uint64_t *size, const uint32_t *alloc, const uint32_t *free_,
                            const uint32_t *kinds, const uint64_t *seeds, uint32_t *perm, uint32_t *tmp,
                            bool any_explicit, hipStream_t st);
hipError_t launch_plan_prep(uint32_t n, uint32_t T, uint32_t B, const uint64_t *size, const uint32_t *alloc,
                            const uint32_t *free_, uint32_t *cntd, uint32_t *lstart, PlanHeader *hdr, void *vrec,
                            uint64_t seg_pool_entries, uint64_t seg_min_vars, BatchTrial batches, hipStream_t st);
hipError_t launch_seg_prep(uint32_t n, uint32_t T, uint32_t B, const uint32_t *alloc, const uint32_t *free_,
                           PlanHeader *hdr, uint32_t *cnt, uint32_t *lst, uint32_t dir_cap, uint64_t pool_entries,
                           hipStream_t st);
// trial_b: ordering whose first ranks are placed ahead of time to see how the searches go (negative:
// no trial); trial_percent: rounds per multi-step variable, times 100, above which the sweep is kept
hipError_t launch_seg_trial(uint32_t n, uint32_t T, uint32_t B, const uint32_t *perm, const uint32_t *fits,
                            int trial_b, uint32_t trial_percent, PlanHeader *hdr, const void *vrec, const uint32_t *lst,
                            uint64_t *pool, uint32_t *lens, uint32_t dir_cap, uint64_t *offs, uint64_t *fps,
                            uint64_t *ticks, hipStream_t st);
hipError_t launch_place_seg(uint32_t n, uint32_t T, uint32_t B, const uint32_t *perm, const uint32_t *fits,
                            bool any_first, PlanHeader *hdr, const void *vrec, const uint32_t *lst,
                            uint64_t *pool, uint32_t *lens, uint32_t dir_cap, uint64_t *offs, uint64_t *fps,
                            uint64_t *ticks, hipStream_t st);
hipError_t launch_place_reg(uint32_t n, uint32_t T, uint32_t B, const uint32_t *perm, const uint32_t *fits, bool any_best,
                            const PlanHeader *hdr, const void *vrec, uint64_t *offs, uint64_t *fps, uint64_t *ticks,
                            hipStream_t st);
// hdr: the second one where the preparation has looked at registers and batches; blocks [B][4 n]: scratch
hipError_t launch_place_batch(uint32_t n, uint32_t B, const uint32_t *perm, PlanHeader *hdr, const void *vrec,
                              uint32_t *blocks, uint64_t *offs, uint64_t *fps, uint64_t *ticks, hipStream_t st);
hipError_t launch_place_fast(uint32_t n, uint32_t T, uint32_t B, const uint64_t *size, const uint32_t *alloc,
                             const uint32_t *free_, const uint32_t *perm, const uint32_t *fits, bool any_first,
                             bool any_best, PlanHeader *hdr, const void *vrec,
                             const uint32_t *lstart, uint64_t *m_oe, uint64_t *m_life, uint64_t *m_oe2,
                             uint64_t *m_life2, uint64_t *r_oe, uint64_t *r_life, uint64_t *r_oe2,
                             uint64_t *r_life2, uint64_t *L, uint64_t capL,
                             uint32_t *l_ns, uint32_t *l_nu, uint64_t *offs, uint64_t *fps, uint64_t *ticks,
                             hipStream_t st);
constexpr uint32_t PLAN_REC = 4096;   // entries of the sorted "recent" list per ordering
hipError_t launch_place_wide(uint32_t n, uint32_t B, const uint64_t *size, const uint32_t *alloc,
                             const uint32_t *free_, const uint32_t *perm, const uint32_t *fits,
                             const PlanHeader *hdr, uint64_t *m_off,
                             uint64_t *m_end, uint64_t *m_life, uint64_t *offs, uint64_t *fps, uint64_t *ticks,
                             hipStream_t st);
hipError_t launch_select(uint32_t n, uint32_t B, const uint64_t *fps, const uint64_t *offs_rank, const uint32_t *perm,
                         uint64_t *best_fp, uint32_t *best_idx, uint64_t *best_offsets, uint64_t *all_offsets,
                         hipStream_t st);

hipError_t launch_swap_prefix(uint32_t T, const uint64_t *load, const uint64_t *step_ns, uint64_t *C, uint64_t *S,
                              uint64_t *PM, uint64_t *SM, uint64_t *peak, uint32_t *t_peak, uint64_t *table,
                              uint32_t levels, hipStream_t st);
hipError_t launch_score(uint32_t n, uint32_t T, const uint64_t *size, const uint32_t *alloc, const uint32_t *free_,
                        const uint32_t *gap_lo, const uint32_t *gap_hi, uint64_t bpus, uint64_t min_bytes,
                        const uint64_t *load, const uint64_t *C, const uint64_t *S, const uint64_t *PM,
                        const uint64_t *SM, const uint64_t *table, const uint64_t *peak, const uint32_t *t_peak,
                        uint8_t *cand, int64_t *doa, double *aoa, uint64_t *wdoa, uint64_t *cut, uint32_t *win_lo,
                        uint32_t *win_hi, hipStream_t st);

// Selection of swap variables (select_swaps.hip).  All pointers are device memory.
struct SelectArgs {
    uint32_t n, T, K, L;
    const uint64_t *size;
    const uint32_t *gap_lo, *gap_hi, *alloc, *free_;
    const uint64_t *load;
    const uint8_t *cand;
    const int64_t *doa;
    const double *aoa;
    const uint64_t *wdoa, *cut;
    const uint32_t *win_lo, *win_hi;
    uint32_t *nc;              // [2] number of candidates (device counter), 1 if the load does not contain them
    uint32_t *cidx;            // [n] candidate slot -> variable
    uint32_t *c_ilo, *c_ihi;   // [n] idle steps [ilo, ihi) of the candidate in a slot
    uint64_t *dmin;            // [T+1] difference array of the load removed for load_min
    const uint32_t *kinds;     // [K]
    bool greedy;               // whether one of them is 3
    const uint64_t *limits;    // [L]
    uint64_t *s_size;          // [K][n] size of the j-th pick
    uint32_t *s_lo, *s_hi;     // [K][n] steps [lo, hi) that the j-th pick leaves
    uint64_t *g_score;         // rows of kind 3, [K][n]: score of every slot when it was last computed
    uint32_t *g_var;           // [K][n]: variable of the slot, 0xFFFFFFFF once taken
    uint64_t *g_diff, *g_sum;  // [K][T+1]: differences and prefix sums of the current load curve
    uint32_t *order, *rank;    // [K][n] outputs (rank may be null)
    uint64_t *peaks;           // [K][n+1]
    uint32_t *n_cand;          // [1]
    uint32_t *n_selected;      // [K][L]
    uint64_t *peak_after;      // [K][L]
    uint64_t *load_min;        // [1]
    const double *custom;      // [K][n] score of kind 5 (custom), row = position in kinds; else null
    uint64_t *pick_wdoa;       // [n] or null: for a SWDOA walk, the score a variable had when it was picked
};
// gather = build the candidate slots and load_min first (once per trace and candidate filter)
hipError_t launch_select_swaps(const SelectArgs &a, bool gather, hipStream_t st);
hipError_t launch_weighted_scores(uint32_t n, uint32_t W, const double *weights, const double *aoa, const int64_t *doa,
                                  const uint64_t *wdoa, const uint64_t *swdoa, double *bo, hipStream_t st);
hipError_t launch_argmin_u64(uint32_t n, const uint64_t *v, uint32_t *best, hipStream_t st);

// perm_lo, perm_hi = the listed variables in the order of (access step, index).  posmap (null where no variable is listed
// twice): position of every listed variable, filled here.  count_dev: the length of the list, where only the device knows
// it (then count is not used, and posmap null)
struct ListedOrder {
    uint32_t n, count;
    const uint32_t *count_dev, *list, *step_lo, *step_hi;
    uint32_t *posmap, *perm_lo, *perm_hi;
};
// Longer lists leave it to the sorts of all variables: counting grows with the square of the list (31 us for 11 000 variables,
// about 70 for 16 384), two sorts take 0.25 ms for 16 384 variables and 0.78 ms for 50 000.  A list whose length only the
// device knows is always counted: 43 us for 16 000 variables, 0.15 ms for 30 000, 0.57 for 60 000, 2.3 for 120 000 and 6.1
// for 200 000 (two sorts 0.13, 0.25, 0.53, 1.05 and 1.8 ms), of a call that takes 20 ms for 16 000 and 340 for 120 000.
constexpr uint32_t RANK_LISTED = 16384;
hipError_t launch_order_listed(const ListedOrder &L, hipStream_t st);
hipError_t launch_sched_mark(uint32_t n, uint32_t k, const uint32_t *list, uint32_t *posmap, hipStream_t st);

// perm_lo, perm_hi: `count` variables in the order of their access steps; those that are listed are the ones in posmap
hipError_t launch_schedule_swaps(uint32_t n, uint32_t T, uint32_t k, uint32_t count, const uint64_t *size,
                                 const uint32_t *step_lo, const uint32_t *step_hi, uint32_t hi_minus, const uint64_t *C,
                                 const uint32_t *perm_lo, const uint32_t *perm_hi, const uint32_t *posmap,
                                 const uint32_t *list, uint64_t bpus, int64_t *out_start, int64_t *out_end,
                                 int64_t *in_start, int64_t *in_end, uint64_t *diff, uint64_t *late,
                                 const uint64_t *load, uint64_t *load_sched, uint64_t *peak, hipStream_t st);

// place_lo: scratch, n entries per list; perm_lo, perm_hi, count as above, or count_dev
hipError_t launch_simulate_swaps(uint32_t n, uint32_t T, uint32_t Q, uint32_t kmax, uint32_t count,
                                 const uint32_t *count_dev, const uint64_t *size,
                                 const uint32_t *alloc, const uint32_t *free_, const uint32_t *step_lo,
                                 const uint32_t *step_hi, uint32_t hi_minus, const uint64_t *C, uint64_t *need,
                                 uint64_t *rel, const uint32_t *list, const uint32_t *perm_lo,
                                 const uint32_t *perm_hi, const uint32_t *posmap, uint32_t *jobs_lo,
                                 uint32_t *jobs_hi, uint32_t *m, const uint32_t *prefix, const uint64_t *limits,
                                 uint32_t *kb, uint32_t *place_lo, uint64_t bpus, uint64_t *total_ns,
                                 uint64_t *overhead_ns, uint64_t *peak_resident, uint32_t *forced, hipStream_t st,
                                 uint32_t n_lists = 1, const uint32_t *n_listed = nullptr);

// Q [M] prefix hashes, totals [DI_MAX_TILES]: scratch
constexpr uint32_t DI_MAX_TILES = 4096;
hipError_t launch_detect_iteration(const uint64_t *tokens, uint32_t M, uint32_t min_period, uint64_t *Q,
                                   uint64_t *totals, uint32_t *period, hipStream_t st);

}  // namespace lap
