// Selection of swap variables down to a load limit (Section IV-D), for K priority scores at
// once, including the submodular WDOA order of Section IV-B (iv), and load_min (Section VI-B1).
//
// Order and curve are computed apart.  A score that the curve does not change gives its order by counting: every
// candidate's rank is the number of better candidates (k_sel_order, one thread per candidate).  The SWDOA order is
// greedy and stays with one workgroup per row, but a pick only looks at a few hundred leading candidates
// (sel_greedy).  The peaks are then taken for stretches of the order side by side: a workgroup builds the curve
// before its stretch from the picks ahead of it and walks the stretch (k_sel_peaks).
// A walk of one workgroup per score over all slots and steps took 9 us a pick: 113.6 ms for the five scores
// of a 14 000-step chain, where these take 10 ms; bound now by the dependent reductions of the greedy picks.
#include "lap_dev.h"
#include "lap_kernels.h"
#include "step_runs.h"

namespace lap {

constexpr int SEL_THREADS = 1024;              // of load_min
constexpr int SEL_WAVES = SEL_THREADS / WAVE;
constexpr int ORD_THREADS = 512, ORD_WAVES = ORD_THREADS / WAVE;
constexpr int ORD_PER = 2;                     // leading candidates a thread holds
constexpr int ORD_BATCH = 8;                   // independent loads of a thread in the passes over slots and steps
constexpr uint32_t ORD_ACTIVE = ORD_THREADS * ORD_PER;
constexpr uint32_t ORD_FEW = 2 * WAVE;         // of these, the ones that one wave picks from at a time
constexpr uint32_t ORD_FEW_YIELD = 24, ORD_SIDE_MAX = 16 * ORD_FEW;
constexpr uint32_t ORD_YIELD = 10;             // picks that a choice of leading candidates has to last for
constexpr uint32_t ORD_WALK_MIN = 8, ORD_WALK_MAX = 128;   // picks without one after a choice that did not
constexpr int PK_THREADS = 256, PK_WAVES = PK_THREADS / WAVE;
constexpr int PK_PER = 8;                      // steps a thread holds
constexpr uint32_t PK_SLICE = PK_THREADS * PK_PER;
constexpr uint32_t PK_MIN_STRETCH = 16;
constexpr uint32_t PK_MAX_SLICES = 65535;      // of one launch: what the grid's y dimension takes (134 million steps)
constexpr uint32_t NONE = 0xFFFFFFFFu;

// slot list of the candidates (any order: ties are decided on the variable index) and the
// difference array of what leaves the curve when every candidate is away on all its idle steps
__global__ __launch_bounds__(256) void k_sel_gather(SelectArgs a)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    if (a.rank)
        for (uint32_t ks = 0; ks < a.K; ++ks) a.rank[(size_t)ks * a.n + i] = NONE;
    if (!a.cand[i]) return;
    const uint32_t tl = a.gap_lo ? a.gap_lo[i] : a.alloc[i];
    const uint32_t th = a.gap_hi ? a.gap_hi[i] : a.free_[i] - 1;
    const uint32_t slot = atomicAdd(a.nc, 1u);
    a.cidx[slot] = i;
    a.c_ilo[slot] = tl + 1;
    a.c_ihi[slot] = th;
    const unsigned long long s = a.size[i];
    if (th > tl + 1) {
        atomicAdd((unsigned long long *)&a.dmin[tl + 1], s);
        atomicAdd((unsigned long long *)&a.dmin[th], 0ull - s);
    }
}

// order-preserving map of a score to an unsigned key (larger = higher priority)
__device__ __forceinline__ uint64_t score_key(const SelectArgs &a, uint32_t kind, uint32_t v)
{
    switch (kind) {
    case 0: return (uint64_t)a.doa[v] ^ (1ull << 63);
    case 1: {
        const uint64_t b = (uint64_t)__double_as_longlong(a.aoa[v]);
        return (b >> 63) ? ~b : (b | (1ull << 63));
    }
    case 4: return a.cut[v];
    default: return a.wdoa[v];
    }
}

__device__ __forceinline__ uint64_t custom_key(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | (1ull << 63));
}

__device__ __forceinline__ uint64_t row_key(const SelectArgs &a, uint32_t ks, uint32_t kind, uint32_t v)
{
    return kind == 5 ? custom_key(a.custom[(size_t)ks * a.n + v]) : score_key(a, kind, v);
}

// var = NONE: no candidate; it is worse than every candidate
struct Best {
    uint64_t score;
    uint32_t var, slot;
};
__device__ __forceinline__ bool better(const Best &x, const Best &y)
{
    return x.score > y.score || (x.score == y.score && x.var < y.var);
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) { return read_lane(wave_scan_max_u32(v), WAVE - 1); }

__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v)
{
    const uint32_t hi = wave_max_u32((uint32_t)(v >> 32));
    const uint32_t lo = wave_max_u32((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
    return ((uint64_t)hi << 32) | lo;
}

// the lane among the first LANES (8 or 64; the others hold none) with the best.  Most often the upper halves of the
// scores decide alone
template <int LANES>
__device__ __forceinline__ int best_lane(uint64_t score, uint32_t var)
{
    auto top = [](uint32_t v) {
        if (LANES == WAVE) return wave_max_u32(v);
        v = max(v, dpp_mov<0x111>(0u, v));
        v = max(v, dpp_mov<0x112>(0u, v));
        v = max(v, dpp_mov<0x114>(0u, v));
        return read_lane(v, LANES - 1);
    };
    const uint32_t hi = (uint32_t)(score >> 32), lo = (uint32_t)score;
    const uint32_t m_hi = top(hi);
    bool in = hi == m_hi;
    uint64_t at = ballot(in);
    if (at & (at - 1)) {
        const uint32_t m_lo = top(in ? lo : 0u);
        in = in && lo == m_lo;
        at = ballot(in);
        if (at & (at - 1)) {
            const uint32_t nv = top(in ? ~var : 0u);
            at = ballot(in && ~var == nv);
        }
    }
    return __ffsll((unsigned long long)at) - 1;
}

// the best of the first LANES lanes, in every lane
template <int LANES>
__device__ __forceinline__ Best wave_best(const Best &b)
{
    const int src = best_lane<LANES>(b.score, b.var);
    return Best{read_lane64(b.score, src), read_lane(b.var, src), read_lane(b.slot, src)};
}

// a wave's best with all that a pick needs
struct alignas(16) Lead {
    uint64_t score, size;
    uint32_t var, slot, lo, hi;
};

struct GreedyLds {
    Best part[2][ORD_WAVES];
    Lead lead[2][ORD_WAVES];
    uint64_t score[ORD_ACTIVE];
    uint32_t var[ORD_ACTIVE], slot[ORD_ACTIVE];
    Lead few[ORD_FEW], picked[ORD_FEW];
    uint32_t few_lo[ORD_FEW], few_hi[ORD_FEW], picks;
    uint64_t wa[ORD_WAVES], wb[ORD_WAVES];
    uint32_t hist[256];
    uint32_t count, fit, held;
};

// the best of the workgroup, in every thread; one barrier.  `turn` alternates between two buffers
__device__ __forceinline__ Best block_best(const Best &mine, GreedyLds &s, int turn)
{
    const uint32_t lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    static_assert(ORD_WAVES <= 8, "one row of lanes");
    const Best w = wave_best<WAVE>(mine);
    if (lane == 0) s.part[turn][wave] = w;
    __syncthreads();
    Best o{0, NONE, NONE};
    if (lane < ORD_WAVES) o = s.part[turn][lane];
    return wave_best<8>(o);
}

// The SWDOA order of one row.  A score only falls while variables leave the curve (all of them are live on the steps
// they leave, so no step goes below zero), so a score taken earlier bounds the present one.  The workgroup holds the
// leading candidates, at most ORD_ACTIVE, in registers and corrects them after every pick (an area drops by
// size * |idle steps the winner leaves|); as long as their best beats the best of the others, as that was when it
// was last computed, it is the next pick.  When it does not, the curve's prefix sums give every score anew, and the
// leading ones are chosen again through a histogram.
//
// A pick is a chain of dependent instructions, so the shortest chain wins: of the held ones the few best, at most
// ORD_FEW, go to one wave, two a lane, which picks without a barrier as long as its best leads the rest; then the
// workgroup corrects the held ones by all of its picks at once and chooses the few again.  Where the few lead for less
// than ORD_FEW_YIELD picks all waves pick together for a while, with one barrier a pick.  3000 variables, 348 steps:
// 0.8 us a pick when all waves did every pick and one lane wrote each, 0.5 now; 4000 candidates, 1000 steps 3.34 and
// 2.28 ms.
//
// Where the scores lie close together (thousands of variables with one idle interval: every pick lowers all of them
// alike) the others soon lead and choosing anew would go with every pick.  A choice that lasts for less than ORD_YIELD
// picks is therefore followed by picks that correct every candidate's score in memory and need no choice, more of
// them each time in a row (a choice costs as much as about ten of them).  5000 candidates with one idle interval,
// 1000 steps: 144 ms when every pick chose anew, 12 ms; 12 000 of them, 14 000 steps: 842 and 54 ms.
//
// On a curve that does not contain the candidates (nc[1]; a load given by the caller may be any) scores may rise:
// nothing is held and every pick corrects every score.  20 000 candidates, 10 000 steps: 154 ms (569 ms when every
// pick took the prefix sums and all scores).
__device__ void sel_greedy(const SelectArgs &a, uint32_t ks, GreedyLds &s)
{
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const uint32_t n = a.n, T = a.T, nc = a.nc[0];
    const uint32_t cap = a.nc[1] ? 0u : ORD_ACTIVE;
    uint64_t *score = a.g_score + (size_t)ks * n;
    uint32_t *var = a.g_var + (size_t)ks * n;
    unsigned long long *dcur = (unsigned long long *)a.g_diff + (size_t)ks * ((size_t)T + 1);  // curve[t] - curve[t-1]
    uint64_t *S = a.g_sum + (size_t)ks * ((size_t)T + 1);                  // S[t] = curve[0] + .. + curve[t-1]
    for (uint32_t c = tid; c < nc; c += ORD_THREADS) var[c] = a.cidx[c];
    for (uint32_t t = tid; t < T; t += ORD_THREADS)
        __hip_atomic_store(&dcur[t], (unsigned long long)(a.load[t] - (t ? a.load[t - 1] : 0)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) S[0] = 0;
    __syncthreads();

    uint32_t k = 0;
    int turn = 0;
    auto pick = [&](uint32_t at, uint32_t v, uint32_t slot, uint64_t sc, uint64_t sz, uint32_t lo, uint32_t hi) {
        a.order[(size_t)ks * n + at] = v;
        if (a.rank) a.rank[(size_t)ks * n + v] = at;
        if (a.pick_wdoa) a.pick_wdoa[v] = sc;
        a.s_size[(size_t)ks * n + at] = sz;
        a.s_lo[(size_t)ks * n + at] = lo;
        a.s_hi[(size_t)ks * n + at] = hi;
        var[slot] = NONE;
        if (hi > lo) {                           // hi < T: the last step of an idle interval is an access
            __hip_atomic_fetch_add(&dcur[lo], 0ull - sz, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(&dcur[hi], (unsigned long long)sz, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    Best b{0, NONE, NONE};                       // the best of all, while `score` is up to date
    bool current = false;                        // whether it is
    uint32_t walk = cap ? 0u : nc, next_walk = ORD_WALK_MIN, side = 0, next_side = ORD_FEW;
    // prefix sums of the present curve, every score, and the best
    auto all_scores = [&]() {
        // the fence drops what this compute unit cached of it before the atomics
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        uint64_t ca = 0, cb = 0;
        for (uint32_t base = 0; base < T; base += ORD_THREADS * ORD_BATCH) {
            const uint32_t t0 = base + tid * ORD_BATCH;
            uint64_t d[ORD_BATCH], c1 = 0, c2 = 0;
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) d[e] = t0 + e < T ? dcur[t0 + e] : 0;
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) { c1 += d[e]; c2 += c1; }
            // over lanes: (sum of d, sum of its prefixes) of 8, 16, .. steps
            uint64_t i1 = c1, i2 = c2;
#pragma unroll
            for (int w = 1; w < WAVE; w <<= 1) {
                const uint64_t o1 = shfl_up64(i1, w), o2 = shfl_up64(i2, w);
                if ((int)lane >= w) {
                    // the lower lane's steps, then the higher one's: `mine` steps of the higher part
                    const uint64_t mine = (uint64_t)ORD_BATCH * (uint64_t)w;
                    i2 += o2 + mine * o1;
                    i1 += o1;
                }
            }
            if (lane == WAVE - 1) { s.wa[wave] = i1; s.wb[wave] = i2; }
            __syncthreads();
            uint64_t pa = ca, pb = cb, qa = 0, qb = 0;
            for (uint32_t q = 0; q < ORD_WAVES; ++q) {
                if (q == wave) { qa = pa; qb = pb; }
                pb += s.wb[q] + (uint64_t)(WAVE * ORD_BATCH) * pa;
                pa += s.wa[q];
            }
            ca = pa;
            cb = pb;
            // before this thread's steps: the waves before, then the lanes before
            const uint64_t l1 = lane_shift_up64(i1, 0), l2 = lane_shift_up64(i2, 0);
            uint64_t cur = qa + l1, sum = qb + l2 + (uint64_t)(lane * ORD_BATCH) * qa;
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) {
                cur += d[e];
                sum += cur;
                if (t0 + e < T) S[t0 + e + 1] = sum;
            }
            __syncthreads();
        }
        b = Best{0, NONE, NONE};
        for (uint32_t base = tid; base < nc; base += ORD_THREADS * ORD_BATCH) {
            uint32_t v[ORD_BATCH], lo[ORD_BATCH], hi[ORD_BATCH];
            uint64_t x[ORD_BATCH];
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) {
                const uint32_t c = min(base + e * ORD_THREADS, nc - 1);
                v[e] = base + e * ORD_THREADS < nc ? var[c] : NONE;
                lo[e] = a.c_ilo[c];
                hi[e] = a.c_ihi[c];
            }
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) x[e] = S[hi[e]] - S[lo[e]];
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) {
                if (v[e] == NONE) continue;
                const Best o{x[e], v[e], base + e * ORD_THREADS};
                score[o.slot] = x[e];
                if (better(o, b)) b = o;
            }
        }
        b = block_best(b, s, turn);
        turn ^= 1;
    };
    // one wave: how many of the 256 bins hold at most `most` candidates together, and how many those are
    auto bins_that_fit = [&](uint32_t most) {
        uint32_t h[4], t4 = 0;
        for (int e = 0; e < 4; ++e) { h[e] = s.hist[4 * lane + e]; t4 += h[e]; }
        uint32_t cum = (uint32_t)wave_scan_add_dpp(t4) - t4, bins = 0, holds = 0;
        for (int e = 0; e < 4; ++e) {
            cum += h[e];
            if (cum <= most) { bins = 4 * lane + e + 1; holds = cum; }
        }
        bins = wave_max_u32(bins);
        holds = wave_max_u32(holds);
        if (lane == 0) { s.fit = bins; s.held = holds; }
    };
    // The last wave keeps the picks, one a lane, and writes 64 of them at a time: nothing else waits for a pick's eight
    // stores.  They are written before the curve or the slots are read again.
    const bool keeps = wave == ORD_WAVES - 1;
    Lead kept{0, 0, NONE, 0, 0, 0};              // pick k_kept + lane
    uint32_t k_kept = 0;
    auto write_kept = [&]() {
        if (keeps && lane < k - k_kept) pick(k_kept + lane, kept.var, kept.slot, kept.score, kept.size, kept.lo, kept.hi);
        k_kept = k;
    };
    auto keep = [&](const Lead &w) {
        if (keeps && lane == k - k_kept) kept = w;
        ++k;
        if (k - k_kept == WAVE) write_kept();
    };
    // up to `count` picks, each followed by a correction of every candidate's score.  The first 4096 candidates' are
    // in registers meanwhile: what a pick waits for is the winner's size and window
    // (4000 candidates with one idle interval, 1000 steps: 3 us a pick when all were read and written, 1.6 now)
    auto walk_on = [&](uint32_t count) {
        constexpr uint32_t IN_REGS = ORD_THREADS * ORD_BATCH;
        uint32_t v[ORD_BATCH], lo[ORD_BATCH], hi[ORD_BATCH];
        uint64_t x[ORD_BATCH];
#pragma unroll
        for (int e = 0; e < ORD_BATCH; ++e) {
            const uint32_t c = min(tid + e * ORD_THREADS, nc - 1);
            v[e] = tid + e * ORD_THREADS < nc ? var[c] : NONE;
            lo[e] = a.c_ilo[c];
            hi[e] = a.c_ihi[c];
            x[e] = score[c];
        }
        while (count > 0 && k < nc) {
            const Lead w{b.score, a.size[b.var], b.var, b.slot, a.win_lo[b.var], a.win_hi[b.var]};
            keep(w);
            --count;
            b = Best{0, NONE, NONE};
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) {
                if (e * ORD_THREADS + wave * WAVE >= nc) break;
                const uint32_t l = max(lo[e], w.lo), h = min(hi[e], w.hi);
                x[e] -= w.size * (uint64_t)(h > l ? h - l : 0u);
                if (v[e] == w.var) v[e] = NONE;
                const Best o{x[e], v[e], tid + e * ORD_THREADS};
                if (v[e] != NONE && better(o, b)) b = o;
            }
            if (nc > IN_REGS) {
                if (tid == 0) var[w.slot] = NONE;
                for (uint32_t base = IN_REGS + tid; base < nc; base += IN_REGS) {
                    uint32_t u[ORD_BATCH], l[ORD_BATCH], h[ORD_BATCH];
                    uint64_t y[ORD_BATCH];
#pragma unroll
                    for (int e = 0; e < ORD_BATCH; ++e) {
                        const uint32_t c = min(base + e * ORD_THREADS, nc - 1);
                        u[e] = base + e * ORD_THREADS < nc && c != w.slot ? var[c] : NONE;
                        l[e] = max(a.c_ilo[c], w.lo);
                        h[e] = min(a.c_ihi[c], w.hi);
                        y[e] = score[c];
                    }
#pragma unroll
                    for (int e = 0; e < ORD_BATCH; ++e) {
                        if (u[e] == NONE) continue;
                        const Best o{y[e] - w.size * (uint64_t)(h[e] > l[e] ? h[e] - l[e] : 0u), u[e], base + e * ORD_THREADS};
                        if (h[e] > l[e]) score[o.slot] = o.score;
                        if (better(o, b)) b = o;
                    }
                }
            }
            b = block_best(b, s, turn);          // its barrier also orders the winner's slot before the next pass
            turn ^= 1;
        }
#pragma unroll
        for (int e = 0; e < ORD_BATCH; ++e)
            if (v[e] != NONE) score[tid + e * ORD_THREADS] = x[e];
        write_kept();
        __syncthreads();                         // the slots of the last picks
    };
    while (k < nc) {
        if (!current) all_scores();
        current = false;
        if (walk > 0 && nc - k > cap) {
            walk_on(cap ? min(walk, nc - k - cap) : walk);
            walk = 0;
            current = true;
            continue;
        }
        const uint32_t k_chosen = k;
        const uint64_t M = b.score;
        // the leading ones: 256 bins below the best score, those that hold at most `cap` candidates in all.  Where a
        // bin is too wide, the bins up to it are cut finer; where the best score alone has too many candidates, the
        // bins divide those by their variable
        const bool whole = nc - k <= cap;
        bool tied = false;
        uint32_t sh = 0, fit = 0, held = whole ? nc - k : 0;
        auto bin_of = [&](uint64_t x, uint32_t v) -> uint64_t {
            if (tied) return x == M ? (uint64_t)((v - b.var) >> sh) : 256ull;
            return (M >> sh) - (x >> sh);
        };
        auto load_slots = [&](uint32_t base, uint32_t (&v)[ORD_BATCH], uint64_t (&x)[ORD_BATCH]) {
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) {
                const uint32_t c = min(base + e * ORD_THREADS, nc - 1);
                v[e] = base + e * ORD_THREADS < nc ? var[c] : NONE;
                x[e] = score[c];
            }
        };
        if (!whole) {
            sh = M >> 8 ? 64 - 8 - __clzll(M) : 0;
            for (;;) {
                __syncthreads();
                if (tid < 256) s.hist[tid] = 0;
                __syncthreads();
                for (uint32_t base = tid; base < nc; base += ORD_THREADS * ORD_BATCH) {
                    uint32_t v[ORD_BATCH];
                    uint64_t x[ORD_BATCH];
                    load_slots(base, v, x);
#pragma unroll
                    for (int e = 0; e < ORD_BATCH; ++e) {
                        if (v[e] == NONE) continue;
                        const uint64_t bin = bin_of(x[e], v[e]);
                        if (bin < 256) atomicAdd(&s.hist[(uint32_t)bin], 1u);
                    }
                }
                __syncthreads();
                if (wave == 0) bins_that_fit(cap);
                __syncthreads();
                fit = s.fit;                     // 0: the first bin alone is too many
                held = s.held;
                if (held >= cap / 2 || fit >= 127) break;
                if (sh == 0 && (fit || tied)) break;   // a variable's bin of width 1 holds one candidate
                if (sh == 0) {
                    tied = true;
                    sh = n >> 8 ? 32 - 8 - __clz(n) : 0;
                    continue;
                }
                sh -= min(sh, (uint32_t)(__clz(fit + 1) - __clz(256)));
            }
        }
        __syncthreads();
        if (tid == 0) s.count = 0;
        __syncthreads();
        Best bound{0, NONE, NONE};
        for (uint32_t base = tid; base < nc; base += ORD_THREADS * ORD_BATCH) {
            uint32_t v[ORD_BATCH];
            uint64_t x[ORD_BATCH];
            load_slots(base, v, x);
#pragma unroll
            for (int e = 0; e < ORD_BATCH; ++e) {
                if (v[e] == NONE) continue;
                const Best o{x[e], v[e], base + e * ORD_THREADS};
                if (whole || bin_of(x[e], v[e]) < fit) {
                    const uint32_t at = atomicAdd(&s.count, 1u);
                    s.score[at] = x[e]; s.var[at] = v[e]; s.slot[at] = o.slot;
                } else if (better(o, bound)) bound = o;
            }
        }
        bound = block_best(bound, s, turn);      // its barrier also publishes the held ones
        turn ^= 1;
        uint64_t r_s[ORD_PER], r_size[ORD_PER];
        uint32_t r_v[ORD_PER], r_slot[ORD_PER], r_lo[ORD_PER], r_hi[ORD_PER], r_wlo[ORD_PER], r_whi[ORD_PER];
#pragma unroll
        for (int r = 0; r < ORD_PER; ++r) {
            const uint32_t e = r * ORD_THREADS + tid;
            r_v[r] = NONE; r_s[r] = r_size[r] = 0; r_slot[r] = r_lo[r] = r_hi[r] = r_wlo[r] = r_whi[r] = 0;
            if (e < held) {
                const uint32_t v = s.var[e], c = s.slot[e];
                r_s[r] = s.score[e]; r_v[r] = v; r_slot[r] = c;
                r_lo[r] = a.c_ilo[c]; r_hi[r] = a.c_ihi[c];
                r_wlo[r] = a.win_lo[v]; r_whi[r] = a.win_hi[v];
                r_size[r] = a.size[v];
            }
        }
        auto correct = [&](const Lead &w) {      // the held ones after a pick
#pragma unroll
            for (int r = 0; r < ORD_PER; ++r) {
                if (r * ORD_THREADS + wave * WAVE >= held) break;
                const uint32_t lo = max(r_lo[r], w.lo), hi = min(r_hi[r], w.hi);
                r_s[r] -= w.size * (uint64_t)(hi > lo ? hi - lo : 0u);
                if (r_v[r] == w.var) { r_v[r] = NONE; r_s[r] = 0; r_hi[r] = 0; }
            }
        };
        uint32_t sh_few = M >> 8 ? 64 - 8 - __clzll(M) : 0;
        for (;;) {
            Best top{0, NONE, NONE};
#pragma unroll
            for (int r = 0; r < ORD_PER; ++r) {
                const Best o{r_s[r], r_v[r], NONE};
                if (better(o, top)) top = o;
            }
            top = block_best(top, s, turn);
            turn ^= 1;
            if (top.var == NONE || !better(top, bound)) break;
            // the few that lead the held ones: bins below the best score again, in the width that served last
            uint32_t few_bins = 0, few = 0;
            auto few_bin = [&](uint64_t x) { return (top.score >> sh_few) - (x >> sh_few); };
            for (int tries = 0; side == 0; ++tries) {
                if (tid < 256) s.hist[tid] = 0;
                __syncthreads();
#pragma unroll
                for (int r = 0; r < ORD_PER; ++r)
                    if (r_v[r] != NONE) {
                        const uint64_t bin = few_bin(r_s[r]);
                        if (bin < 256) atomicAdd(&s.hist[(uint32_t)bin], 1u);
                    }
                __syncthreads();
                if (wave == 0) bins_that_fit(ORD_FEW);
                __syncthreads();
                few_bins = s.fit;
                few = s.held;
                if (few >= ORD_FEW / 2 || tries == 3) break;
                if (few_bins >= 255) {           // all there is nearby: a wider look, unless it is all
                    if (sh_few >= 56 || few_bin(0) < 256) break;
                    sh_few += 3;
                } else {
                    if (sh_few == 0) break;
                    sh_few -= min(sh_few, (uint32_t)(__clz(few_bins + 1) - __clz(256)));
                }
            }
            if (few == 0 || side > 0) {
                // Too many share the best score, or the few did not lead for long: all waves look for the next picks.
                // Every wave publishes its best with
                // all that the pick needs of it, so that after the barrier one look at eight entries gives the winner
                // and what it takes from the others
                Lead w{0, 0, NONE, 0, 0, 0};
                for (uint32_t picks = 0;; ++picks) {
                    correct(w);
                    if (picks == max(side, ORD_FEW)) break;
                    Best m{0, NONE, 0};
#pragma unroll
                    for (int r = 0; r < ORD_PER; ++r) {
                        const Best o{r_s[r], r_v[r], (uint32_t)r};
                        if (better(o, m)) m = o;
                    }
                    if ((int)lane == best_lane<WAVE>(m.score, m.var)) {
                        Lead o{m.score, r_size[0], m.var, r_slot[0], r_wlo[0], r_whi[0]};
#pragma unroll
                        for (int r = 1; r < ORD_PER; ++r)
                            if (m.slot == (uint32_t)r) { o.size = r_size[r]; o.slot = r_slot[r]; o.lo = r_wlo[r]; o.hi = r_whi[r]; }
                        s.lead[turn][wave] = o;
                    }
                    __syncthreads();
                    Lead g{0, 0, NONE, 0, 0, 0};
                    if (lane < ORD_WAVES) g = s.lead[turn][lane];
                    turn ^= 1;
                    const int src = best_lane<8>(g.score, g.var);
                    w.score = read_lane64(g.score, src);
                    w.var = read_lane(g.var, src);
                    if (w.var == NONE || !better(Best{w.score, w.var, 0}, bound)) break;
                    w.size = read_lane64(g.size, src);
                    w.slot = read_lane(g.slot, src);
                    w.lo = read_lane(g.lo, src);
                    w.hi = read_lane(g.hi, src);
                    keep(w);
                }
                write_kept();
                side = 0;
                continue;
            }
            if (tid == 0) s.count = 0;
            __syncthreads();
            Best rest = Best{0, NONE, NONE};
#pragma unroll
            for (int r = 0; r < ORD_PER; ++r) {
                if (r_v[r] == NONE) continue;
                if (few_bin(r_s[r]) < few_bins) {
                    const uint32_t at = atomicAdd(&s.count, 1u);
                    s.few[at] = Lead{r_s[r], r_size[r], r_v[r], r_slot[r], r_wlo[r], r_whi[r]};
                    s.few_lo[at] = r_lo[r];
                    s.few_hi[at] = r_hi[r];
                } else {
                    const Best o{r_s[r], r_v[r], NONE};
                    if (better(o, rest)) rest = o;
                }
            }
            rest = block_best(rest, s, turn);    // its barrier also publishes the few
            turn ^= 1;
            if (better(bound, rest)) rest = bound;
            if (wave == 0) {
                // one wave picks alone as long as its best leads: no barrier and no LDS between one pick and the next
                Lead c[ORD_FEW / WAVE];
                uint32_t c_lo[ORD_FEW / WAVE], c_hi[ORD_FEW / WAVE], picks = 0;
#pragma unroll
                for (int r = 0; r < (int)(ORD_FEW / WAVE); ++r) {
                    const uint32_t at = r * WAVE + lane;
                    c[r] = Lead{0, 0, NONE, 0, 0, 0};
                    c_lo[r] = c_hi[r] = 0;
                    if (at < few) { c[r] = s.few[at]; c_lo[r] = s.few_lo[at]; c_hi[r] = s.few_hi[at]; }
                }
                while (picks < ORD_FEW) {
                    Lead m = c[0];
#pragma unroll
                    for (int r = 1; r < (int)(ORD_FEW / WAVE); ++r)
                        if (better(Best{c[r].score, c[r].var, 0}, Best{m.score, m.var, 0})) m = c[r];
                    const int src = best_lane<WAVE>(m.score, m.var);
                    Lead w;
                    w.score = read_lane64(m.score, src);
                    w.var = read_lane(m.var, src);
                    if (w.var == NONE || !better(Best{w.score, w.var, 0}, rest)) break;
                    w.size = read_lane64(m.size, src);
                    w.slot = read_lane(m.slot, src);
                    w.lo = read_lane(m.lo, src);
                    w.hi = read_lane(m.hi, src);
                    if ((int)lane == src) s.picked[picks] = m;
                    ++picks;
#pragma unroll
                    for (int r = 0; r < (int)(ORD_FEW / WAVE); ++r) {
                        const uint32_t lo = max(c_lo[r], w.lo), hi = min(c_hi[r], w.hi);
                        c[r].score -= w.size * (uint64_t)(hi > lo ? hi - lo : 0u);
                        if (c[r].var == w.var) { c[r].var = NONE; c[r].score = 0; c_hi[r] = 0; }
                    }
                }
                if (lane == 0) s.picks = picks;
            }
            __syncthreads();
            const uint32_t picks = s.picks;
            if (tid < picks) {
                const Lead w = s.picked[tid];
                pick(k + tid, w.var, w.slot, w.score, w.size, w.lo, w.hi);
            }
            for (uint32_t q = 0; q < picks; ++q) correct(s.picked[q]);
            k += picks;
            k_kept = k;
            // a choice of the few costs as much as about a dozen picks by all waves
            if (picks < ORD_FEW_YIELD) {
                side = next_side;
                next_side = min(2 * next_side, ORD_SIDE_MAX);
            } else {
                next_side = ORD_FEW;
            }
        }
        if (k - k_chosen < ORD_YIELD) {
            walk = next_walk;
            next_walk = min(2 * next_walk, ORD_WALK_MAX);
        } else {
            next_walk = ORD_WALK_MIN;
        }
        __builtin_amdgcn_s_waitcnt(0);           // the curve's atomics, before the barrier that lets them be read
        __syncthreads();
    }
}

// The order of every row.  Grid: x over candidate slots (strided), y over rows.  Counting compares every pair, in
// tiles of the workgroup's width: bound by the comparisons, 11 000 candidates need 1.2e8 a row.  Greedy rows run beside
// the counted ones (one launch after the other: swap planning of 50 000 variables 1 ms longer); calls without them have
// a form of their own, since most workgroups of many rows find nothing to do and start faster with a tenth of the
// registers (64 weight vectors on 200 000 variables: 0.2 ms of 1.1).
template <bool GREEDY>
__global__ __launch_bounds__(ORD_THREADS) void k_sel_order(SelectArgs a)
{
    __shared__ uint64_t t_score[ORD_THREADS];
    __shared__ uint32_t t_var[ORD_THREADS];
    const uint32_t ks = blockIdx.y, kind = a.kinds[ks], n = a.n, nc = a.nc[0], tid = threadIdx.x;
    uint64_t *peaks = a.peaks + (size_t)ks * ((size_t)n + 1);
    for (uint32_t i = blockIdx.x * ORD_THREADS + tid; i <= nc; i += gridDim.x * ORD_THREADS) peaks[i] = 0;
    if constexpr (GREEDY) {
        __shared__ GreedyLds g;
        if (kind == 3) {
            if (blockIdx.x == 0) sel_greedy(a, ks, g);
            return;
        }
    }
    for (uint32_t base = blockIdx.x * ORD_THREADS; base < nc; base += gridDim.x * ORD_THREADS) {
        const uint32_t c = base + tid;
        const uint32_t v = c < nc ? a.cidx[c] : NONE;
        const uint64_t x = c < nc ? row_key(a, ks, kind, v) : 0;
        uint32_t before = 0;
        for (uint32_t d0 = 0; d0 < nc; d0 += ORD_THREADS) {
            __syncthreads();
            const uint32_t d = d0 + tid;
            if (d < nc) {
                const uint32_t u = a.cidx[d];
                t_var[tid] = u;
                t_score[tid] = row_key(a, ks, kind, u);
            }
            __syncthreads();
            const uint32_t cnt = min((uint32_t)ORD_THREADS, nc - d0);
#pragma unroll 8
            for (uint32_t q = 0; q < cnt; ++q) {
                const uint64_t y = t_score[q];
                before += (y > x || (y == x && t_var[q] < v)) ? 1u : 0u;
            }
        }
        if (c < nc) {
            const size_t o = (size_t)ks * n + before;
            a.order[o] = v;
            if (a.rank) a.rank[(size_t)ks * n + v] = before;
            a.s_size[o] = a.size[v];
            a.s_lo[o] = a.win_lo[v];
            a.s_hi[o] = a.win_hi[v];
        }
    }
}

// peaks[k] for one stretch of the order and one slice of the steps.  Grid: stretches, slices from `first` on, rows.  A
// wave holds 512 steps: a winner that leaves all of them lowers their maximum by its size, one that leaves none
// changes nothing, and only at the edges of its window are the steps updated and reduced.
__global__ __launch_bounds__(PK_THREADS) void k_sel_peaks(SelectArgs a, uint32_t first)
{
    __shared__ unsigned long long diff[PK_SLICE + 1];
    __shared__ uint64_t part[PK_WAVES][WAVE];
    __shared__ uint64_t wsum[PK_WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const uint32_t ks = blockIdx.z, n = a.n, T = a.T, nc = a.nc[0];
    const bool plain = a.nc[1] == 0;             // no step goes below zero
    const uint32_t len = max(PK_MIN_STRETCH, nc / gridDim.x + 1);
    const uint64_t k64 = (uint64_t)blockIdx.x * len;
    if (k64 > nc) return;
    const uint32_t k0 = (uint32_t)k64, k1 = (uint32_t)umin64((uint64_t)nc + 1, k64 + len);
    const uint64_t *sz = a.s_size + (size_t)ks * n;
    const uint32_t *slo = a.s_lo + (size_t)ks * n, *shi = a.s_hi + (size_t)ks * n;
    uint64_t *peaks = a.peaks + (size_t)ks * ((size_t)n + 1);
    const uint32_t base = (first + blockIdx.y) * PK_SLICE;
    for (uint32_t i = tid; i <= PK_SLICE; i += PK_THREADS) diff[i] = 0;
    __syncthreads();
    for (uint32_t j = tid; j < k0; j += PK_THREADS) {
        const uint32_t lo = max(slo[j], base) - base, end = shi[j];
        const uint32_t hi = end > base ? min(end - base, PK_SLICE) : 0u;
        if (hi > lo) {
            atomicAdd(&diff[lo], (unsigned long long)sz[j]);
            atomicAdd(&diff[hi], 0ull - sz[j]);
        }
    }
    __syncthreads();
    uint64_t x[PK_PER], sum = 0;
#pragma unroll
    for (int e = 0; e < PK_PER; ++e) { sum += diff[tid * PK_PER + e]; x[e] = sum; }
    const uint64_t incl = wave_scan_add(sum);
    if (lane == WAVE - 1) wsum[wave] = incl;
    __syncthreads();
    uint64_t pre = incl - sum;
    for (uint32_t q = 0; q < wave; ++q) pre += wsum[q];
    const uint32_t t0 = base + tid * PK_PER;
    uint64_t mx = 0;
#pragma unroll
    for (int e = 0; e < PK_PER; ++e) {
        x[e] = t0 + e < T ? a.load[t0 + e] - (pre + x[e]) : 0;
        mx = umax64(mx, x[e]);
    }
    mx = wave_max_u64(mx);
    // steps past the end are zero and stay out of every window (a window ends before T)
    const uint32_t w0 = base + wave * WAVE * PK_PER, w1 = w0 + min(T - w0, (uint32_t)(WAVE * PK_PER));
    uint64_t off = 0;                            // what the whole span has been lowered by and x does not show yet
    for (uint32_t kb = k0; kb < k1; kb += WAVE) {
        // lane j: the pick that leads from peak kb+j to the next one
        const uint32_t kj = kb + lane;
        uint64_t m_sz = 0;
        uint32_t m_lo = 0, m_hi = 0;
        if (kj < nc) { m_sz = sz[kj]; m_lo = slo[kj]; m_hi = shi[kj]; }
        uint64_t res = 0;
        const uint32_t cnt = min((uint32_t)WAVE, k1 - kb);
        for (uint32_t j = 0; j < cnt; ++j) {
            if (lane == j) res = mx;
            const uint64_t s = read_lane64(m_sz, (int)j);
            const uint32_t lo = read_lane(m_lo, (int)j), hi = read_lane(m_hi, (int)j);
            if (hi <= lo || hi <= w0 || lo >= w1) continue;
            if (plain && lo <= w0 && hi >= w1) {
                off += s;
                mx -= s;
                continue;
            }
            mx = 0;
#pragma unroll
            for (int e = 0; e < PK_PER; ++e) {
                const uint32_t t = t0 + e;
                if (t < T) x[e] -= off;
                if (t >= lo && t < hi) x[e] -= s;
                mx = umax64(mx, x[e]);
            }
            off = 0;
            mx = wave_max_u64(mx);
        }
        part[wave][lane] = res;
        __syncthreads();
        if (wave == 0 && lane < cnt) {
            for (int q = 1; q < PK_WAVES; ++q) res = umax64(res, part[q][lane]);
            if (T <= PK_SLICE) peaks[kj] = res;
            else atomicMax((unsigned long long *)&peaks[kj], (unsigned long long)res);
        }
        __syncthreads();
    }
}

// every limit: the shortest prefix of the order whose peak is within the limit
__global__ __launch_bounds__(256) void k_sel_limits(SelectArgs a)
{
    const uint32_t ks = blockIdx.x, nc = a.nc[0];
    const uint64_t *peaks = a.peaks + (size_t)ks * ((size_t)a.n + 1);
    if (ks == 0 && threadIdx.x == 0) *a.n_cand = nc;
    for (uint32_t q = threadIdx.x; q < a.L; q += blockDim.x) {
        const uint64_t lim = a.limits[q];
        uint32_t lo = 0, hi = nc;        // first k in [0, nc] with peaks[k] <= lim, else nc
        while (lo < hi) {
            const uint32_t m = (lo + hi) >> 1;
            if (peaks[m] <= lim) hi = m; else lo = m + 1;
        }
        a.n_selected[(size_t)ks * a.L + q] = lo;
        a.peak_after[(size_t)ks * a.L + q] = peaks[lo];
    }
}

// load_min: prefix sum of the difference array = load that leaves each step; one workgroup.  *irregular is set if a
// step would go below zero or the area under the curve may not fit in 64 bits (possible with a caller's load only)
__global__ __launch_bounds__(SEL_THREADS) void k_load_min(uint32_t T, const uint64_t *__restrict__ load,
                                                         const uint64_t *__restrict__ dmin,
                                                         uint64_t *__restrict__ out, uint32_t *irregular)
{
    __shared__ uint64_t wsum[SEL_WAVES], wmax[SEL_WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    uint64_t carry = 0, mx = 0;
    for (uint32_t base = 0; base < T; base += SEL_THREADS) {
        const uint32_t t = base + tid;
        const uint64_t d = t < T ? dmin[t] : 0;
        const uint64_t incl = wave_scan_add(d);
        if (lane == WAVE - 1) wsum[wave] = incl;
        __syncthreads();
        uint64_t pre = 0, tot = 0;
        for (int q = 0; q < SEL_WAVES; ++q) { const uint64_t x = wsum[q]; if (q < (int)wave) pre += x; tot += x; }
        __syncthreads();
        if (t < T) {
            const uint64_t x = load[t], gone = carry + pre + incl;
            if (x < gone || x > U64_MAX / T) *irregular = 1u;
            mx = umax64(mx, x - gone);
        }
        carry += tot;
    }
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) mx = umax64(mx, shfl_xor64(mx, d));
    if (lane == 0) wmax[wave] = mx;
    __syncthreads();
    if (tid == 0) {
        uint64_t m = 0;
        for (int q = 0; q < SEL_WAVES; ++q) m = umax64(m, wmax[q]);
        *out = m;
    }
}

hipError_t launch_select_swaps(const SelectArgs &a, bool gather, hipStream_t st)
{
    if (gather) {
        hipLaunchKernelGGL(k_sel_gather, dim3((a.n + 255) / 256), dim3(256), 0, st, a);
        hipLaunchKernelGGL(k_load_min, dim3(1), dim3(SEL_THREADS), 0, st, a.T, a.load, a.dmin, a.load_min, a.nc + 1);
    }
    // the number of candidates is not known here: enough workgroups for many, and few enough that the idle ones of a
    // small list cost little
    const uint32_t groups = (a.n + ORD_THREADS - 1) / ORD_THREADS, slices = (a.T - 1) / PK_SLICE + 1;
    uint32_t wide = 2048 / a.K;
    wide = wide < 16 ? 16 : wide > 128 ? 128 : wide;
    const dim3 grid(groups < wide ? groups : wide, a.K);
    if (a.greedy) hipLaunchKernelGGL(k_sel_order<true>, grid, dim3(ORD_THREADS), 0, st, a);
    else hipLaunchKernelGGL(k_sel_order<false>, grid, dim3(ORD_THREADS), 0, st, a);
    uint32_t stretches = 8192 / (slices * a.K);
    stretches = stretches < 32 ? 32 : stretches > 256 ? 256 : stretches;
    const uint32_t most = a.n / PK_MIN_STRETCH + 1;
    if (stretches > most) stretches = most;
    for (uint32_t first = 0; first < slices; first += PK_MAX_SLICES)
        hipLaunchKernelGGL(k_sel_peaks, dim3(stretches, slices - first < PK_MAX_SLICES ? slices - first : PK_MAX_SLICES, a.K),
                           dim3(PK_THREADS), 0, st, a, first);
    hipLaunchKernelGGL(k_sel_limits, dim3(a.K), dim3(256), 0, st, a);
    return hipGetLastError();
}

// Section IV-C, Eq. 3 on the raw scores: one binary64 expression per (weight vector, variable),
// evaluated left to right without contraction
__global__ __launch_bounds__(256) void k_weighted_scores(uint32_t n, uint32_t W, const double *__restrict__ weights,
                                                         const double *__restrict__ aoa,
                                                         const int64_t *__restrict__ doa,
                                                         const uint64_t *__restrict__ wdoa,
                                                         const uint64_t *__restrict__ swdoa, double *__restrict__ bo)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x, w = blockIdx.y;
    if (i >= n) return;
    const double a = weights[4 * w], b = weights[4 * w + 1], c = weights[4 * w + 2], d = weights[4 * w + 3];
    const double t1 = a * aoa[i], t2 = b * (double)doa[i];
    const double t3 = t1 + t2, t4 = c * (double)wdoa[i];
    const double t5 = t3 + t4, t6 = d * (double)swdoa[i];
    bo[(size_t)w * n + i] = t5 + t6;
}

hipError_t launch_weighted_scores(uint32_t n, uint32_t W, const double *weights, const double *aoa, const int64_t *doa,
                                  const uint64_t *wdoa, const uint64_t *swdoa, double *bo, hipStream_t st)
{
    hipLaunchKernelGGL(k_weighted_scores, dim3((n + 255) / 256, W), dim3(256), 0, st, n, W, weights, aoa, doa, wdoa,
                       swdoa, bo);
    return hipGetLastError();
}

// index of the smallest of n values, the lowest index among equals (n is small)
__global__ __launch_bounds__(WAVE) void k_argmin_u64(uint32_t n, const uint64_t *__restrict__ v, uint32_t *best)
{
    if (threadIdx.x != 0) return;
    uint32_t b = 0;
    for (uint32_t i = 1; i < n; ++i)
        if (v[i] < v[b]) b = i;
    *best = b;
}

hipError_t launch_argmin_u64(uint32_t n, const uint64_t *v, uint32_t *best, hipStream_t st)
{
    hipLaunchKernelGGL(k_argmin_u64, dim3(1), dim3(WAVE), 0, st, n, v, best);
    return hipGetLastError();
}

}  // namespace lap
