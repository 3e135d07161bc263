// The swap schedule under a memory-load limit (Section IV-E): a Malloc that would exceed the limit
// waits until enough has been swapped out, a swap-in starts only when its bytes fit.  One iteration
// is replayed as a discrete-event machine with three actors (compute, the swap-out stream, the
// swap-in stream); the result is the time lost against the plain iteration.
//
// The machine is sequential; the parallel dimension is the set of (swap list prefix, limit) pairs to
// evaluate -- a sweep of limits, several priority orders -- one workgroup each for the planned swap-in
// starts and one wave each for the machine.  Shared by all of them and built by data-parallel kernels:
// bytes allocated and freed per step, and the listed variables in swap-out order and in swap-in order
// (positions in the list, so that "the first k of the list" is a filter).
#include "lap_dev.h"
#include "lap_kernels.h"
#include "step_runs.h"
#include "stream_scan.h"
#include <type_traits>

namespace lap {

constexpr int SIM_THREADS = 1024;
constexpr int SIM_WAVES = SIM_THREADS / WAVE;
constexpr int SIM_PER = 8;                         // ranks per thread and round of the job lists
constexpr int RUN_THREADS = 512, RUN_WAVES = RUN_THREADS / WAVE;
constexpr int RUN_BATCH = 4;                       // entries a lane loads side by side
constexpr uint32_t RUN_WIN = RUN_BATCH * WAVE;     // entries of each stream held in LDS
constexpr uint32_t SIM_NONE = 0xFFFFFFFFu;
constexpr uint32_t SIM_NEVER = 0x7FFFFFFFu;        // what the narrow machine does not hold: times, sums of sizes, steps
constexpr uint32_t SIM_WIDE = 64;                  // instead of a granule's shift

// Bytes allocated and freed per step.  Neighbours allocate at the same step and long-lived ones free at the same: a wave's
// runs are summed before they reach memory (200 000 variables over 580 steps: 4.4 us, 114 with an atomic per variable).
__global__ __launch_bounds__(256) void k_sim_steps(uint32_t n, const uint64_t *__restrict__ size,
                                                   const uint32_t *__restrict__ alloc,
                                                   const uint32_t *__restrict__ free_, unsigned long long *need,
                                                   unsigned long long *rel)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool in = i < n;
    const uint64_t s = in ? size[i] : 0;
    wave_add_runs(in ? alloc[i] : NO_KEY, s, [&](uint32_t t, uint64_t v) { atomicAdd(&need[t], (unsigned long long)v); });
    wave_add_runs(in ? free_[i] - 1 : NO_KEY, s, [&](uint32_t t, uint64_t v) { atomicAdd(&rel[t], (unsigned long long)v); });
}

// several lists, one row of n entries each: position map of list r = row r.  Row r lists the first
// n_listed[0] entries of its row of `lists`.
__global__ __launch_bounds__(256) void k_sim_mark_rows(uint32_t n, const uint32_t *__restrict__ lists,
                                                       const uint32_t *__restrict__ n_listed,
                                                       uint32_t *__restrict__ posmap)
{
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x, r = blockIdx.y;
    if (j < *n_listed) posmap[(size_t)r * n + min(lists[(size_t)r * n + j], n - 1)] = j;
}

// The bytes resident when nothing is swapped, at their highest, and the bitwise or of all that a step allocates or
// frees: what the machine's numbers have to hold.  One workgroup.
__device__ void sim_extent(uint32_t T, const unsigned long long *__restrict__ need, const unsigned long long *__restrict__ rel,
                           uint64_t *__restrict__ peak, uint64_t *__restrict__ bits)
{
    __shared__ uint64_t wsum[2][SIM_WAVES], wmax[SIM_WAVES], wor[SIM_WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    uint64_t carry = 0, mx = 0, all = 0;
    int buf = 0;
    for (uint64_t base = 0; base < T; base += SIM_THREADS, buf ^= 1) {
        const uint64_t t = base + tid;
        const uint64_t a = t < T ? need[t] : 0, r = t < T ? rel[t] : 0;
        const uint64_t incl = wave_scan_add_dpp(a - r);
        if (lane == WAVE - 1) wsum[buf][wave] = incl;
        __syncthreads();
        uint64_t at = carry + incl + r;                // during the step: what it frees is still there
        for (int q = 0; q < SIM_WAVES; ++q) { const uint64_t x = wsum[buf][q]; if (q < (int)wave) at += x; carry += x; }
        mx = umax64(mx, at);
        all |= a | r;
    }
    mx = wave_reduce_max(mx);
#pragma unroll
    for (int d = WAVE / 2; d > 0; d >>= 1) all |= shfl_xor64(all, d);
    if (lane == 0) { wmax[wave] = mx; wor[wave] = all; }
    __syncthreads();
    if (tid == 0) {
        for (int q = 1; q < SIM_WAVES; ++q) { mx = umax64(mx, wmax[q]); all |= wor[q]; }
        *peak = mx;
        *bits = all;
    }
}

// jobs[0..m) = list positions of the listed variables that have an idle gap, in the order of perm (count entries);
// one workgroup per list (rows of n entries of posmap and jobs, one count each) and direction
// (blockIdx.y: swap-outs, swap-ins); place_lo: the place of a list position in jobs_lo.  Every round
// waits for two dependent loads, so a thread takes SIM_PER ranks per round.
__global__ __launch_bounds__(SIM_THREADS) void k_sim_jobs(uint32_t n, uint32_t count,
                                                          const uint32_t *__restrict__ count_dev,
                                                          const uint32_t *__restrict__ perm_lo,
                                                          const uint32_t *__restrict__ perm_hi,
                                                          const uint32_t *__restrict__ posmap_all,
                                                          const uint32_t *__restrict__ step_lo,
                                                          const uint32_t *__restrict__ step_hi, uint32_t hi_minus,
                                                          uint32_t *__restrict__ jobs_lo,
                                                          uint32_t *__restrict__ jobs_hi,
                                                          uint32_t *__restrict__ place_lo_all,
                                                          uint32_t *__restrict__ m_all, uint32_t T,
                                                          const unsigned long long *__restrict__ need,
                                                          const unsigned long long *__restrict__ rel,
                                                          uint64_t *__restrict__ extent_peak, uint64_t *__restrict__ extent_bits)
{
    __shared__ uint32_t wsum[2][SIM_WAVES];
    if (blockIdx.y == 2) {
        if (blockIdx.x == 0) sim_extent(T, need, rel, extent_peak, extent_bits);
        return;
    }
    uint32_t *place_lo = place_lo_all + (size_t)blockIdx.x * n;
    const uint32_t *perm = blockIdx.y ? perm_hi : perm_lo;
    const uint32_t *posmap = posmap_all + (size_t)blockIdx.x * n;
    uint32_t *jobs = (blockIdx.y ? jobs_hi : jobs_lo) + (size_t)blockIdx.x * n;
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    const uint64_t below = (1ull << lane) - 1ull;
    if (count_dev) count = *count_dev;
    uint32_t carry = 0;
    int buf = 0;
    for (uint64_t base = 0; base < count; base += SIM_THREADS * SIM_PER, buf ^= 1) {
        const uint64_t r0 = base + wave * (WAVE * SIM_PER) + lane;
        uint32_t v[SIM_PER], pos[SIM_PER];
        uint64_t mine[SIM_PER];
#pragma unroll
        for (int j = 0; j < SIM_PER; ++j) v[j] = r0 + j * WAVE < count ? perm[r0 + j * WAVE] : SIM_NONE;
#pragma unroll
        for (int j = 0; j < SIM_PER; ++j) pos[j] = v[j] != SIM_NONE ? posmap[v[j]] : SIM_NONE;
        uint32_t tot = 0;
#pragma unroll
        for (int j = 0; j < SIM_PER; ++j) {
            if (pos[j] != SIM_NONE && step_hi[v[j]] - hi_minus <= step_lo[v[j]]) pos[j] = SIM_NONE;
            mine[j] = ballot(pos[j] != SIM_NONE);
            tot += (uint32_t)__popcll(mine[j]);
        }
        if (lane == 0) wsum[buf][wave] = tot;
        __syncthreads();
        uint32_t at = carry;
        for (int q = 0; q < SIM_WAVES; ++q) { const uint32_t x = wsum[buf][q]; if (q < (int)wave) at += x; carry += x; }
#pragma unroll
        for (int j = 0; j < SIM_PER; ++j) {
            if (pos[j] != SIM_NONE) {
                const uint32_t to = at + (uint32_t)__popcll(mine[j] & below);
                jobs[to] = pos[j];
                if (blockIdx.y == 0) place_lo[pos[j]] = to;
            }
            at += (uint32_t)__popcll(mine[j]);
        }
    }
    if (tid == 0 && blockIdx.y == 0) m_all[blockIdx.x] = carry;     // the same number both ways
}

struct SimArgs {
    uint32_t n, T, Q, kmax;
    const uint64_t *size;
    const uint32_t *step_lo, *step_hi;
    uint32_t hi_minus;
    const uint64_t *C;
    const unsigned long long *need, *rel;
    const uint32_t *list;
    const uint32_t *jobs_lo, *jobs_hi, *place_lo, *m;
    const uint32_t *prefix;            // [Q]
    const uint64_t *limits;            // [Q]
    uint32_t *kb;                      // [Q][kmax] issue boundary of a swap-in, by its place in jobs_hi
    uint32_t per_run_lists;            // 1: run q has its own list (row q of list / jobs / m), 0: all share row 0
    uint64_t bpus;
    uint64_t *total_ns, *overhead_ns, *peak_resident;
    uint32_t *forced;
};

// What the machine reads next of each of its three streams.  Its state goes from event to event in
// registers; the entries come from here, RUN_WIN of a stream fetched by the whole wave at a time, so
// that an event waits for LDS and not for the chain jobs -> list -> size, steps in global memory.
struct SimWin {
    uint64_t need[RUN_WIN], rel[RUN_WIN], dt[RUN_WIN];
    uint64_t osize[RUN_WIN], odur[RUN_WIN], okey[RUN_WIN];      // key: step << 32 | variable, the order of the jobs
    uint64_t isize[RUN_WIN], idur[RUN_WIN], ikey[RUN_WIN];      // ikey: the key of the same variable's swap-out
    uint32_t ihi[RUN_WIN], ikb[RUN_WIN];
};

__device__ __forceinline__ void win_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint64_t sim_dur(uint64_t size, uint64_t bpus) { return (size * 1000ull + bpus - 1) / bpus; }

// The next swap-outs or swap-ins of the prefix from jobs[raw..m): returns how many entries the window
// holds (0: none left) and moves raw behind them.
template <bool OUT>
__device__ uint32_t win_fill(const SimArgs &A, const uint32_t *jobs, const uint32_t *list, const uint32_t *kb,
                             uint32_t k, uint32_t m, uint32_t &raw, SimWin &W)
{
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t cnt = 0;
    win_sync();
    while (cnt == 0 && raw < m) {
        uint32_t pos[RUN_BATCH], v[RUN_BATCH];
#pragma unroll
        for (int j = 0; j < RUN_BATCH; ++j) {
            const uint32_t r = raw + j * WAVE + lane;
            pos[j] = r < m ? jobs[r] : SIM_NONE;
        }
#pragma unroll
        for (int j = 0; j < RUN_BATCH; ++j) v[j] = pos[j] < k ? min(list[pos[j]], A.n - 1) : 0;
#pragma unroll
        for (int j = 0; j < RUN_BATCH; ++j) {
            const bool on = pos[j] < k;
            const uint64_t who = ballot(on);
            if (on) {
                const uint32_t at = cnt + (uint32_t)__popcll(who & below);
                const uint64_t sz = A.size[v[j]], key = (uint64_t)A.step_lo[v[j]] << 32 | v[j];
                if (OUT) {
                    W.osize[at] = sz; W.odur[at] = sim_dur(sz, A.bpus); W.okey[at] = key;
                } else {
                    W.isize[at] = sz; W.idur[at] = sim_dur(sz, A.bpus); W.ikey[at] = key;
                    W.ihi[at] = A.step_hi[v[j]] - A.hi_minus;
                    W.ikb[at] = kb[raw + j * WAVE + lane];
                }
            }
            cnt += (uint32_t)__popcll(who);
        }
        raw = m - raw > RUN_WIN ? raw + RUN_WIN : m;
    }
    win_sync();
    return cnt;
}

// last step boundary t <= th with C[t] <= start (0 if none), and not before lo + 1
__device__ __forceinline__ uint32_t sim_boundary(const uint64_t *C, uint32_t lo, uint32_t th, long long start)
{
    uint32_t l0 = 0, h0 = th;
    while (l0 < h0) { const uint32_t mid = (l0 + h0 + 1) >> 1; if ((long long)C[mid] <= start) l0 = mid; else h0 = mid - 1; }
    return max(l0, lo + 1);
}

// The plan's swap-in starts of one run, from the last access backwards, which are a scan (stream_scan.h): RUN_THREADS
// jobs a round.  Each gives the step boundary at which the swap-in is issued.
__global__ __launch_bounds__(RUN_THREADS) void k_sim_starts(SimArgs A)
{
    __shared__ Fn wtmp[RUN_WAVES];
    const uint32_t q = blockIdx.x, tid = threadIdx.x;
    const size_t row = A.per_run_lists ? (size_t)q * A.n : 0;
    const uint32_t *list = A.list + row, *jobs_hi = A.jobs_hi + row;
    const uint32_t k = A.prefix[q], m = A.m[A.per_run_lists ? q : 0];
    uint32_t *kb = A.kb + (size_t)q * A.kmax;

    // whether the run fits the narrow machine, and with which granule
    __shared__ uint32_t s_shift;
    const uint64_t extent = A.peak_resident[0], bits = A.total_ns[0];      // sim_extent left them there
    if (tid == 0) s_shift = bits ? (uint32_t)__ffsll((unsigned long long)bits) - 1 : 0;
    bool wide = A.T >= SIM_NEVER;
    for (uint32_t t = tid; t < A.T; t += RUN_THREADS) wide |= A.C[t + 1] - A.C[t] - 1 >= SIM_NEVER;
    uint64_t sizes = 0;                                    // bitwise or of this thread's
    uint64_t served = 0;                                   // this thread's durations, up to 2^61
    Fn carry{0, SC_POS};
    for (uint32_t base = 0; base < m; base += RUN_THREADS) {
        const uint32_t back = base + tid, jj = m - 1 - back;
        Fn f{0, SC_POS};
        uint32_t lo = 0, th = 0;
        bool on = false;
        if (back < m) {
            const uint32_t pos = jobs_hi[jj];
            if (pos < k) {
                const uint32_t v = min(list[pos], A.n - 1);
                const long long d = (long long)sim_dur(A.size[v], A.bpus);
                served = umin64(served + umin64((uint64_t)d, 1ull << 60), 1ull << 61);
                wide |= (uint64_t)d - 1 >= SIM_NEVER;
                sizes |= A.size[v];
                on = true;
                lo = A.step_lo[v];
                th = A.step_hi[v] - A.hi_minus;
                f = Fn{d, (long long)A.C[th] - d};
            }
        }
        const Fn g = block_scan_fn<false, RUN_WAVES>(f, carry, wtmp);
        if (on) kb[jj] = sim_boundary(A.C, lo, th, g.b);
    }
    if (sizes) atomicMin(&s_shift, (uint32_t)__ffsll((unsigned long long)sizes) - 1);
    wide = __syncthreads_or(wide) != 0;
    // (all workgroups have read what the first run's outputs held before: they are written by the next launch)
    if (tid == 0) A.forced[q] = wide || (extent >> s_shift) >= SIM_NEVER ? SIM_WIDE : s_shift;
    // The scan adds durations up.  Where they may not fit (transfers of years: 52 days in one thread's share), starts
    // wrap around, and where they do depends on the order: one job after the other, then.
    if (__syncthreads_or(served >= 1ull << 52) && tid == 0) {
        long long next = SC_POS;
        for (uint32_t jj = m; jj-- > 0;) {
            const uint32_t pos = jobs_hi[jj];
            if (pos >= k) continue;
            const uint32_t v = min(list[pos], A.n - 1), th = A.step_hi[v] - A.hi_minus;
            const long long due = (long long)A.C[th];
            next = (long long)((uint64_t)(due < next ? due : next) - sim_dur(A.size[v], A.bpus));
            kb[jj] = sim_boundary(A.C, A.step_lo[v], th, next);
        }
    }
}

// The machine of one run, by one wave, all lanes with the same state.  Transfers are served in order, so "the swap-out
// of this variable is done" is a comparison of its key with that of the last one done, and "the swap-in is issued" one of
// the largest issue boundary up to it.  Here with 64 bits throughout, for what sim_run_narrow does not hold.
__device__ void sim_run_wide(const SimArgs &A, SimWin &W)
{
    const uint32_t q = blockIdx.x, tid = threadIdx.x;
    const size_t row = A.per_run_lists ? (size_t)q * A.n : 0;
    const uint32_t *list = A.list + row, *jobs_lo = A.jobs_lo + row, *jobs_hi = A.jobs_hi + row;
    const uint32_t k = A.prefix[q], m = A.m[A.per_run_lists ? q : 0], T = A.T;
    const uint64_t limit = A.limits[q];
    const uint32_t *kb = A.kb + (size_t)q * A.kmax;

    uint64_t now = 0, R = 0, peak = 0;
    uint32_t t = 0, nforced = 0;                           // t is also the last step boundary reached
    bool step_run = false, out_run = false, in_run = false;
    uint64_t step_end = 0, out_end = 0, in_end = 0;
    // the current entry of each stream; `_at` inside the window of `_cnt` entries, `_raw` what follows it
    uint64_t need = 0, rel = 0, dt = 0, osize = 0, odur = 0, okey = 0, isize = 0, idur = 0, ikey = 0;
    uint64_t done = 0;                                     // key of the last swap-out done, plus one
    uint32_t ihi = 0, issue = 0;
    uint32_t o_at = 0, o_cnt = 0, o_raw = 0, i_at = 0, i_cnt = 0, i_raw = 0;
    bool o_any, i_any;
    auto step_load = [&]() {
        if (t >= T) return;
        if (t % RUN_WIN == 0) {
            win_sync();
#pragma unroll
            for (int j = 0; j < RUN_BATCH; ++j) {
                const uint32_t e = j * WAVE + tid;
                if (e < T - t) { W.need[e] = A.need[t + e]; W.rel[e] = A.rel[t + e]; W.dt[e] = A.C[t + e + 1] - A.C[t + e]; }
            }
            win_sync();
        }
        const uint32_t e = t % RUN_WIN;
        need = W.need[e]; rel = W.rel[e]; dt = W.dt[e];
    };
    auto out_load = [&]() {
        if (o_at == o_cnt) { o_cnt = win_fill<true>(A, jobs_lo, list, kb, k, m, o_raw, W); o_at = 0; }
        o_any = o_cnt != 0;
        if (o_any) { osize = W.osize[o_at]; odur = W.odur[o_at]; okey = W.okey[o_at]; ++o_at; }
    };
    auto in_load = [&]() {
        if (i_at == i_cnt) { i_cnt = win_fill<false>(A, jobs_hi, list, kb, k, m, i_raw, W); i_at = 0; }
        i_any = i_cnt != 0;
        if (i_any) {
            isize = W.isize[i_at]; idur = W.idur[i_at]; ikey = W.ikey[i_at]; ihi = W.ihi[i_at];
            issue = max(issue, W.ikb[i_at]);
            ++i_at;
        }
    };
    step_load();
    out_load();
    in_load();
    for (;;) {
        // ends at this instant
        if (step_run && step_end == now) {
            step_run = false;
            R -= rel;
            ++t;
            step_load();
        }
        if (out_run && out_end == now) {
            out_run = false;
            R -= osize;
            done = okey + 1;
            out_load();
        }
        if (in_run && in_end == now) {
            in_run = false;
            in_load();
        }
        if (t == T && !step_run) break;
        // starts: swap-out, step, swap-in
        if (!out_run && o_any && (uint32_t)(okey >> 32) < t) {
            out_run = true;
            out_end = now + odur;
        }
        bool step_blocked = false, in_blocked = false;
        if (!step_run && t < T && (!i_any || ihi > t)) {
            if (need == 0 || R + need <= limit) {
                step_run = true; R += need; step_end = now + dt;
                peak = umax64(peak, R);
            } else step_blocked = true;
        }
        if (!in_run && i_any && issue <= t && ikey < done) {
            if (R + isize <= limit) {
                in_run = true; R += isize; in_end = now + idur;
                peak = umax64(peak, R);
            } else in_blocked = true;
        }
        if (!step_run && !out_run && !in_run) {
            // nothing will change by itself: the limit is overridden once
            ++nforced;
            if (step_blocked) {
                step_run = true; R += need; step_end = now + dt;
            } else if (in_blocked) {
                in_run = true; R += isize; in_end = now + idur;
            } else {
                nforced = SIM_NONE;           // an inconsistent trace; leave rather than spin
                break;
            }
            peak = umax64(peak, R);
        }
        uint64_t nx = U64_MAX;
        if (step_run) nx = umin64(nx, step_end);
        if (out_run) nx = umin64(nx, out_end);
        if (in_run) nx = umin64(nx, in_end);
        now = nx;
    }
    if (tid == 0) {
        A.total_ns[q] = now;
        A.overhead_ns[q] = now - A.C[T];
        A.peak_resident[q] = peak;
        A.forced[q] = nforced;
    }
}

// The same machine in scalar registers, sizes in granules and times in nanoseconds in 31 bits.  One event after the other
// is a chain that its instructions and branches make long, not memory: 4 cycles an instruction, 17 to 24 a branch, 20 from
// the vector to the scalar unit.  So an event is one straight line of scalar instructions.  The entries to come are in
// vector registers, one per lane, 64 of a stream at a time by way of the window in LDS, the first of them in the highest
// lane: the lane counts down and is negative when the chunk is used up.  Every event reads the current entry of each stream
// from its lane whether it has changed or not, and conditions are signs, so that several are one `and`.  An actor's word
// is its remaining time less one, and -1 when it does nothing: max(word - elapsed, -1) is the next word in all cases.
// The limit is kept as what it leaves.  A stretch in which only one of the two streams can be at work leaves the other one
// out: some 125 ns an event there, 200 where both are.  14 000 steps and 11 000 transfers, every one blocked, with
// both at work in half of the events: 6.3 ms (7.4 ms when every event looked at both, 14.8 with 64-bit state and a branch a
// question); 348 steps and 257 transfers 0.145 ms (0.18, 0.36).  8000 steps and 4000 transfers without a limit: nested idle
// gaps 2.2 ms (2.9), gaps of a few steps, whose transfers take turns, 2.85 (2.87).
struct NarrowWin {
    uint32_t need[RUN_WIN], rel[RUN_WIN], dt[RUN_WIN];               // dt, like all times here, less one
    uint32_t osize[RUN_WIN], odur[RUN_WIN], olo[RUN_WIN], oplace[RUN_WIN];
    uint32_t isize[RUN_WIN], idur[RUN_WIN], iplace[RUN_WIN], ihi[RUN_WIN], ikb[RUN_WIN];
};

__device__ __forceinline__ bool negative(uint32_t x) { return (int32_t)x < 0; }
// (of two and more of these the compiler makes one in the vector unit, and a detour)
__device__ __forceinline__ uint32_t s_min(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("s_min_u32 %0, %1, %2" : "=s"(r) : "s"(a), "s"(b) : "scc");
    return r;
}

// as win_fill
template <bool OUT>
__device__ uint32_t narrow_fill(const SimArgs &A, const uint32_t *jobs, const uint32_t *list, const uint32_t *place_lo,
                                const uint32_t *kb, uint32_t k, uint32_t m, uint32_t shift, uint32_t &raw, NarrowWin &W)
{
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    const uint64_t below = (1ull << lane) - 1ull;
    uint32_t cnt = 0;
    win_sync();
    while (cnt == 0 && raw < m) {
        uint32_t pos[RUN_BATCH], v[RUN_BATCH];
#pragma unroll
        for (int j = 0; j < RUN_BATCH; ++j) {
            const uint32_t r = raw + j * WAVE + lane;
            pos[j] = r < m ? jobs[r] : SIM_NONE;
        }
#pragma unroll
        for (int j = 0; j < RUN_BATCH; ++j) v[j] = pos[j] < k ? min(list[pos[j]], A.n - 1) : 0;
#pragma unroll
        for (int j = 0; j < RUN_BATCH; ++j) {
            const bool on = pos[j] < k;
            const uint64_t who = ballot(on);
            if (on) {
                const uint32_t at = cnt + (uint32_t)__popcll(who & below);
                const uint64_t sz = A.size[v[j]];
                const uint32_t dur = (uint32_t)sim_dur(sz, A.bpus) - 1u;
                if (OUT) {
                    W.osize[at] = (uint32_t)(sz >> shift); W.odur[at] = dur; W.olo[at] = A.step_lo[v[j]];
                    W.oplace[at] = raw + j * WAVE + lane;
                } else {
                    W.isize[at] = (uint32_t)(sz >> shift); W.idur[at] = dur; W.iplace[at] = place_lo[pos[j]];
                    W.ihi[at] = A.step_hi[v[j]] - A.hi_minus;
                    W.ikb[at] = kb[raw + j * WAVE + lane];
                }
            }
            cnt += (uint32_t)__popcll(who);
        }
        raw = m - raw > RUN_WIN ? raw + RUN_WIN : m;
    }
    win_sync();
    return cnt;
}

__device__ void sim_run_narrow(const SimArgs &A, uint32_t shift, NarrowWin &W)
{
    const uint32_t q = blockIdx.x, lane = threadIdx.x;
    const size_t row = A.per_run_lists ? (size_t)q * A.n : 0;
    const uint32_t *list = A.list + row, *jobs_lo = A.jobs_lo + row, *jobs_hi = A.jobs_hi + row, *place_lo = A.place_lo + row;
    const uint32_t *kb = A.kb + (size_t)q * A.kmax;
    const uint32_t T = A.T;
    const uint32_t k = (uint32_t)__builtin_amdgcn_readfirstlane((int)A.prefix[q]);
    const uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)A.m[A.per_run_lists ? q : 0]);
    // all that is resident is below SIM_NEVER, so a limit beyond that is none
    const uint32_t limit = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)umin64(A.limits[q] >> shift, SIM_NEVER));

    uint32_t c_need = 0, c_rel = 0, c_dt = 0;                             // a step's time shares its word with the sign "needs nothing"
    uint32_t c_osize = 0, c_odur = 0, c_olo = 0, c_oplace = 0;
    uint32_t c_isize = 0, c_idur = 0, c_iplace = 0, c_ihi = 0, c_issue = 0;
    // nothing has happened: everything is idle before its first entry
    uint32_t t = 0, te = ~0u, oe = ~0u, ie = ~0u;                         // the step; the lanes of the current entries
    uint32_t o_at = 0, o_cnt = 0, o_raw = 0, i_at = 0, i_cnt = 0, i_raw = 0, issued = 0, nforced = 0;
    uint32_t step = ~0u, out = ~0u, in = ~0u;                             // the actors' words
    uint64_t now = 0;
    uint32_t left = limit, least = limit;                                 // what the limit leaves; its smallest after a start
    do {
        if (__builtin_expect(negative(te | oe | ie), 0)) {
            if (negative(te)) {
                if (t % RUN_WIN == 0) {
                    win_sync();
#pragma unroll
                    for (int j = 0; j < RUN_BATCH; ++j) {
                        const uint32_t e = j * WAVE + lane;
                        if (e >= T - t) continue;
                        const uint64_t need = A.need[t + e];
                        W.need[e] = (uint32_t)(need >> shift);
                        W.rel[e] = (uint32_t)(A.rel[t + e] >> shift);
                        W.dt[e] = ((uint32_t)(A.C[t + e + 1] - A.C[t + e]) - 1u) | (need ? 0u : 1u << 31);
                    }
                    win_sync();
                }
                const uint32_t have = min(T - t, (uint32_t)WAVE), e = t % RUN_WIN + (have - 1 - min(lane, have - 1));
                c_need = W.need[e]; c_rel = W.rel[e]; c_dt = W.dt[e];
                te = have - 1;
            }
            // entries that are not there: a swap-out after all steps, a swap-in that no step waits for and that is never
            // issued; their words stay idle
            if (negative(oe)) {
                if (o_at == o_cnt) { o_cnt = narrow_fill<true>(A, jobs_lo, list, place_lo, kb, k, m, shift, o_raw, W); o_at = 0; }
                const uint32_t have = min(o_cnt - o_at, (uint32_t)WAVE), e = lane < have ? o_at + have - 1 - lane : 0;
                c_osize = W.osize[e]; c_odur = W.odur[e];
                c_olo = lane < have ? W.olo[e] : SIM_NEVER;
                c_oplace = lane < have ? W.oplace[e] : SIM_NEVER;
                oe = have ? have - 1 : 0;
                o_at += have;
            }
            if (negative(ie)) {
                if (i_at == i_cnt) { i_cnt = narrow_fill<false>(A, jobs_hi, list, place_lo, kb, k, m, shift, i_raw, W); i_at = 0; }
                const uint32_t have = min(i_cnt - i_at, (uint32_t)WAVE), e = lane < have ? i_at + have - 1 - lane : 0;
                c_isize = W.isize[e]; c_idur = W.idur[e]; c_iplace = W.iplace[e];
                c_ihi = lane < have ? W.ihi[e] : SIM_NEVER;
                // a swap-in is issued when the largest boundary up to it is reached
                const uint32_t upto = max(wave_scan_max_u32(lane < have ? W.ikb[i_at + lane] : 0u), issued);
                issued = read_lane(upto, WAVE - 1);
                const uint32_t mine = (uint32_t)__shfl((int)upto, (int)(lane < have ? have - 1 - lane : 0), WAVE);
                c_issue = lane < have ? mine : SIM_NEVER;
                ie = have ? have - 1 : 0;
                i_at += have;
            }
        }
        // One event.  OUT, IN: whether a swap-out, a swap-in can be under way or start; what is not is not looked at.
        auto event = [&](auto with_out, auto with_in) {
            constexpr bool OUT = decltype(with_out)::value, IN = decltype(with_in)::value;
            uint32_t need = read_lane(c_need, (int)te), rel = read_lane(c_rel, (int)te), dt = read_lane(c_dt, (int)te);
            uint32_t olo = 0, odur = 0, osize = 0, oplace = 0, ihi = 0, issue = 0, isize = 0, iplace = 0, idur = 0;
            if constexpr (OUT) { olo = read_lane(c_olo, (int)oe); odur = read_lane(c_odur, (int)oe); osize = read_lane(c_osize, (int)oe); }
            if constexpr (IN) {
                ihi = read_lane(c_ihi, (int)ie); issue = read_lane(c_issue, (int)ie);
                isize = read_lane(c_isize, (int)ie); idur = read_lane(c_idur, (int)ie);
            }
            if constexpr (OUT && IN) { oplace = read_lane(c_oplace, (int)oe); iplace = read_lane(c_iplace, (int)ie); }
            // all of them before the first scalar instruction: one that follows a read of a lane waits 20 cycles, and they
            // would alternate
            if constexpr (OUT && IN)
                asm volatile("" : "+s"(need), "+s"(rel), "+s"(dt), "+s"(olo), "+s"(odur), "+s"(osize), "+s"(oplace), "+s"(ihi),
                             "+s"(issue), "+s"(isize), "+s"(iplace), "+s"(idur));
            else if constexpr (OUT)
                asm volatile("" : "+s"(need), "+s"(rel), "+s"(dt), "+s"(olo), "+s"(odur), "+s"(osize));
            else
                asm volatile("" : "+s"(need), "+s"(rel), "+s"(dt), "+s"(ihi), "+s"(issue), "+s"(isize), "+s"(idur));
            // starts: swap-out, step, swap-in (its variable is out if the current swap-out is one behind it)
            if constexpr (OUT) out = negative(out & (olo - t)) ? odur : out;
            uint32_t step_may = step;
            if constexpr (IN) step_may &= t - ihi;
            const uint32_t after_step = left - need, step_go = step_may & (dt | ~after_step);
            step = negative(step_go) ? dt & SIM_NEVER : step;
            left = negative(step_go) ? after_step : left;
            uint32_t in_may = 0, after_in = 0, soon = step;
            if constexpr (OUT) soon = s_min(soon, out);
            if constexpr (IN) {
                in_may = in & ~(t - issue);
                if constexpr (OUT) in_may &= iplace - oplace;
                after_in = left - isize;
                const uint32_t in_go = in_may & ~after_in;
                in = negative(in_go) ? idur : in;
                left = negative(in_go) ? after_in : left;
                soon = s_min(soon, in);
            }
            if (__builtin_expect(negative(soon), 0)) {
                // nothing will change by itself: the limit is overridden once
                if (negative(step_may)) { soon = step = dt & SIM_NEVER; left = after_step; }
                else if (negative(in_may)) { soon = in = idur; left = after_in; }
                else { nforced = SIM_NONE - 1; t = T; te = ~0u; }          // an inconsistent trace; leave rather than spin
                ++nforced;
            }
            least = (uint32_t)min((int32_t)left, (int32_t)least);
            const uint32_t nx = soon + 1u;
            now += nx;
            // ends at the next instant
            const uint32_t step_next = (uint32_t)max((int32_t)(step - nx), -1);
            const uint32_t step_ends = (uint32_t)((int32_t)(step_next & ~step) >> 31);
            left += rel & step_ends;
            if constexpr (OUT) {
                const uint32_t out_next = (uint32_t)max((int32_t)(out - nx), -1);
                const uint32_t out_ends = (uint32_t)((int32_t)(out_next & ~out) >> 31);
                left += osize & out_ends;
                oe += out_ends;
                out = out_next;
            }
            if constexpr (IN) {
                const uint32_t in_next = (uint32_t)max((int32_t)(in - nx), -1);
                const uint32_t in_ends = (uint32_t)((int32_t)(in_next & ~in) >> 31);
                ie += in_ends;
                in = in_next;
            }
            t -= step_ends;
            te += step_ends;
            step = step_next;
        };
        // Two thirds of the instructions do where only one stream is at work.  No swap-in can start before the next one is
        // issued, or before the swap-out of its variable is done, which is late in an iteration: the first one needed back
        // was the last one to leave.
        const uint32_t next_place = read_lane(c_iplace, (int)ie);
        uint32_t quiet = min(read_lane(c_ihi, (int)ie), T), oe_last = 0;
        if (read_lane(c_oplace, (int)oe) <= next_place) oe_last = (uint32_t)__ffsll((unsigned long long)ballot(c_oplace <= next_place)) - 1;
        else quiet = min(quiet, read_lane(c_issue, (int)ie));
        if (negative(in) && (int32_t)(t - quiet) < 0) {
            do event(std::true_type{}, std::false_type{});
            while (!negative(te | (oe - oe_last) | (quiet - 1u - t)));
        } else if (negative(out) && read_lane(c_olo, (int)oe) == SIM_NEVER) {
            do event(std::false_type{}, std::true_type{});
            while (!negative(te | ie));
        } else {
            // (some events before the question is asked again; after the last step there is no next one)
            uint32_t more = 64;
            do event(std::true_type{}, std::true_type{});
            while (!negative(te | oe | ie | (--more - 1u)));
        }
    } while (t != T);
    if (lane == 0) {
        A.total_ns[q] = now;
        A.overhead_ns[q] = now - A.C[T];
        A.peak_resident[q] = (uint64_t)(limit - least) << shift;
        A.forced[q] = nforced;
    }
}

__global__ __launch_bounds__(WAVE) void k_sim_run(SimArgs A)
{
    __shared__ union {
        SimWin wide;
        NarrowWin narrow;
    } W;
    const uint32_t shift = (uint32_t)__builtin_amdgcn_readfirstlane((int)A.forced[blockIdx.x]);     // (of the launch before)
    if (shift >= SIM_WIDE) sim_run_wide(A, W.wide);
    else sim_run_narrow(A, shift, W.narrow);
}

hipError_t launch_simulate_swaps(uint32_t n, uint32_t T, uint32_t Q, uint32_t kmax, uint32_t count,
                                 const uint32_t *count_dev, const uint64_t *size,
                                 const uint32_t *alloc, const uint32_t *free_, const uint32_t *step_lo,
                                 const uint32_t *step_hi, uint32_t hi_minus, const uint64_t *C, uint64_t *need,
                                 uint64_t *rel, const uint32_t *list, const uint32_t *perm_lo,
                                 const uint32_t *perm_hi, const uint32_t *posmap, uint32_t *jobs_lo,
                                 uint32_t *jobs_hi, uint32_t *m, const uint32_t *prefix, const uint64_t *limits,
                                 uint32_t *kb, uint32_t *place_lo, uint64_t bpus, uint64_t *total_ns,
                                 uint64_t *overhead_ns, uint64_t *peak_resident, uint32_t *forced, hipStream_t st,
                                 uint32_t n_lists, const uint32_t *n_listed)
{
    // n_listed given: run q replays row q of `list` (n_lists rows of n entries, *n_listed valid entries
    // each, the same variables in all rows and in perm); the n_lists position maps are filled here
    if (n_listed)
        hipLaunchKernelGGL(k_sim_mark_rows, dim3((n + 255) / 256, n_lists), dim3(256), 0, st, n, list, n_listed,
                           const_cast<uint32_t *>(posmap));
    hipLaunchKernelGGL(k_sim_steps, dim3((n + 255) / 256), dim3(256), 0, st, n, size, alloc, free_,
                       (unsigned long long *)need, (unsigned long long *)rel);
    hipLaunchKernelGGL(k_sim_jobs, dim3(n_lists, 3), dim3(SIM_THREADS), 0, st, n, count, count_dev, perm_lo, perm_hi, posmap, step_lo,
                       step_hi, hi_minus, jobs_lo, jobs_hi, place_lo, m, T, (const unsigned long long *)need,
                       (const unsigned long long *)rel, peak_resident, total_ns);
    SimArgs A{n, T, Q, kmax, size, step_lo, step_hi, hi_minus, C, (const unsigned long long *)need,
              (const unsigned long long *)rel, list, jobs_lo, jobs_hi, place_lo, m, prefix, limits, kb,
              n_listed ? 1u : 0u, bpus,
              total_ns, overhead_ns, peak_resident, forced};
    hipLaunchKernelGGL(k_sim_starts, dim3(Q), dim3(RUN_THREADS), 0, st, A);
    hipLaunchKernelGGL(k_sim_run, dim3(Q), dim3(WAVE), 0, st, A);
    return hipGetLastError();
}

}  // namespace lap
