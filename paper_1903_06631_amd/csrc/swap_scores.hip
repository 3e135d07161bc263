// Swap-candidate filter and priority scores (Section IV-A, IV-B).
//
// Prefix arrays over the T steps are built first, a workgroup each:
//   C[t]  wall-clock start of step t (prefix sum of step_ns), C[T] = total
//   S[t]  sum of load over steps < t (area under the load curve)
//   PM[t] max load over steps < t,   SM[t] max load over steps >= t
// A sparse table over load answers range-maximum queries in O(1).  Then one
// thread per variable evaluates its scores with two binary searches over C.
#include "lap_dev.h"
#include "lap_kernels.h"

namespace lap {

constexpr int PFX_THREADS = 1024, PFX_WAVES = PFX_THREADS / WAVE;
constexpr int PFX_ITEMS = 4;             // steps per thread and round of a scan
constexpr int PFX_SCANS = 4;             // workgroups 0..3: C, S, PM (with the peak), SM
constexpr uint32_t TAB_STEPS = PFX_THREADS;   // steps of a table workgroup, one per thread
constexpr uint32_t TAB_LOW = 10;         // levels that two such stretches of the load decide: 2^10 = TAB_STEPS
constexpr uint32_t TAB_HIGH = 4;         // further levels per launch of k_table_high

struct PfxScan {
    uint64_t wtot[2][PFX_WAVES];         // wave totals, alternating: one barrier per round
    uint64_t best[PFX_WAVES];
    uint32_t first[PFX_WAVES];
};

template <bool MAX> __device__ __forceinline__ uint64_t pfx_join(uint64_t a, uint64_t b)
{
    return MAX ? umax64(a, b) : a + b;
}

// Inclusive scan (sum or maximum, identity 0) of get(0..T-1); put(t, value) receives the results.
template <bool MAX, class Get, class Put>
__device__ __forceinline__ void scan_steps(uint32_t T, PfxScan &s, Get get, Put put)
{
    const uint32_t tid = threadIdx.x, l = tid & (WAVE - 1), w = tid / WAVE;
    uint64_t carry = 0;
    int buf = 0;
    for (uint64_t base = 0; base < T; base += PFX_THREADS * PFX_ITEMS, buf ^= 1) {
        const uint64_t t0 = base + tid * PFX_ITEMS;
        uint64_t v[PFX_ITEMS];
#pragma unroll
        for (int j = 0; j < PFX_ITEMS; ++j) v[j] = t0 + j < T ? get((uint32_t)(t0 + j)) : 0;
#pragma unroll
        for (int j = 1; j < PFX_ITEMS; ++j) v[j] = pfx_join<MAX>(v[j - 1], v[j]);
        const uint64_t incl = MAX ? wave_scan_max(v[PFX_ITEMS - 1]) : wave_scan_add(v[PFX_ITEMS - 1]);
        if (l == WAVE - 1) s.wtot[buf][w] = incl;
        __syncthreads();
        uint64_t pre = lane_shift_up64(incl, 0), tot = carry;
#pragma unroll
        for (uint32_t k = 0; k < PFX_WAVES; ++k) {
            if (k == w) pre = pfx_join<MAX>(pre, tot);
            tot = pfx_join<MAX>(tot, s.wtot[buf][k]);
        }
        carry = tot;
#pragma unroll
        for (int j = 0; j < PFX_ITEMS; ++j)
            if (t0 + j < T) put((uint32_t)(t0 + j), pfx_join<MAX>(pre, v[j]));
    }
}

// The four scans, and levels 0 .. min(10, levels - 1) of the sparse table (level k of it:
// M[k][t] = max load[t .. t + 2^k)), side by side.  What bounds it is latency: a few KB of curve,
// read by launches that wait for each other.  One workgroup that scanned everything in turn and one
// launch per level took 11 launches at 580 steps and 15 at 14 000; the scans and the stretches of
// the table depend on nothing but the load, so each has a workgroup.  A table workgroup holds its
// 1024 steps and the 1024 after them in LDS, which is what levels up to 10 of its steps cover.
__global__ __launch_bounds__(PFX_THREADS) void k_swap_prefix(uint32_t T, const uint64_t *__restrict__ load,
                                                             const uint64_t *__restrict__ step_ns,
                                                             uint64_t *__restrict__ C, uint64_t *__restrict__ S,
                                                             uint64_t *__restrict__ PM, uint64_t *__restrict__ SM,
                                                             uint64_t *__restrict__ peak_out,
                                                             uint32_t *__restrict__ tpeak_out,
                                                             uint64_t *__restrict__ table, uint32_t levels)
{
    __shared__ union {
        PfxScan scan;
        uint64_t row[2][2 * TAB_STEPS];
    } s;
    const uint32_t tid = threadIdx.x, l = tid & (WAVE - 1), w = tid / WAVE;
    if (blockIdx.x >= PFX_SCANS) {
        const uint32_t t = (blockIdx.x - PFX_SCANS) * TAB_STEPS + tid;
        const bool in = t < T;
        // a: this thread's step, b: the one TAB_STEPS later; steps past the end count as 0
        uint64_t a = in ? load[t] : 0, b = (uint64_t)t + TAB_STEPS < T ? load[t + TAB_STEPS] : 0;
        if (in) table[t] = a;
        for (uint32_t k = 1; k < levels && k <= TAB_LOW; ++k) {
            uint64_t *row = s.row[k & 1];
            row[tid] = a;
            row[tid + TAB_STEPS] = b;
            __syncthreads();
            const uint32_t half = 1u << (k - 1), far = tid + TAB_STEPS + half;
            a = umax64(a, row[tid + half]);
            // the last entries of the second stretch lack the values past it: level k is right up to
            // entry 2048 - 2^k, the first 1024 entries need no more
            if (far < 2 * TAB_STEPS) b = umax64(b, row[far]);
            if (in) table[(size_t)k * T + t] = a;
        }
        return;
    }
    if (blockIdx.x == 0) {
        if (tid == 0) C[0] = 0;
        scan_steps<false>(T, s.scan, [=](uint32_t t) { return step_ns ? step_ns[t] : 1000000ull; },
                          [=](uint32_t t, uint64_t v) { C[t + 1] = v; });
    } else if (blockIdx.x == 1) {
        if (tid == 0) S[0] = 0;
        scan_steps<false>(T, s.scan, [=](uint32_t t) { return load[t]; },
                          [=](uint32_t t, uint64_t v) { S[t + 1] = v; });
    } else if (blockIdx.x == 2) {
        if (tid == 0) PM[0] = 0;
        // the peak and the earliest step that attains it: a thread meets its steps in ascending order
        uint64_t best = 0;
        uint32_t first = 0xFFFFFFFFu;
        scan_steps<true>(T, s.scan,
                         [&](uint32_t t) {
                             const uint64_t v = load[t];
                             if (v > best || first == 0xFFFFFFFFu) { best = v; first = t; }
                             return v;
                         },
                         [=](uint32_t t, uint64_t v) { PM[t + 1] = v; });
        const uint64_t wave_best = wave_reduce_max(best);
        if (best != wave_best) first = 0xFFFFFFFFu;
#pragma unroll
        for (int m = WAVE / 2; m > 0; m >>= 1) first = min(first, (uint32_t)__shfl_xor(first, m, WAVE));
        if (l == 0) { s.scan.best[w] = wave_best; s.scan.first[w] = first; }
        __syncthreads();
        if (tid == 0) {
            uint64_t pk = 0;
            uint32_t at = 0xFFFFFFFFu;
            for (int k = 0; k < PFX_WAVES; ++k) {
                const uint64_t x = s.scan.best[k];
                if (x > pk) { pk = x; at = s.scan.first[k]; }
                else if (x == pk) at = min(at, s.scan.first[k]);
            }
            *peak_out = pk; *tpeak_out = at;
        }
    } else {
        if (tid == 0) SM[T] = 0;
        scan_steps<true>(T, s.scan, [=](uint32_t t) { return load[T - 1 - t]; },
                         [=](uint32_t t, uint64_t v) { SM[T - 1 - t] = v; });
    }
}

// levels k0 + 1 .. k0 + TAB_HIGH (below `levels`) of the sparse table from its level k0: a level-k entry
// covers 2^(k - k0) entries of level k0, 2^k0 steps apart
__global__ __launch_bounds__(256) void k_table_high(uint32_t T, uint64_t *__restrict__ table, uint32_t k0,
                                                    uint32_t levels)
{
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    const uint64_t *src = table + (size_t)k0 * T;
    uint64_t m = src[t];
    for (uint32_t k = k0 + 1; k < levels && k <= k0 + TAB_HIGH; ++k) {
        const uint32_t hi = 1u << (k - k0);
#pragma unroll 8
        for (uint32_t j = hi / 2; j < hi; ++j) {
            const uint64_t at = t + ((uint64_t)j << k0);
            if (at < T) m = umax64(m, src[at]);
        }
        table[(size_t)k * T + t] = m;
    }
}

__global__ __launch_bounds__(256) void k_score(uint32_t n, uint32_t T, const uint64_t *__restrict__ size,
                                               const uint32_t *__restrict__ alloc, const uint32_t *__restrict__ free_,
                                               const uint32_t *__restrict__ gap_lo, const uint32_t *__restrict__ gap_hi,
                                               uint64_t bpus, uint64_t min_bytes,
                                               const uint64_t *__restrict__ load, const uint64_t *__restrict__ C,
                                               const uint64_t *__restrict__ S, const uint64_t *__restrict__ PM,
                                               const uint64_t *__restrict__ SM, const uint64_t *__restrict__ table,
                                               const uint64_t *__restrict__ peak_p, const uint32_t *__restrict__ tpeak_p,
                                               uint8_t *__restrict__ cand, int64_t *__restrict__ doa,
                                               double *__restrict__ aoa, uint64_t *__restrict__ wdoa,
                                               uint64_t *__restrict__ cut, uint32_t *__restrict__ win_lo,
                                               uint32_t *__restrict__ win_hi)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t peak = *peak_p;
    const uint32_t t_peak = *tpeak_p;
    const uint64_t s = size[i];
    const uint32_t a = alloc[i], f = free_[i];
    const uint32_t tl = gap_lo ? gap_lo[i] : a;
    const uint32_t th = gap_hi ? gap_hi[i] : f - 1;
    uint8_t c = 0; int64_t d = 0; double ar = 0.0; uint64_t w = 0, pc = 0;
    uint32_t wl = 0, wh = 0;          // whole steps [wl, wh) during which a swapped variable is away
    if (th > tl) {
        c = (s >= min_bytes && a <= t_peak && t_peak < f) ? 1 : 0;
        const uint64_t delta = (s * 1000ull + bpus - 1) / bpus;
        const uint64_t idle_from = C[tl + 1], idle_to = C[th];
        d = (int64_t)(idle_to - idle_from) - 2 * (int64_t)delta;
        ar = d >= 0 ? (double)d * (double)s : (double)d / (double)s;
        w = S[th] - S[tl + 1];
        if (d >= 0) {
            const uint64_t out_done = idle_from + delta, in_start = idle_to - delta;
            // lo = first t with C[t] >= out_done ; hi = last t with C[t] <= in_start   (t in [0, T])
            uint32_t l0 = 0, h0 = T;
            while (l0 < h0) { const uint32_t m = (l0 + h0) >> 1; if (C[m] < out_done) l0 = m + 1; else h0 = m; }
            const uint32_t lo = l0;
            l0 = 0; h0 = T;
            while (l0 < h0) { const uint32_t m = (l0 + h0 + 1) >> 1; if (C[m] <= in_start) l0 = m; else h0 = m - 1; }
            const uint32_t hi = l0;
            if (hi > lo) {
                wl = lo; wh = hi;
                const uint32_t len = hi - lo;
                const uint32_t k = 31 - __clz(len);
                const uint64_t *lvl = table + (size_t)k * T;
                const uint64_t inside = umax64(lvl[lo], lvl[hi - (1u << k)]);
                const uint64_t np = umax64(umax64(PM[lo], SM[hi]), inside - s);
                pc = peak - np;
            }
        }
    }
    cand[i] = c; doa[i] = d; aoa[i] = ar; wdoa[i] = w; cut[i] = pc;
    if (win_lo) { win_lo[i] = wl; win_hi[i] = wh; }
}

// levels = 0: no table
hipError_t launch_swap_prefix(uint32_t T, const uint64_t *load, const uint64_t *step_ns, uint64_t *C, uint64_t *S,
                              uint64_t *PM, uint64_t *SM, uint64_t *peak, uint32_t *t_peak, uint64_t *table,
                              uint32_t levels, hipStream_t st)
{
    const uint32_t stretches = levels ? (uint32_t)(((uint64_t)T + TAB_STEPS - 1) / TAB_STEPS) : 0;
    hipLaunchKernelGGL(k_swap_prefix, dim3(PFX_SCANS + stretches), dim3(PFX_THREADS), 0, st, T, load, step_ns, C, S,
                       PM, SM, peak, t_peak, table, levels);
    for (uint32_t k0 = TAB_LOW; k0 + 1 < levels; k0 += TAB_HIGH)
        hipLaunchKernelGGL(k_table_high, dim3((uint32_t)(((uint64_t)T + 255) / 256)), dim3(256), 0, st, T, table, k0,
                           levels);
    return hipGetLastError();
}

hipError_t launch_score(uint32_t n, uint32_t T, const uint64_t *size, const uint32_t *alloc, const uint32_t *free_,
                        const uint32_t *gap_lo, const uint32_t *gap_hi, uint64_t bpus, uint64_t min_bytes,
                        const uint64_t *load, const uint64_t *C, const uint64_t *S, const uint64_t *PM,
                        const uint64_t *SM, const uint64_t *table, const uint64_t *peak, const uint32_t *t_peak,
                        uint8_t *cand, int64_t *doa, double *aoa, uint64_t *wdoa, uint64_t *cut, uint32_t *win_lo,
                        uint32_t *win_hi, hipStream_t st)
{
    const uint32_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(k_score, dim3(blocks), dim3(256), 0, st, n, T, size, alloc, free_, gap_lo, gap_hi, bpus,
                       min_bytes, load, C, S, PM, SM, table, peak, t_peak, cand, doa, aoa, wdoa, cut, win_lo, win_hi);
    return hipGetLastError();
}

}  // namespace lap
