// Swap schedule (Section IV-E): one stream carries the swap-outs in access order, each as soon
// as its access is over and the stream is free; a second stream carries the swap-ins in the
// order of the next accesses, each as late as its access and the swap-in after it allow.
//
// Both are scans (stream_scan.h).  A stream that serves job j (ready r_j, duration d_j) after it is
// free at x is free again at f_j(x) = max(x, r_j) + d_j = max(x + d_j, r_j + d_j); such functions
// compose as (a, b) pairs -- f(x) = max(x + a, b), (f2 o f1) = (a1 + a2, max(b1 + a2, b2)) -- so the end
// times of all swap-outs are one inclusive scan in (max, +), and the start times of all swap-ins
// the mirror image in (min, -) taken from the last job backwards.  The variables arrive sorted
// by access step: the listed ones (k_rank_steps), or all of them where the list is long, and then
// those that are not listed are the identity of the scan.
#include "lap_dev.h"
#include "lap_kernels.h"
#include "stream_scan.h"

namespace lap {

constexpr int SC_THREADS = 1024;
constexpr int SC_WAVES = SC_THREADS / WAVE;
constexpr uint32_t SC_NONE = 0xFFFFFFFFu;

__global__ __launch_bounds__(256) void k_sched_mark(uint32_t n, uint32_t k, const uint32_t *__restrict__ list,
                                                    uint32_t *__restrict__ posmap)
{
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < k) posmap[min(list[j], n - 1)] = j;
}

// Listed variables in the order of their access steps (ties: by index), by counting: a variable's rank is the number of
// smaller keys.  A workgroup takes 64 of them, one per lane, and its waves count through the keys 64 at a time
// each.  Blocks of one direction: x; direction: y.  An entry of the list whose variable is listed again (posmap names the
// other one) comes last, as no variable.  Bound by the comparisons and three dependent loads a key: 250 of 3000 variables 4.5 us,
// 3600 of 50 000 9 us, 11 000 of them 31 us, both directions (two sorts of all variables by one workgroup each: 56 us, 0.78 ms).
constexpr int RANK_THREADS = 1024, RANK_WAVES = RANK_THREADS / WAVE;

__global__ __launch_bounds__(RANK_THREADS) void k_rank_steps(uint32_t n, uint32_t count, const uint32_t *__restrict__ count_dev,
                                                             const uint32_t *__restrict__ list,
                                                             const uint32_t *__restrict__ posmap,
                                                             const uint32_t *__restrict__ step_lo,
                                                             const uint32_t *__restrict__ step_hi,
                                                             uint32_t *__restrict__ perm_lo, uint32_t *__restrict__ perm_hi)
{
    __shared__ __align__(16) uint64_t s_key[RANK_WAVES][WAVE];
    __shared__ uint32_t s_rank[RANK_WAVES][WAVE];
    const uint32_t lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    const uint32_t *step = blockIdx.y ? step_hi : step_lo;
    uint32_t *perm = blockIdx.y ? perm_hi : perm_lo;
    if (count_dev) count = *count_dev;
    auto key_of = [&](uint32_t j) -> uint64_t {
        if (j >= count) return U64_MAX;
        const uint32_t v = min(list[j], n - 1);
        if (posmap && posmap[v] != j) return (uint64_t)SC_NONE << 32 | j;
        return (uint64_t)step[v] << 32 | v;
    };
    for (uint32_t j0 = blockIdx.x * WAVE; j0 < count; j0 += gridDim.x * WAVE) {
        const uint64_t mine = key_of(j0 + lane);
        uint32_t below = 0;
        for (uint32_t i0 = wave * WAVE; i0 < count; i0 += RANK_THREADS) {
            s_key[wave][lane] = key_of(i0 + lane);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll 16
            for (int q = 0; q < WAVE; ++q) below += s_key[wave][q] < mine ? 1u : 0u;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        s_rank[wave][lane] = below;
        __syncthreads();
        if (wave == 0 && j0 + lane < count) {
            uint32_t r = 0;
#pragma unroll
            for (int w = 0; w < RANK_WAVES; ++w) r += s_rank[w][lane];
            perm[r] = (uint32_t)(mine >> 32) == SC_NONE ? SC_NONE : (uint32_t)mine;
        }
        __syncthreads();
    }
}

struct SchedArgs {
    uint32_t n, T, k, count;
    const uint64_t *size;
    const uint32_t *step_lo, *step_hi;   // access steps: gap_lo or alloc, gap_hi or free (see hi_minus)
    uint32_t hi_minus;                   // 1 when step_hi holds free (the access is step free - 1)
    const uint64_t *C;                   // [T+1] start time of every step
    const uint32_t *perm_lo, *perm_hi;   // [count] listed variables by (step_lo, index) and by (step_hi, index), and others
    const uint32_t *posmap;              // variable -> position in the swap list, or none
    const uint32_t *list;
    uint64_t bpus;
    long long *out_start, *out_end, *in_start, *in_end;
    unsigned long long *diff;            // [T+1] what leaves the load curve (difference array)
    unsigned long long *late;            // [1]
};

__global__ __launch_bounds__(SC_THREADS) void k_sched_streams(SchedArgs A)
{
    __shared__ Fn wtmp[SC_WAVES];
    const uint32_t tid = threadIdx.x, n = A.n, count = A.count;
    // swap-outs, first to last
    Fn carry{0, SC_NEG};
    for (uint32_t base = 0; base < count; base += SC_THREADS) {
        const uint32_t r = base + tid;
        Fn f{0, SC_NEG};
        uint32_t pos = SC_NONE;
        long long d = 0;
        if (r < count) {
            const uint32_t v = A.perm_lo[r];
            if (v != SC_NONE) pos = A.posmap[v];
            if (pos != SC_NONE) {
                d = (long long)((A.size[v] * 1000ull + A.bpus - 1) / A.bpus);
                f = Fn{d, (long long)A.C[A.step_lo[v] + 1] + d};
            }
        }
        const Fn g = block_scan_fn<true, SC_WAVES>(f, carry, wtmp);
        if (pos != SC_NONE) { A.out_end[pos] = g.b; A.out_start[pos] = g.b - d; }
    }
    // swap-ins, last to first
    carry = Fn{0, SC_POS};
    for (uint32_t base = 0; base < count; base += SC_THREADS) {
        const uint32_t rr = base + tid;
        Fn f{0, SC_POS};
        uint32_t pos = SC_NONE;
        long long d = 0;
        if (rr < count) {
            const uint32_t v = A.perm_hi[count - 1 - rr];
            if (v != SC_NONE) pos = A.posmap[v];
            if (pos != SC_NONE) {
                d = (long long)((A.size[v] * 1000ull + A.bpus - 1) / A.bpus);
                f = Fn{d, (long long)A.C[A.step_hi[v] - A.hi_minus] - d};
            }
        }
        const Fn g = block_scan_fn<false, SC_WAVES>(f, carry, wtmp);
        if (pos != SC_NONE) { A.in_start[pos] = g.b; A.in_end[pos] = g.b + d; }
    }
    __syncthreads();
    // what each selected variable takes out of the load curve: the whole steps between the end of
    // its swap-out and the start of its swap-in; transfers that overlap are counted as late
    unsigned long long late = 0;
    for (uint32_t j = tid; j < A.k; j += SC_THREADS) {
        const long long eo = A.out_end[j], si = A.in_start[j];
        if (eo > si) { late += (unsigned long long)(eo - si); continue; }
        const uint32_t T = A.T;
        uint32_t l0 = 0, h0 = T;                  // first t with C[t] >= eo
        while (l0 < h0) { const uint32_t m = (l0 + h0) >> 1; if ((long long)A.C[m] < eo) l0 = m + 1; else h0 = m; }
        const uint32_t lo = l0;
        l0 = 0; h0 = T;                           // last t with C[t] <= si
        while (l0 < h0) { const uint32_t m = (l0 + h0 + 1) >> 1; if ((long long)A.C[m] <= si) l0 = m; else h0 = m - 1; }
        const uint32_t hi = l0;
        if (hi > lo) {
            const unsigned long long s = A.size[min(A.list[j], n - 1)];
            atomicAdd(&A.diff[lo], s);
            atomicAdd(&A.diff[hi], 0ull - s);
        }
    }
    late = wave_reduce_add(late);
    if ((tid & (WAVE - 1)) == 0 && late) atomicAdd(A.late, late);
}

__global__ __launch_bounds__(SC_THREADS) void k_sched_load(uint32_t T, const uint64_t *__restrict__ load,
                                                           const unsigned long long *__restrict__ diff,
                                                           uint64_t *__restrict__ load_sched,
                                                           uint64_t *__restrict__ peak)
{
    __shared__ uint64_t wsum[SC_WAVES], wmax[SC_WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    uint64_t carry = 0, mx = 0;
    for (uint32_t base = 0; base < T; base += SC_THREADS) {
        const uint32_t t = base + tid;
        const uint64_t d = t < T ? diff[t] : 0;
        const uint64_t incl = wave_scan_add(d);
        if (lane == WAVE - 1) wsum[wave] = incl;
        __syncthreads();
        uint64_t pre = 0, tot = 0;
        for (int q = 0; q < SC_WAVES; ++q) { const uint64_t x = wsum[q]; if (q < (int)wave) pre += x; tot += x; }
        __syncthreads();
        if (t < T) {
            const uint64_t v = load[t] - (carry + pre + incl);
            load_sched[t] = v;
            mx = umax64(mx, v);
        }
        carry += tot;
    }
    mx = wave_reduce_max(mx);
    if (lane == 0) wmax[wave] = mx;
    __syncthreads();
    if (tid == 0) {
        uint64_t m = 0;
        for (int q = 0; q < SC_WAVES; ++q) m = umax64(m, wmax[q]);
        *peak = m;
    }
}

hipError_t launch_order_listed(const ListedOrder &L, hipStream_t st)
{
    // (of a list whose length only the device knows, as many workgroups as take one turn for 16 384 variables; longer ones
    // take more turns)
    const uint32_t most = L.count_dev ? (L.n < RANK_LISTED ? L.n : RANK_LISTED) : L.count;
    if (most == 0) return hipSuccess;
    if (L.posmap) hipLaunchKernelGGL(k_sched_mark, dim3((L.count + 255) / 256), dim3(256), 0, st, L.n, L.count, L.list, L.posmap);
    hipLaunchKernelGGL(k_rank_steps, dim3((most + WAVE - 1) / WAVE, 2), dim3(RANK_THREADS), 0, st, L.n, L.count, L.count_dev,
                       L.list, L.posmap, L.step_lo, L.step_hi, L.perm_lo, L.perm_hi);
    return hipGetLastError();
}

hipError_t launch_sched_mark(uint32_t n, uint32_t k, const uint32_t *list, uint32_t *posmap, hipStream_t st)
{
    if (k) hipLaunchKernelGGL(k_sched_mark, dim3((k + 255) / 256), dim3(256), 0, st, n, k, list, posmap);
    return hipGetLastError();
}

hipError_t launch_schedule_swaps(uint32_t n, uint32_t T, uint32_t k, uint32_t count, const uint64_t *size,
                                 const uint32_t *step_lo, const uint32_t *step_hi, uint32_t hi_minus, const uint64_t *C,
                                 const uint32_t *perm_lo, const uint32_t *perm_hi, const uint32_t *posmap,
                                 const uint32_t *list, uint64_t bpus, int64_t *out_start, int64_t *out_end,
                                 int64_t *in_start, int64_t *in_end, uint64_t *diff, uint64_t *late,
                                 const uint64_t *load, uint64_t *load_sched, uint64_t *peak, hipStream_t st)
{
    SchedArgs A{n, T, k, count, size, step_lo, step_hi, hi_minus, C, perm_lo, perm_hi, posmap, list, bpus,
                (long long *)out_start, (long long *)out_end, (long long *)in_start, (long long *)in_end,
                (unsigned long long *)diff, (unsigned long long *)late};
    hipLaunchKernelGGL(k_sched_streams, dim3(1), dim3(SC_THREADS), 0, st, A);
    hipLaunchKernelGGL(k_sched_load, dim3(1), dim3(SC_THREADS), 0, st, T, load, (const unsigned long long *)diff,
                       load_sched, peak);
    return hipGetLastError();
}

}  // namespace lap
