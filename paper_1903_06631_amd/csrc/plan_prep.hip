// Preparation of a plan: granule shift, lifetime statistics, layout of the per-step lists, which kernel places the trace,
// and the variables' records.
#include "lap_dev.h"
#include "lap_kernels.h"
#include "step_runs.h"

namespace lap {

namespace {

// the variables first, first + stride, ..: difference of the numbers live per step (modulo 2^32), and the header's sums;
// those of the segment lists (segs) only where the trace is large enough for them
__device__ __forceinline__ void prep_sums(uint32_t first, uint32_t stride, uint32_t n, uint32_t T,
                                          const uint64_t *__restrict__ size, const uint32_t *__restrict__ alloc,
                                          const uint32_t *__restrict__ free_, uint32_t *cntd, PlanHeader *hdr, bool segs)
{
    unsigned long long orv = 0, sum = 0;
    unsigned long long seg[PLAN_SEG_CAND];
#pragma unroll
    for (uint32_t c = 0; c < PLAN_SEG_CAND; ++c) seg[c] = 0;
    uint32_t multi = 0;
    // whole waves go round: neighbours' equal steps are summed before they reach the counters
    for (uint32_t i = first; i - (uint32_t)lane_id() < n; i += stride) {
        const bool in = i < n;
        const uint64_t s = in ? size[i] : 0;
        const uint32_t a = in ? alloc[i] : 0, f = in ? free_[i] : 0;
        wave_add_runs(in && a < T ? a : NO_KEY, 1, [&](uint32_t t, uint64_t c) { atomicAdd(&cntd[t], (uint32_t)c); });
        wave_add_runs(in && f < T ? f : NO_KEY, 1, [&](uint32_t t, uint64_t c) { atomicAdd(&cntd[t], 0u - (uint32_t)c); });
        if (!in) break;
        orv |= s;
        sum += s;
        multi += (f - a > 1) ? 1u : 0u;
        if (!segs) continue;
        // lists the block would enter with segments of 2^sh steps: one per segment it touches,
        // one more per segment it lives through, one per step in the others
#pragma unroll
        for (uint32_t c = 0; c < PLAN_SEG_CAND; ++c) {
            const uint32_t sh = PLAN_SEG_SHIFT0 + c, w = 1u << sh, K = (uint32_t)(((uint64_t)T + w - 1) >> sh);
            const uint32_t k0 = a >> sh, k1 = (f - 1) >> sh;
            const uint32_t kf0 = (uint32_t)(((uint64_t)a + w - 1) >> sh), kf1 = f == T ? K : f >> sh;
            const uint32_t nf = kf1 > kf0 ? kf1 - kf0 : 0;
            uint32_t steps = f - a;
            if (nf) {
                const uint64_t hi = (uint64_t)kf1 << sh;
                steps -= (uint32_t)((hi < T ? hi : (uint64_t)T) - ((uint64_t)kf0 << sh));
            }
            seg[c] += 1ull + (k1 - k0 + 1) + nf + steps;      // (the first: the list of everything)
        }
    }
    for (int m = WAVE / 2; m > 0; m >>= 1) orv |= shfl_xor64(orv, m);
    sum = wave_reduce_add(sum);
    multi = wave_reduce_add32(multi);
    if (segs)
#pragma unroll
        for (uint32_t c = 0; c < PLAN_SEG_CAND; ++c) seg[c] = wave_reduce_add(seg[c]);
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        atomicOr((unsigned long long *)&hdr->or_sizes, orv);
        atomicAdd((unsigned long long *)&hdr->sum_sizes, sum);
        atomicAdd(&hdr->n_multi, multi);
        if (segs)
#pragma unroll
            for (uint32_t c = 0; c < PLAN_SEG_CAND; ++c) atomicAdd(&hdr->seg_tot[c], seg[c]);
    }
}

constexpr uint32_t HDR_WORDS = sizeof(PlanHeader) / 8;
static_assert(sizeof(PlanHeader) % 8 == 0, "the header is cleared in 64-bit words");

// 200 000 variables over 580 steps: 18 us; 308 us when every wave of a thousand workgroups added its sums to the header.
__global__ __launch_bounds__(256) void k_plan_prep1(uint32_t n, uint32_t T, const uint64_t *__restrict__ size,
                                                    const uint32_t *__restrict__ alloc,
                                                    const uint32_t *__restrict__ free_, uint32_t *cntd,
                                                    PlanHeader *hdr, bool segs)
{
    __shared__ PlanHeader h;                     // the workgroup's sums: adds to one word of the header are served one by one
    const uint32_t tid = threadIdx.x;
    if (tid < HDR_WORDS) ((uint64_t *)&h)[tid] = 0;
    __syncthreads();
    prep_sums(blockIdx.x * blockDim.x + tid, gridDim.x * blockDim.x, n, T, size, alloc, free_, cntd, &h, segs);
    __syncthreads();
    if (segs && tid < PLAN_SEG_CAND) atomicAdd(&hdr->seg_tot[tid], h.seg_tot[tid]);
    if (tid == WAVE) {
        atomicOr(&hdr->or_sizes, h.or_sizes);
        atomicAdd(&hdr->sum_sizes, h.sum_sizes);
        atomicAdd(&hdr->n_multi, h.n_multi);
    }
}

constexpr int PREP_THREADS = 1024;

__device__ __forceinline__ uint64_t prep_block_scan(uint64_t v, uint64_t *wtmp, uint64_t &total)
{
    const int tid = threadIdx.x, l = tid & (WAVE - 1), w = tid / WAVE;
    const uint64_t incl = wave_scan_add(v);
    if (l == WAVE - 1) wtmp[w] = incl;
    __syncthreads();
    uint64_t pre = 0, tot = 0;
    for (int k = 0; k < PREP_THREADS / WAVE; ++k) {
        const uint64_t x = wtmp[k];
        if (k < w) pre += x;
        tot += x;
    }
    __syncthreads();
    total = tot;
    return pre + incl;
}

// Two pairs of variables a thread that are listed close to each other, read before anything else so that nobody waits for them
struct PrepPairs {
    static constexpr uint32_t PAIRS = 2;
    uint64_t si[PAIRS], sj[PAIRS];
    uint32_t ai[PAIRS], fi[PAIRS], aj[PAIRS], fj[PAIRS];
    bool turned[PAIRS];          // j is listed before i
    __device__ __forceinline__ void load(uint32_t n, const uint64_t *__restrict__ size, const uint32_t *__restrict__ alloc,
                                         const uint32_t *__restrict__ free_)
    {
#pragma unroll
        for (uint32_t k = 0; k < PAIRS; ++k) {
            const uint32_t q = threadIdx.x * PAIRS + k, i = (uint32_t)((uint64_t)q * n / (PREP_THREADS * PAIRS)),
                           d = i + 1 + q * 37 % 63, j = d < n ? d : d - n;
            turned[k] = d >= n;
            ai[k] = alloc[i]; fi[k] = free_[i]; si[k] = size[i];
            aj[k] = alloc[j]; fj[k] = free_[j]; sj[k] = size[j];
        }
    }
    // adds to three counts of 16 bits: pairs that meet, cross, and have one size (batches_lose)
    __device__ __forceinline__ void count(unsigned long long *sum) const
    {
        unsigned long long mine = 0;
#pragma unroll
        for (uint32_t k = 0; k < PAIRS; ++k) {
            const bool meet = ai[k] < fj[k] && aj[k] < fi[k];
            // of two allocated in one step the first in the list
            const bool cross = ai[k] == aj[k] ? (fi[k] < fj[k]) != turned[k] && fi[k] != fj[k] : (ai[k] < aj[k]) == (fi[k] < fj[k]) && fi[k] != fj[k];
            mine += (unsigned long long)__popcll(ballot(meet)) | (unsigned long long)__popcll(ballot(meet && cross)) << 16 |
                    (unsigned long long)__popcll(ballot(meet && si[k] == sj[k])) << 32;
        }
        if ((threadIdx.x & (WAVE - 1)) == 0) atomicAdd(sum, mine);
    }
};

// live[t] = number of variables live at step t; lstart = exclusive prefix sum of live + 1; one workgroup
__device__ __forceinline__ void prep_lists(uint32_t n, uint32_t T, uint32_t B, const uint32_t *cntd,
                                           uint32_t *__restrict__ lstart, PlanHeader *hdr, PlanHeader *for_batches,
                                           uint64_t *wtmp, const unsigned long long *pairs,
                                           uint64_t seg_pool_entries, uint64_t seg_min_vars, BatchTrial batches)
{
    const uint32_t tid = threadIdx.x;
    uint64_t c1 = 0, c2 = 0, tot;
    for (uint32_t base = 0; base < T; base += PREP_THREADS) {
        const uint32_t t = base + tid;
        const bool in = t < T;
        const uint64_t d = in ? (uint64_t)(int64_t)(int32_t)cntd[t] : 0;     // signed delta
        const uint64_t live = c1 + prep_block_scan(d, wtmp, tot); c1 += tot;
        // room for the holes: blocks + 1, rounded up to 16 entries so that every list starts on a
        // 128-byte line (a fetch of n entries then touches ceil(n / 16) lines, not one more)
        const uint64_t lv = in ? ((live + 1 + 15) & ~15ull) : 0;
        const uint64_t incl = c2 + prep_block_scan(lv, wtmp, tot);
        if (in) lstart[t] = (uint32_t)(incl - lv);
        c2 += tot;
    }
    if (tid == 0) {
        lstart[T] = (uint32_t)c2;
        const uint64_t orv = hdr->or_sizes, sum = hdr->sum_sizes;
        const uint32_t shift = orv ? (uint32_t)__ffsll((unsigned long long)orv) - 1 : 0;
        const bool fast = (sum >> shift) < (1ull << 32);
        const bool lists = fast && c2 <= (uint64_t)PLAN_CL * n;
        hdr->shift = shift;
        hdr->fast = fast ? 1u : 0u;
        hdr->mode1 = lists && !reg_before_lists(n, T, hdr->n_multi, B) ? 1u : 0u;
        if (batches.look) {                      // (only where n < seg_min_vars)
            const uint64_t c = *pairs;
            const bool batch = fast && !lists && !batches_lose(n, B, batches.by_trace, (uint32_t)c & 0xFFFF, (uint32_t)(c >> 16) & 0xFFFF, (uint32_t)(c >> 32));
            hdr->mode2 = batch ? 2u : 0u;
            for_batches->fast = batch ? 1u : 0u;
            for_batches->shift = shift;
            for_batches->mode1 = for_batches->mode2 = 0;
        }
        if (n < seg_min_vars) return;            // no segment lists, and none of their figures (the header is zero)
        // Segment lists: the width that enters the fewest blocks into lists; every list has one
        // entry more than the blocks it sees.  Taken when per-step lists are not, the trace has
        // enough variables for them to pay (below that, sweeping the sorted blocks is faster), the
        // list directory and one ordering fit 32-bit indices, addresses stay below the end marker
        // of the top range, and the pool has room for at least one ordering.
        uint32_t best_c = 0;
        uint64_t best_need = ~0ull;
        for (uint32_t c = 0; c < PLAN_SEG_CAND; ++c) {
            const uint32_t sh = PLAN_SEG_SHIFT0 + c;
            const uint64_t K = ((uint64_t)T + (1ull << sh) - 1) >> sh;
            const uint64_t need = hdr->seg_tot[c] + 2 * K + T + 1;
            if (need < best_need) { best_need = need; best_c = c; }
        }
        // ... or rather the narrowest width within an eighth of that: narrower segments mean fewer
        // lists per variable (a variable asks about lifetime / w + w of them)
        for (uint32_t c = 0; c < best_c; ++c) {
            const uint32_t sh = PLAN_SEG_SHIFT0 + c;
            const uint64_t K = ((uint64_t)T + (1ull << sh) - 1) >> sh;
            const uint64_t need = hdr->seg_tot[c] + 2 * K + T + 1;
            if (need <= best_need + best_need / 8) { best_need = need; best_c = c; break; }
        }
        const uint32_t ssh = PLAN_SEG_SHIFT0 + best_c;
        const uint64_t K = ((uint64_t)T + (1ull << ssh) - 1) >> ssh;
        const uint64_t slots = best_need ? seg_pool_entries / best_need : 0;
        const bool seg = fast && !lists && (sum >> shift) < 0xFFFFFFFEull &&
                         best_need < 0xFFFFFFFFull && T < 0x7FFF0000u && slots >= 1 &&
                         !(batches.first && batches_before_segments(n, B, best_need));
        hdr->mode2 = seg ? 1u : 0u;
        hdr->seg_shift = ssh;
        hdr->seg_K = (uint32_t)K;
        hdr->seg_slots = (uint32_t)(slots < B ? slots : B);
        hdr->seg_need = best_need;
    }
}

__global__ __launch_bounds__(PREP_THREADS) void k_plan_prep2(uint32_t n, uint32_t T, uint32_t B,
                                                             const uint64_t *__restrict__ size,
                                                             const uint32_t *__restrict__ alloc,
                                                             const uint32_t *__restrict__ free_,
                                                             const uint32_t *__restrict__ cntd,
                                                             uint32_t *__restrict__ lstart, PlanHeader *hdr,
                                                             uint64_t seg_pool_entries, uint64_t seg_min_vars,
                                                             BatchTrial batches)
{
    __shared__ uint64_t wtmp[PREP_THREADS / WAVE];
    __shared__ unsigned long long pairs;
    PrepPairs P;
    if (batches.look) {
        P.load(n, size, alloc, free_);
        if (threadIdx.x == 0) pairs = 0;
        __syncthreads();
        P.count(&pairs);
        __syncthreads();
    }
    prep_lists(n, T, B, cntd, lstart, hdr, hdr + 1, wtmp, &pairs, seg_pool_entries, seg_min_vars, batches);
}

// What the placement kernel reads of a variable, in one 16-byte record (one gather per rank
// instead of three): first step, end of life, size in granules.  Only meaningful on the
// 32-bit path (size >> shift fits 32 bits there).
__global__ __launch_bounds__(256) void k_plan_pack(uint32_t n, const uint64_t *__restrict__ size,
                                                   const uint32_t *__restrict__ alloc,
                                                   const uint32_t *__restrict__ free_, const PlanHeader *hdr,
                                                   uint4 *__restrict__ vrec)
{
    if (!hdr->fast) return;
    const uint32_t sh = hdr->shift;
    for (uint32_t v = blockIdx.x * 256 + threadIdx.x; v < n; v += gridDim.x * 256)
        vrec[v] = make_uint4(alloc[v], free_[v], (uint32_t)(size[v] >> sh), 0u);
}

// All of the preparation by one workgroup, the counters and the header in LDS: bound by its launch.  Two fills and the
// three kernels above took 20 us of the 100 that a plan of 120 variables and 22 steps takes, this one 6; up to the sizes
// below a workgroup is done before five launches are.
constexpr uint32_t PREP_SMALL_VARS = 4096, PREP_SMALL_STEPS = 4096;
__global__ __launch_bounds__(PREP_THREADS) void k_plan_prep_small(uint32_t n, uint32_t T, uint32_t B,
                                                                  const uint64_t *__restrict__ size,
                                                                  const uint32_t *__restrict__ alloc,
                                                                  const uint32_t *__restrict__ free_,
                                                                  uint32_t *__restrict__ lstart, PlanHeader *hdr,
                                                                  uint4 *__restrict__ vrec, uint64_t seg_pool_entries,
                                                                  uint64_t seg_min_vars, BatchTrial batches)
{
    __shared__ PlanHeader h;
    __shared__ uint32_t cntd[PREP_SMALL_STEPS + 1];
    __shared__ uint64_t wtmp[PREP_THREADS / WAVE];
    __shared__ unsigned long long pairs;
    const uint32_t tid = threadIdx.x;
    PrepPairs P;
    if (batches.look) P.load(n, size, alloc, free_);
    if (tid == 0) pairs = 0;
    for (uint32_t t = tid; t <= T; t += PREP_THREADS) cntd[t] = 0;
    if (tid < HDR_WORDS) ((uint64_t *)&h)[tid] = 0;
    __syncthreads();
    prep_sums(tid, PREP_THREADS, n, T, size, alloc, free_, cntd, &h, n >= seg_min_vars);
    if (batches.look) P.count(&pairs);
    __syncthreads();
    prep_lists(n, T, B, cntd, lstart, &h, hdr + 1, wtmp, &pairs, seg_pool_entries, seg_min_vars, batches);
    __syncthreads();
    if (tid < HDR_WORDS) ((uint64_t *)hdr)[tid] = ((const uint64_t *)&h)[tid];
    if (!h.fast) return;
    for (uint32_t v = tid; v < n; v += PREP_THREADS)
        vrec[v] = make_uint4(alloc[v], free_[v], (uint32_t)(size[v] >> h.shift), 0u);
}

}  // namespace

hipError_t launch_plan_prep(uint32_t n, uint32_t T, uint32_t B, const uint64_t *size, const uint32_t *alloc,
                            const uint32_t *free_, uint32_t *cntd, uint32_t *lstart, PlanHeader *hdr, void *vrec,
                            uint64_t seg_pool_entries, uint64_t seg_min_vars, BatchTrial batches, hipStream_t st)
{
    if (n <= PREP_SMALL_VARS && T <= PREP_SMALL_STEPS) {
        hipLaunchKernelGGL(k_plan_prep_small, dim3(1), dim3(PREP_THREADS), 0, st, n, T, B, size, alloc, free_, lstart, hdr,
                           (uint4 *)vrec, seg_pool_entries, seg_min_vars, batches);
        return hipGetLastError();
    }
    // the header and the counters lie one after the other: one fill clears both
    hipError_t e = launch_fill_u64((uint64_t *)hdr, (size_t)((char *)(cntd + T) - (char *)hdr) / 8 + 1, 0, st);
    if (e != hipSuccess) return e;
    uint32_t blocks = (n + 255) / 256;
    blocks = blocks > 1024 ? 1024 : blocks;
    hipLaunchKernelGGL(k_plan_prep1, dim3(blocks > 128 ? 128 : blocks), dim3(256), 0, st, n, T, size, alloc, free_, cntd, hdr, n >= seg_min_vars);
    hipLaunchKernelGGL(k_plan_prep2, dim3(1), dim3(PREP_THREADS), 0, st, n, T, B, size, alloc, free_, cntd, lstart, hdr, seg_pool_entries,
                       seg_min_vars, batches);
    hipLaunchKernelGGL(k_plan_pack, dim3(blocks), dim3(256), 0, st, n, size, alloc, free_, hdr, (uint4 *)vrec);
    return hipGetLastError();
}

}  // namespace lap
