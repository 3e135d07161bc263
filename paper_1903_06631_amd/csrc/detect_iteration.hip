// Iteration detection on a recorded request stream (Section V): the list ends with two equal
// consecutive subsequences of length p; the smallest such p (>= min_period) is reported.
//
// A polynomial hash of every prefix (mod 2^64, odd base) is built with a scan; the two halves of a
// candidate p then compare in O(1):
//     (P[M-p] - P[M-2p]) * r^p == P[M] - P[M-p]
// and the smallest candidate whose hashes agree is checked element by element (hashes mod 2^64 can
// collide, the answer never depends on them); if the check fails the search resumes behind it.
//
// Short lists (up to DI_ONE requests) are one workgroup's work in one launch.  Longer ones take four
// launches that fill the chip: tile totals, prefix hashes, candidates, and the check, whose last
// workgroup to finish writes the answer -- or, when the hashes of a wrong candidate agreed, goes on
// by itself.  2 000 003 requests (16 MB of tokens and as much of hashes, all of it in the last-level
// cache) take 38 us (7.5 ms when one workgroup did all of it): launches that follow each other, and in
// the second one, the longest, every wave's sum over the totals of all tiles before its own (up to 31
// rounds of a load and an add; 14 to 17 us where the first launch reads the same tokens in 9 to 10).
#include "lap_dev.h"
#include "lap_kernels.h"

namespace lap {

constexpr int DI_THREADS = 1024;
constexpr int DI_WAVES = DI_THREADS / WAVE;
constexpr uint64_t DI_BASE = 0x9E3779B97F4A7C15ull | 1ull;
constexpr uint32_t DI_NONE = 0xFFFFFFFFu;
constexpr uint32_t DI_CHUNK = 4 * WAVE;        // tokens a wave takes per step: 4 neighbours per lane
constexpr uint32_t DI_PER = 16;                // candidates per thread

constexpr uint64_t pow_const(uint32_t e)
{
    uint64_t r = 1;
    for (uint32_t i = 0; i < e; ++i) r *= DI_BASE;
    return r;
}
constexpr uint64_t DI_POW256 = pow_const(256);

__device__ __forceinline__ uint64_t pow_base(uint32_t e)
{
    uint64_t r = 1, b = DI_BASE;
    while (e) { if (e & 1u) r *= b; b *= b; e >>= 1; }
    return r;
}

__device__ __forceinline__ uint64_t tok_hash(uint64_t x)
{
    x ^= x >> 31; x *= 0xBF58476D1CE4E5B9ull; x ^= x >> 29; x *= 0x94D049BB133111EBull; x ^= x >> 32;
    return x | 1ull;
}

// Q[i] = P[i + 1]: the hash of the first i + 1 tokens
__device__ __forceinline__ uint64_t prefix_hash(const uint64_t *Q, uint32_t len) { return len ? Q[len - 1] : 0ull; }

__device__ __forceinline__ bool halves_hash_alike(const uint64_t *Q, uint32_t M, uint32_t p, uint64_t pw)
{
    const uint64_t mid = prefix_hash(Q, M - p);
    return (mid - prefix_hash(Q, M - 2 * p)) * pw == Q[M - 1] - mid;
}

// One workgroup of DI_THREADS: candidates from `lo` on in ascending order, DI_THREADS at a time; the
// first one whose hashes agree is checked element by element, and the search resumes behind it if
// the check fails.
__device__ uint32_t search_from(const uint64_t *tok, const uint64_t *Q, uint32_t M, uint32_t lo)
{
    __shared__ uint32_t s_first, s_bad;
    const uint32_t tid = threadIdx.x, pmax = M / 2;
    while (lo <= pmax) {
        if (tid == 0) { s_first = DI_NONE; s_bad = 0; }
        __syncthreads();
        const uint32_t p = lo + tid;
        if (p >= lo && p <= pmax && halves_hash_alike(Q, M, p, pow_base(p))) atomicMin(&s_first, p);
        __syncthreads();
        const uint32_t c = s_first;
        __syncthreads();                 // everyone has read the batch result before it is reset
        if (c == DI_NONE) {
            if (pmax - lo < (uint32_t)DI_THREADS) break;
            lo += DI_THREADS;
            continue;
        }
        bool bad = false;
        for (uint32_t i = tid; i < c && !bad; i += DI_THREADS) bad = tok[M - 2 * c + i] != tok[M - c + i];
        if (bad) s_bad = 1;
        __syncthreads();
        if (!s_bad) return c;
        lo = c + 1;
        __syncthreads();
    }
    return 0;
}

__global__ __launch_bounds__(DI_THREADS) void k_detect_short(const uint64_t *__restrict__ tok, uint32_t M,
                                                             uint32_t min_period, uint64_t *Q,
                                                             uint32_t *__restrict__ period)
{
    __shared__ uint64_t wsum[DI_WAVES];
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    uint64_t carry = 0;
    for (uint32_t base = 0; base < M; base += DI_THREADS) {
        const uint32_t j = base + tid;
        const uint64_t v = j < M ? tok_hash(tok[j]) * pow_base(j) : 0;
        const uint64_t incl = wave_scan_add(v);
        if (lane == WAVE - 1) wsum[wave] = incl;
        __syncthreads();
        uint64_t pre = 0, tot = 0;
        for (int q = 0; q < DI_WAVES; ++q) { const uint64_t x = wsum[q]; if (q < (int)wave) pre += x; tot += x; }
        __syncthreads();
        if (j < M) Q[j] = carry + pre + incl;
        carry += tot;
    }
    __syncthreads();
    const uint32_t p = search_from(tok, Q, M, min_period);
    if (tid == 0) *period = p;
}

// the 4 neighbouring tokens of a lane (hash 0 beyond the list); vec: the list is 16-byte aligned
__device__ __forceinline__ void load_hashes(const uint64_t *__restrict__ tok, uint32_t M, uint64_t j, bool vec, uint64_t (&h)[4])
{
    if (j < M && M - j >= 4) {
        if (vec) {
            const ulonglong2 x = *(const ulonglong2 *)(tok + j), y = *(const ulonglong2 *)(tok + j + 2);
            h[0] = x.x; h[1] = x.y; h[2] = y.x; h[3] = y.y;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) h[k] = tok[j + k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = tok_hash(h[k]);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = (j < M && M - j > (uint32_t)k) ? tok_hash(tok[j + k]) : 0ull;
    }
}

// One wave per tile of `tile` tokens (a multiple of DI_CHUNK).  FINAL false: the tile's total.
// FINAL true: the hash of every prefix that ends in the tile; the totals before it are summed by the
// wave itself (there are at most DI_MAX_TILES).
template <bool FINAL>
__global__ __launch_bounds__(256) void k_detect_hash(const uint64_t *__restrict__ tok, uint32_t M, uint32_t tile,
                                                     uint32_t n_tiles, uint64_t *__restrict__ totals, uint64_t *__restrict__ Q,
                                                     uint32_t *__restrict__ ctrl)
{
    const uint32_t lane = threadIdx.x & (WAVE - 1);
    const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + threadIdx.x / WAVE));
    if (!FINAL && blockIdx.x == 0 && threadIdx.x == 0) { ctrl[0] = DI_NONE; ctrl[1] = 0; }
    if (t >= n_tiles) return;
    const uint32_t first = t * tile, end = M - first < tile ? M : first + tile;
    const bool vec = ((uintptr_t)tok & 15) == 0;
    uint64_t w = pow_base(first) * pow_base(lane * 4);
    uint64_t carry = 0;
    if (FINAL) {
        for (uint32_t q = lane; q < t; q += WAVE) carry += totals[q];
        carry = wave_reduce_add(carry);
    }
    for (uint64_t base = first; base < end; base += DI_CHUNK) {        // (64 bits: the list may end near 2^32)
        uint64_t h[4];
        load_hashes(tok, M, base + lane * 4, vec, h);
        if (FINAL) {
            h[1] = h[1] * DI_BASE + h[0];
            h[2] = h[2] * (DI_BASE * DI_BASE) + h[1];
            h[3] = h[3] * (DI_BASE * DI_BASE * DI_BASE) + h[2];
            const uint64_t own = h[3] * w, incl = wave_scan_add(own), pre = carry + incl - own;
            const uint64_t j = base + lane * 4;
            if (j < M && M - j >= 4) {
                *(ulonglong2 *)(Q + j) = make_ulonglong2(pre + h[0] * w, pre + h[1] * w);
                *(ulonglong2 *)(Q + j + 2) = make_ulonglong2(pre + h[2] * w, pre + own);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (j < M && M - j > (uint32_t)k) Q[j + k] = pre + h[k] * w;
            }
            carry += read_lane64(incl, WAVE - 1);
        } else {
            carry += (((h[3] * DI_BASE + h[2]) * DI_BASE + h[1]) * DI_BASE + h[0]) * w;
        }
        w *= DI_POW256;
    }
    if (!FINAL) {
        carry = wave_reduce_add(carry);
        if (lane == 0) totals[t] = carry;
    }
}

// smallest candidate whose halves hash alike -> ctrl[0]
__global__ __launch_bounds__(256) void k_detect_find(const uint64_t *__restrict__ Q, uint32_t M, uint32_t min_period,
                                                     uint32_t *ctrl)
{
    const uint64_t p0 = (uint64_t)min_period + (uint64_t)blockIdx.x * (256 * DI_PER);
    uint64_t pw = pow_base((uint32_t)p0) * pow_base(threadIdx.x);
#pragma unroll 4
    for (uint32_t k = 0; k < DI_PER; ++k, pw *= DI_POW256) {
        const uint64_t p = p0 + k * 256 + threadIdx.x;
        if (p <= M / 2 && halves_hash_alike(Q, M, (uint32_t)p, pw)) atomicMin(&ctrl[0], (uint32_t)p);
    }
}

// the candidate element by element, by all workgroups; the last one to finish has the answer
__global__ __launch_bounds__(DI_THREADS) void k_detect_check(const uint64_t *__restrict__ tok, uint32_t M,
                                                             const uint64_t *__restrict__ Q, uint32_t *ctrl,
                                                             uint32_t *__restrict__ period)
{
    __shared__ uint32_t s_last, s_wrong;
    const uint32_t c = ctrl[0];          // written by the launch before
    if (c == DI_NONE) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *period = 0;
        return;
    }
    bool bad = false;
    for (uint64_t i = (uint64_t)blockIdx.x * DI_THREADS + threadIdx.x; i < c; i += (uint64_t)gridDim.x * DI_THREADS)
        bad |= tok[M - 2 * c + (uint32_t)i] != tok[M - c + (uint32_t)i];
    // one atomic per workgroup carries both "one more is done" (low half) and "it found a difference"
    bad = __syncthreads_or(bad ? 1 : 0) != 0;
    if (threadIdx.x == 0) {
        const uint32_t mine = bad ? 0x10001u : 1u, all = atomicAdd(&ctrl[1], mine) + mine;
        s_last = (all & 0xFFFFu) == gridDim.x ? 1u : 0u;
        s_wrong = all >> 16;
    }
    __syncthreads();
    if (!s_last) return;
    const uint32_t p = s_wrong ? search_from(tok, Q, M, c + 1) : c;
    if (threadIdx.x == 0) *period = p;
}

// One workgroup takes 27 us for 8192 requests and 15 us for 4000; the four launches take about 20 us
// whatever the length up to 40 000 requests.
constexpr uint32_t DI_ONE = 6144;

hipError_t launch_detect_iteration(const uint64_t *tokens, uint32_t M, uint32_t min_period, uint64_t *Q,
                                   uint64_t *totals, uint32_t *ctrl, uint32_t *period, hipStream_t st)
{
    if (M <= DI_ONE) {
        hipLaunchKernelGGL(k_detect_short, dim3(1), dim3(DI_THREADS), 0, st, tokens, M, min_period, Q, period);
        return hipGetLastError();
    }
    // tiles of at least 1024 tokens (four steps of a wave), at most DI_MAX_TILES of them
    uint32_t tile = 4 * DI_CHUNK;
    if ((M - 1) / tile + 1 > DI_MAX_TILES) tile = ((M - 1) / DI_MAX_TILES / DI_CHUNK + 1) * DI_CHUNK;
    const uint32_t nt = (M - 1) / tile + 1, blocks = (nt + 3) / 4;
    hipLaunchKernelGGL((k_detect_hash<false>), dim3(blocks), dim3(256), 0, st, tokens, M, tile, nt, totals, Q, ctrl);
    hipLaunchKernelGGL((k_detect_hash<true>), dim3(blocks), dim3(256), 0, st, tokens, M, tile, nt, totals, Q, ctrl);
    const uint32_t cands = M / 2 >= min_period ? M / 2 - min_period + 1 : 0;
    if (cands)
        hipLaunchKernelGGL(k_detect_find, dim3((cands - 1) / (256 * DI_PER) + 1), dim3(256), 0, st, Q, M, min_period, ctrl);
    const uint32_t cb = (M - 1) / (4 * DI_THREADS) + 1;
    hipLaunchKernelGGL(k_detect_check, dim3(cb < 256 ? cb : 256), dim3(DI_THREADS), 0, st, tokens, M, Q, ctrl, period);
    return hipGetLastError();
}

}  // namespace lap
