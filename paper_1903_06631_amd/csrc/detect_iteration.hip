// Iteration detection on a recorded request stream (Section V): the list ends with two equal
// consecutive subsequences of length p; the smallest such p (>= min_period) is reported.
//
// First the direct way.  The last DI_SUFFIX tokens are looked for at every distance p (nearly every one is refused by its first
// token, so half of the list is read once).  A workgroup goes on with the smallest distances that remain of its own: a wave
// compares up to DI_DEEP more tokens of each, which refuses most of what a repeated piece inside an iteration leaves, and settles
// short repeats.  The DI_FEW smallest that are still open and below the smallest that is settled are then compared element by element by all
// workgroups, the last of which has the answer -- unless all of them differ and there are more.  Only then it
// comes to hashes, whose cost does not depend on what is in the list: a polynomial hash of every prefix (mod 2^64, odd
// base) is built with a scan; the two halves of a candidate p then compare in O(1):
//     (P[M-p] - P[M-2p]) * r^p == P[M] - P[M-p]
// and the smallest candidate whose hashes agree is checked element by element (hashes mod 2^64 can
// collide, the answer never depends on them); if the check fails the search resumes behind it.
//
// Short lists (up to DI_ONE requests) are one workgroup's work in one launch.  Longer ones take three, the last of which nearly
// always finds nothing to do.  An iteration in 2 000 003 requests: 16 us, of which the first launch takes 6 and the second 9; by
// hashes it took 38.  One in 4000: 9.5 and 14.7 us.  700 000 requests that end in a short period: 24 us, 64 and more by hashes.  What
// it comes to hashes for -- a run of a short period that is shorter than twice the smallest iteration asked for, of thousands of
// requests -- takes 51 us for 40 000 of them and 154 for 2 000 003 (20 and 32 by hashes at once).
#include "lap_dev.h"
#include "lap_kernels.h"

namespace lap {

constexpr int DI_THREADS = 1024;
constexpr int DI_WAVES = DI_THREADS / WAVE;
constexpr uint64_t DI_BASE = 0x9E3779B97F4A7C15ull | 1ull;
constexpr uint32_t DI_NONE = 0xFFFFFFFFu;
constexpr uint32_t DI_CHUNK = 4 * WAVE;        // tokens a wave takes per step: 4 neighbours per lane
constexpr uint32_t DI_SUFFIX = 32, DI_DEEP = 1024;       // tokens that a distance has to agree in, and more
constexpr uint32_t DI_FEW = 4;                 // distances that are compared by all workgroups, at most
constexpr uint32_t DI_SPAN = 8;                // distances per thread
constexpr uint32_t DI_ONE = 6144;             // requests that one workgroup looks at
constexpr uint32_t DI_TILES = 1024, DI_LISTS = 512;      // at most

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

// whether the last tokens, DI_SUFFIX of them or p, are also found at distance p (2 p <= M)
__device__ __forceinline__ bool suffix_repeats(const uint64_t *__restrict__ tok, uint32_t M, uint32_t p)
{
    const uint32_t most = min(p, DI_SUFFIX);
    for (uint32_t j = 1; j <= most; j += 8) {            // eight at a time: a wave waits for each round
        uint64_t differ = 0;
#pragma unroll
        for (uint32_t k = 0; k < 8; ++k) {
            const uint32_t e = M - min(j + k, most);
            differ |= tok[e] ^ tok[e - p];
        }
        if (differ) return false;
    }
    return true;
}

// What a wave finds out about distance p, whose last DI_SUFFIX tokens agree, from `deep` more
enum { DI_DIFFERS, DI_OPEN, DI_SAME };
__device__ __forceinline__ uint32_t look_deep(const uint64_t *__restrict__ tok, uint32_t M, uint32_t p, uint32_t deep)
{
    constexpr uint32_t STEP = 4 * WAVE;
    const uint32_t most = min(p, DI_SUFFIX + deep);
    for (uint32_t j = DI_SUFFIX + 1 + (uint32_t)lane_id(); ballot(j <= most); j += STEP) {
        uint64_t differ = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t e = M - min(j + k * WAVE, most);
            differ |= tok[e] ^ tok[e - p];
        }
        if (ballot(differ != 0)) return DI_DIFFERS;
    }
    return most == p ? DI_SAME : DI_OPEN;
}

// the smallest of the listed distances that are not marked as different, 0 if there is none
__device__ __forceinline__ uint32_t smallest_same(const uint32_t *list, uint32_t found, uint32_t differ)
{
    uint32_t best = DI_NONE;
    for (uint32_t q = 0; q < found; ++q)
        if (!((differ >> q) & 1)) best = min(best, list[q]);
    return best == DI_NONE ? 0 : best;
}

__global__ __launch_bounds__(DI_THREADS) void k_detect_short(const uint64_t *__restrict__ tok, uint32_t M,
                                                             uint32_t min_period, uint64_t *Q,
                                                             uint32_t *__restrict__ period)
{
    __shared__ uint64_t wsum[DI_WAVES];
    constexpr uint32_t DEEP = 4 * DI_WAVES;              // distances that waves compare, at most
    __shared__ uint32_t s_bits[2 * WAVE], s_list[DEEP], s_found, s_same;
    static_assert(DI_ONE / 2 < 2 * WAVE * 32, "a bit per distance");
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    if (tid < 2 * WAVE) s_bits[tid] = 0;
    if (tid == 0) s_same = DI_NONE;
    __syncthreads();
    for (uint32_t p = min_period + tid; p >= min_period && p <= M / 2; p += DI_THREADS)
        if (suffix_repeats(tok, M, p)) atomicOr(&s_bits[p / 32], 1u << (p % 32));
    __syncthreads();
    if (wave == 0) {                                       // the smallest of them, in ascending order
        uint64_t bits = (uint64_t)s_bits[2 * lane + 1] << 32 | s_bits[2 * lane];
        const uint32_t own = (uint32_t)__popcll(bits);
        uint32_t at = own;
        for (int d = 1; d < WAVE; d <<= 1) { const uint32_t y = (uint32_t)__shfl_up((int)at, d, WAVE); if ((int)lane >= d) at += y; }
        if (lane == WAVE - 1) s_found = at;
        for (at -= own; bits && at < DEEP; bits &= bits - 1, ++at) s_list[at] = lane * 64 + (uint32_t)__ffsll((unsigned long long)bits) - 1;
    }
    __syncthreads();
    const uint32_t found = s_found;
    uint32_t same = DI_NONE;
    for (uint32_t base = 0; base < min(found, DEEP) && same == DI_NONE; base += DI_WAVES) {
        const uint32_t q = base + wave;
        if (q < min(found, DEEP) && look_deep(tok, M, s_list[q], M) == DI_SAME && lane == 0) atomicMin(&s_same, s_list[q]);
        __syncthreads();
        same = s_same;
        __syncthreads();
    }
    if (same != DI_NONE || found <= DEEP) {
        if (tid == 0) *period = same != DI_NONE ? same : 0;
        return;
    }
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

// Scratch of longer lists, in the words after each other that lap_kernels.h calls totals
struct DiScratch {
    uint64_t totals[DI_TILES];
    uint32_t counts[DI_LISTS], lists[DI_LISTS * DI_FEW];      // of a workgroup: its open distances, and the smallest of them
    uint32_t settled[DI_LISTS];                // the smallest of its distances that is known to be a repeat
    uint32_t done, differ, hashes;             // workgroups that have compared, which distances differ, whether it comes to hashes
    uint32_t next[2], ready[2];                // tiles given out and finished: totals, hashes
    uint32_t candidate, searched;              // the smallest distance whose hashes agree; workgroups that have searched
};
static_assert(sizeof(DiScratch) <= DI_MAX_TILES * 8, "");

__global__ __launch_bounds__(256) void k_detect_suffix(const uint64_t *__restrict__ tok, uint32_t M, uint32_t min_period,
                                                       DiScratch *S)
{
    constexpr uint32_t SPAN = 256 * DI_SPAN, DEEP = 8;                // distances a round; that waves look at, at most
    __shared__ uint32_t s_bits[SPAN / 32], s_list[DEEP + DI_FEW], s_what[DEEP], s_found;
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    if (blockIdx.x == 0 && tid == 0) {
        S->done = 0; S->differ = 0; S->hashes = 0; S->next[0] = S->next[1] = S->ready[0] = S->ready[1] = 0; S->candidate = DI_NONE; S->searched = 0;
    }
    const uint64_t last = tok[M - 1];
    const uint32_t most = M / 2;
    uint32_t open = 0, same = DI_NONE;         // thread 0: this workgroup's
    for (uint64_t base = (uint64_t)min_period + (uint64_t)blockIdx.x * SPAN; base <= most; base += (uint64_t)gridDim.x * SPAN) {
        if (tid < SPAN / 32) s_bits[tid] = 0;
        if (tid == 0) s_found = 0;
        __syncthreads();
        uint64_t x[DI_SPAN];
#pragma unroll
        for (uint32_t k = 0; k < DI_SPAN; ++k) {
            const uint64_t p = base + k * 256 + tid;
            x[k] = tok[M - 1 - (p <= most ? (uint32_t)p : 0u)];
        }
#pragma unroll
        for (uint32_t k = 0; k < DI_SPAN; ++k) {
            const uint64_t p = base + k * 256 + tid;
            if (x[k] == last && p <= most && suffix_repeats(tok, M, (uint32_t)p)) {
                atomicOr(&s_bits[(k * 256 + tid) / 32], 1u << (tid % 32));
                s_found = 1;
            }
        }
        __syncthreads();
        if (!s_found) continue;
        // the smallest of them, in ascending order
        static_assert(SPAN / 32 == WAVE, "");
        if (wave == 0) {
            uint32_t bits = s_bits[lane];
            const uint32_t own = (uint32_t)__popc(bits);
            uint32_t at = own;
            for (int d = 1; d < WAVE; d <<= 1) { const uint32_t y = (uint32_t)__shfl_up((int)at, d, WAVE); if ((int)lane >= d) at += y; }
            if (lane == WAVE - 1) s_found = at;
            for (at -= own; bits && at < DEEP + DI_FEW; bits &= bits - 1, ++at)
                s_list[at] = (uint32_t)base + lane * 32 + (uint32_t)__ffs((int)bits) - 1;
        }
        __syncthreads();
        const uint32_t found = s_found, look = min(found, DEEP);
        for (uint32_t q = wave; q < look; q += 4) {
            const uint32_t what = look_deep(tok, M, s_list[q], DI_DEEP);
            if (lane == 0) s_what[q] = what;
            if (what == DI_SAME) break;        // (those above do not matter)
        }
        __syncthreads();
        if (tid == 0 && same == DI_NONE) {
            uint32_t q = 0;
            for (; q < look && same == DI_NONE; ++q) {
                if (s_what[q] == DI_SAME) {
                    same = s_list[q];
                } else if (s_what[q] == DI_OPEN) {
                    if (open < DI_FEW) S->lists[blockIdx.x * DI_FEW + open] = s_list[q];
                    ++open;
                }
            }
            if (same == DI_NONE) {             // those that were not looked at are open
                for (; q < found && open < DI_FEW; ++q, ++open) S->lists[blockIdx.x * DI_FEW + open] = s_list[q];
                open += found - q;
            }
        }
        __syncthreads();
    }
    if (tid == 0) { S->counts[blockIdx.x] = open; S->settled[blockIdx.x] = same; }
}

// The smallest open distances element by element, by all workgroups; the last one to finish has the answer.
__global__ __launch_bounds__(DI_THREADS) void k_detect_compare(const uint64_t *__restrict__ tok, uint32_t M, DiScratch *S,
                                                               uint32_t n_lists, uint32_t *__restrict__ period)
{
    static_assert(DI_LISTS <= DI_THREADS, "a thread per list");
    __shared__ uint32_t s_best, s_list[DI_FEW + 1], s_more, s_last;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) { s_best = DI_NONE; s_more = 0; }
    if (tid <= DI_FEW) s_list[tid] = DI_NONE;
    __syncthreads();
    uint32_t mine[DI_FEW], count = 0;
#pragma unroll
    for (uint32_t q = 0; q < DI_FEW; ++q) mine[q] = DI_NONE;
    if (tid < n_lists) {
        count = S->counts[tid];
#pragma unroll
        for (uint32_t q = 0; q < DI_FEW; ++q)
            if (q < count) mine[q] = S->lists[tid * DI_FEW + q];
        const uint32_t same = S->settled[tid];
        if (same != DI_NONE) atomicMin(&s_best, same);
    }
    __syncthreads();
    const uint32_t best = s_best;
    // the smallest ones below that, one after the other
    uint32_t found = 0;
    for (; found <= DI_FEW; ++found) {
        uint32_t x = DI_NONE;
#pragma unroll
        for (uint32_t q = 0; q < DI_FEW; ++q)
            if (mine[q] < best && (found == 0 || mine[q] > s_list[found - 1])) x = min(x, mine[q]);
        if (x != DI_NONE) atomicMin(&s_list[found], x);
        __syncthreads();
        if (s_list[found] == DI_NONE) break;
    }
    // more than those: a fifth, or a list that is not complete
    if (found > DI_FEW) found = DI_FEW;
    if (count > DI_FEW && mine[DI_FEW - 1] < best) s_more = 1;
    if (tid == 0 && s_list[DI_FEW] != DI_NONE) s_more = 1;
    __syncthreads();
    uint32_t differ = 0;
    for (uint32_t q = 0; q < found; ++q) {
        const uint32_t c = s_list[q];
        bool bad = false;
#pragma unroll 4
        for (uint64_t i = (uint64_t)blockIdx.x * DI_THREADS + tid; i < c; i += (uint64_t)gridDim.x * DI_THREADS)
            bad |= tok[M - 2 * c + (uint32_t)i] != tok[M - c + (uint32_t)i];
        if (__syncthreads_or(bad ? 1 : 0)) differ |= 1u << q;
    }
    if (tid == 0) {
        if (differ) atomicOr(&S->differ, differ);
        __threadfence();
        s_last = atomicAdd(&S->done, 1u) + 1 == gridDim.x ? 1u : 0u;
    }
    __syncthreads();
    if (s_last && tid == 0) {
        __threadfence();
        const uint32_t p = smallest_same(s_list, found, atomicOr(&S->differ, 0u));
        if (!p && s_more) S->hashes = 1;
        *period = p ? p : best == DI_NONE ? 0 : best;
    }
}

// A barrier of the workgroup does not wait for its waves' stores and atomics to global memory.  Where one thread then tells other
// workgroups that all of them have been made, every wave waits for its own before the barrier.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Adds the tiles that this wave has finished, and waits until all are.  The workgroup's stores reach memory once, with the
// counter: a write-back by every wave took three times as long as all of the hashes.
__device__ __forceinline__ void wait_tiles(uint32_t *ready, uint32_t mine, uint32_t n_tiles, uint32_t *s_sum)
{
    wait_stores();
    if (threadIdx.x == 0) *s_sum = 0;
    __syncthreads();
    if (lane_id() == 0 && mine) atomicAdd(s_sum, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (*s_sum) __hip_atomic_fetch_add(ready, *s_sum, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        while (__hip_atomic_load(ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n_tiles) __builtin_amdgcn_s_sleep(8);
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// the workgroup's next tiles, one for each of its waves (a counter for single waves took 0.2 ms: the chip adds to one address one
// after the other)
__device__ __forceinline__ uint32_t next_tiles(uint32_t *next, uint32_t *s_next)
{
    __syncthreads();
    if (threadIdx.x == 0) *s_next = atomicAdd(next, (uint32_t)DI_WAVES);
    __syncthreads();
    return *s_next;
}

// The hashes: the totals of tiles of `tile` tokens (a multiple of DI_CHUNK), the hash of every prefix, the candidates; the last
// workgroup to finish checks the smallest.  A workgroup takes tiles from a counter, so what others wait for is held by one
// that runs already, and every wait ends.
__global__ __launch_bounds__(DI_THREADS) void k_detect_hash(const uint64_t *__restrict__ tok, uint32_t M, uint32_t min_period,
                                                            uint32_t tile, uint32_t n_tiles, DiScratch *S, uint64_t *Q,
                                                            uint32_t *__restrict__ period)
{
    __shared__ uint32_t s_last, s_sum, s_next;
    if (!S->hashes) return;
    const uint32_t lane = threadIdx.x & (WAVE - 1), tid = threadIdx.x;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / WAVE));
    const bool vec = ((uintptr_t)tok & 15) == 0;
    uint32_t mine = 0;
    for (uint32_t t0 = next_tiles(&S->next[0], &s_next); t0 < n_tiles; t0 = next_tiles(&S->next[0], &s_next)) {
        const uint32_t t = t0 + wave;
        if (t >= n_tiles) continue;
        const uint32_t first = t * tile, end = M - first < tile ? M : first + tile;
        uint64_t w = pow_base(first) * pow_base(lane * 4), total = 0;
        for (uint64_t base = first; base < end; base += DI_CHUNK, w *= DI_POW256) {        // (64 bits: the list may end near 2^32)
            uint64_t h[4];
            load_hashes(tok, M, base + lane * 4, vec, h);
            total += (((h[3] * DI_BASE + h[2]) * DI_BASE + h[1]) * DI_BASE + h[0]) * w;
        }
        total = wave_reduce_add(total);
        if (lane == 0) S->totals[t] = total;
        ++mine;
    }
    wait_tiles(&S->ready[0], mine, n_tiles, &s_sum);
    mine = 0;
    for (uint32_t t0 = next_tiles(&S->next[1], &s_next); t0 < n_tiles; t0 = next_tiles(&S->next[1], &s_next)) {
        const uint32_t t = t0 + wave;
        if (t >= n_tiles) continue;
        const uint32_t first = t * tile, end = M - first < tile ? M : first + tile;
        uint64_t w = pow_base(first) * pow_base(lane * 4), carry = 0;
        for (uint32_t q = lane; q < t; q += WAVE) carry += S->totals[q];
        carry = wave_reduce_add(carry);
        for (uint64_t base = first; base < end; base += DI_CHUNK) {
            uint64_t h[4];
            load_hashes(tok, M, base + lane * 4, vec, h);
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
            w *= DI_POW256;
        }
        ++mine;
    }
    wait_tiles(&S->ready[1], mine, n_tiles, &s_sum);
    const uint32_t most = M / 2;
    for (uint64_t p0 = (uint64_t)min_period + (uint64_t)blockIdx.x * DI_THREADS; p0 <= most; p0 += (uint64_t)gridDim.x * DI_THREADS) {
        const uint64_t p = p0 + tid;
        if (p <= most && halves_hash_alike(Q, M, (uint32_t)p, pow_base((uint32_t)p))) atomicMin(&S->candidate, (uint32_t)p);
    }
    wait_stores();
    __syncthreads();
    if (tid == 0) {
        __threadfence();
        s_last = atomicAdd(&S->searched, 1u) + 1 == gridDim.x ? 1u : 0u;
    }
    __syncthreads();
    if (!s_last) return;
    const uint32_t c = atomicMin(&S->candidate, DI_NONE);
    const uint32_t p = c == DI_NONE ? 0 : search_from(tok, Q, M, c);
    if (tid == 0) *period = p;
}

hipError_t launch_detect_iteration(const uint64_t *tokens, uint32_t M, uint32_t min_period, uint64_t *Q,
                                   uint64_t *totals, uint32_t *period, hipStream_t st)
{
    if (M <= DI_ONE) {
        hipLaunchKernelGGL(k_detect_short, dim3(1), dim3(DI_THREADS), 0, st, tokens, M, min_period, Q, period);
        return hipGetLastError();
    }
    // tiles of at least 1024 tokens (four steps of a wave), at most DI_TILES of them
    uint32_t tile = 4 * DI_CHUNK;
    if ((M - 1) / tile + 1 > DI_TILES) tile = ((M - 1) / DI_TILES / DI_CHUNK + 1) * DI_CHUNK;
    const uint32_t nt = (M - 1) / tile + 1;
    const uint32_t cands = M / 2 >= min_period ? M / 2 - min_period + 1 : 0;
    uint32_t n_lists = cands ? (cands - 1) / (256 * DI_SPAN) + 1 : 1;
    n_lists = n_lists < DI_LISTS ? n_lists : DI_LISTS;
    const uint32_t cb = (M - 1) / (4 * DI_THREADS) + 1, blocks = cb < 256 ? cb : 256;
    DiScratch *S = (DiScratch *)totals;
    hipLaunchKernelGGL(k_detect_suffix, dim3(n_lists), dim3(256), 0, st, tokens, M, min_period, S);
    hipLaunchKernelGGL(k_detect_compare, dim3(blocks), dim3(DI_THREADS), 0, st, tokens, M, S, n_lists, period);
    hipLaunchKernelGGL(k_detect_hash, dim3(blocks), dim3(DI_THREADS), 0, st, tokens, M, min_period, tile, nt, S, Q, period);
    return hipGetLastError();
}

}  // namespace lap
