// Iteration detection on a recorded request stream (Section V): the list ends with two equal
// consecutive subsequences of length p; the smallest such p (>= min_period) is reported.
//
// First the direct way.  Every distance p is looked at: whether the last p tokens end as the p before them (nearly every one is
// refused by its last token, so half of the list is read once).  A workgroup goes on with the smallest distances that
// remain of its own, where these are many only with those that start alike as well: a wave compares up to DI_DEEP tokens of
// each, which refuses most of what a repeated piece inside an iteration leaves, and settles short repeats.  The DI_FEW smallest that
// are still open and below the smallest that is settled are then compared element by element by all workgroups, the last
// of which has the answer -- unless all of them differ and there are more.  Then the places where they differ refuse most of the
// others, and up to DI_LEFT that remain are compared in the same way.  Only where more do it comes to hashes, whose cost does
// not depend on what is in the list: a polynomial hash of every prefix (mod 2^64, odd base) is built with a scan; the two
// halves of a candidate p then compare in O(1):
//     (P[M-p] - P[M-2p]) * r^p == P[M] - P[M-p]
// and the smallest candidate whose hashes agree is checked element by element (hashes mod 2^64 can
// collide, the answer never depends on them); if the check fails the search resumes behind it.
//
// Short lists (up to DI_ONE requests) are one workgroup's work in one launch, which refuses distances by places until none is left.
// Longer ones take three, the last of which nearly always finds nothing to do.  us of calls that follow each other, by
// hashes at once, and now:
//     requests                                             6144        40 000       2 000 003
//     an iteration                                         21.6   9.2   22.2  14.1   38.5  15.2
//     iterations that end in a run, or in equal layers     21.5   9.3   22.5  18.1   38.4  24.4
//     a run of a short period, too short to be asked for   19.0   9.0   20.9  16.8   33.3  22.5
//     one of it that is asked for                          20.5  14.8   54.3  20.6  127    30.4
//     a list of a short period with single other tokens    20.5  24     22    49     36   114
//     a Fibonacci word, where it comes to hashes           19.0  12.2   21.1  69     32   220
// The last two are slower than by hashes at once: many distances are looked at in vain, and a hand-over between workgroups writes
// the caches back.  An iteration in a list of 2 000 003 that no cache holds yet: 50 and 29.
#include "lap_dev.h"
#include "lap_kernels.h"

namespace lap {

constexpr int DI_THREADS = 1024;
constexpr int DI_WAVES = DI_THREADS / WAVE;
constexpr uint64_t DI_BASE = 0x9E3779B97F4A7C15ull | 1ull;
constexpr uint32_t DI_NONE = 0xFFFFFFFFu;
constexpr uint32_t DI_CHUNK = 4 * WAVE;        // tokens a wave takes per step: 4 neighbours per lane
constexpr uint32_t DI_DEEP = 1024;             // tokens that a distance has to agree in to be compared by all
constexpr uint32_t DI_FEW = 4, DI_LEFT = 8;    // distances that are compared by all workgroups, at most: first, and of those left
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

// The first looks at distance p (2 p <= M): whether the p tokens before the last p end, and start, as these do.  The end is read by
// neighbouring lanes anyway.  The start refuses what a run of a short period at the end of the list leaves: a distance
// that is shorter than the run and longer than half of it reaches out of the run there.
template <bool START>
__device__ __forceinline__ bool alike(const uint64_t *__restrict__ tok, uint32_t M, uint32_t p)
{
    uint64_t differ = 0;
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {                   // (at once: a wave waits for each round)
        const uint32_t e = START ? M - p + min(k, p - 1) : M - min(k + 1, p);
        differ |= tok[e] ^ tok[e - p];
    }
    return differ == 0;
}
__device__ __forceinline__ bool ends_alike(const uint64_t *__restrict__ tok, uint32_t M, uint32_t p)
{
    return alike<false>(tok, M, p) && alike<true>(tok, M, p);
}

// What a wave finds out about distance p from its last `deep` tokens; at: one that differs from the one p before it
enum { DI_DIFFERS, DI_OPEN, DI_SAME };
__device__ __forceinline__ uint32_t look_deep(const uint64_t *__restrict__ tok, uint32_t M, uint32_t p, uint32_t deep, uint32_t &at)
{
    constexpr uint32_t STEP = 4 * WAVE;
    const uint32_t most = min(p, deep);
    for (uint32_t j = 1 + (uint32_t)lane_id(); ballot(j <= most); j += STEP) {
        uint64_t differ[4];                              // (read at once, looked at one by one only if there is a reason)
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t e = M - min(j + k * WAVE, most);
            differ[k] = tok[e] ^ tok[e - p];
        }
        const uint64_t who = ballot((differ[0] | differ[1] | differ[2] | differ[3]) != 0);
        if (who) {
            const uint32_t k = differ[0] ? 0 : differ[1] ? 1 : differ[2] ? 2 : 3;
            at = read_lane(M - min(j + k * WAVE, most), __builtin_ctzll(who));
            return DI_DIFFERS;
        }
    }
    return most == p ? DI_SAME : DI_OPEN;
}

// Where one distance differs others mostly do: those of a run differ in what comes before it, nearly equal pieces in what is not
// equal.  Whether the token x at place w is also found at distance p, before or behind it, if it is among the last 2 p.
__device__ __forceinline__ bool place_repeats(const uint64_t *__restrict__ tok, uint32_t M, uint32_t p, uint32_t w, uint64_t x)
{
    const uint32_t back = M - w;                         // (2 p <= M)
    return tok[back > 2 * p ? w : back > p ? w + p : w - p] == x;
}

__global__ __launch_bounds__(DI_THREADS) void k_detect_short(const uint64_t *__restrict__ tok, uint32_t M,
                                                             uint32_t min_period, uint32_t *__restrict__ period)
{
    __shared__ uint32_t s_bits[2 * WAVE], s_list[DI_WAVES], s_at[DI_WAVES], s_found, s_same;
    static_assert(DI_ONE / 2 < 2 * WAVE * 32, "a bit per distance");
    const uint32_t tid = threadIdx.x, lane = tid & (WAVE - 1), wave = tid / WAVE;
    if (tid < 2 * WAVE) s_bits[tid] = 0;
    if (tid == 0) s_same = DI_NONE;
    __syncthreads();
    const uint64_t last = tok[M - 1];
    for (uint32_t p = min_period + tid; p >= min_period && p <= M / 2; p += DI_THREADS)
        if (tok[M - 1 - p] == last && ends_alike(tok, M, p)) atomicOr(&s_bits[p / 32], 1u << (p % 32));
    for (;;) {                                             // each turn leaves out the distances that it has looked at
        __syncthreads();
        if (wave == 0) {                                   // the smallest of them, in ascending order
            uint64_t bits = (uint64_t)s_bits[2 * lane + 1] << 32 | s_bits[2 * lane];
            const uint32_t own = (uint32_t)__popcll(bits);
            uint32_t at = own;
            for (int d = 1; d < WAVE; d <<= 1) { const uint32_t y = (uint32_t)__shfl_up((int)at, d, WAVE); if ((int)lane >= d) at += y; }
            if (lane == WAVE - 1) s_found = at;
            for (at -= own; bits && at < DI_WAVES; bits &= bits - 1, ++at) s_list[at] = lane * 64 + (uint32_t)__ffsll((unsigned long long)bits) - 1;
        }
        __syncthreads();
        const uint32_t found = s_found, look = min(found, (uint32_t)DI_WAVES);
        if (wave < look) {
            uint32_t at = 0;
            const uint32_t p = s_list[wave], what = look_deep(tok, M, p, M, at);
            if (lane == 0) {
                s_at[wave] = at;
                if (what == DI_SAME) atomicMin(&s_same, p);
                else atomicAnd(&s_bits[p / 32], ~(1u << (p % 32)));
            }
        }
        __syncthreads();
        if (s_same != DI_NONE || found <= look) {
            if (tid == 0) *period = s_same != DI_NONE ? s_same : 0;
            return;
        }
        // the others where those differed (all of them did)
#pragma unroll 1
        for (uint32_t p = min_period + tid; p >= min_period && p <= M / 2; p += DI_THREADS) {
            bool stays = (s_bits[p / 32] >> (p % 32)) & 1;
            if (!stays) continue;
#pragma unroll 1
            for (uint32_t q = 0; q < DI_WAVES && stays; ++q) {
                const uint32_t w = s_at[q], v = w - s_list[q];
                stays = place_repeats(tok, M, p, w, tok[w]) && place_repeats(tok, M, p, v, tok[v]);
            }
            if (!stays) atomicAnd(&s_bits[p / 32], ~(1u << (p % 32)));
        }
    }
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
    uint32_t done, more, top;                  // workgroups that have compared; whether that was not all, up to which distance
    uint32_t at[DI_FEW];                       // 1 + the last of the distance's tokens that differs from the one before, 0: none
    uint32_t places[2 * DI_FEW];               // where those are in the list, and the ones that they differ from
    uint32_t n_left, left[DI_LEFT], differs[DI_LEFT], checked;           // distances that are left, and which of them differ; workgroups that have compared
    uint32_t next[3], ready[3];                // tiles given out and finished: distances, totals, hashes
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
        S->done = 0; S->more = 0;
        for (uint32_t q = 0; q < DI_FEW; ++q) S->at[q] = 0;
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
        uint32_t hits = 0;
#pragma unroll
        for (uint32_t k = 0; k < DI_SPAN; ++k) hits |= x[k] == last && base + k * 256 + tid <= most ? 1u << k : 0u;
        // (few lanes have one: the longer look once in the code, not once for each of them)
#pragma unroll 1
        for (; hits; hits &= hits - 1) {
            const uint32_t at = (uint32_t)__builtin_ctz(hits) * 256 + tid;
            if (alike<false>(tok, M, (uint32_t)base + at)) {
                atomicOr(&s_bits[at / 32], 1u << (at % 32));
                s_found = 1;
            }
        }
        __syncthreads();
        if (!s_found) continue;
        static_assert(SPAN / 32 == WAVE, "");
        for (bool again = false;; again = true) {
            if (wave == 0) {                               // the smallest of them, in ascending order
                uint32_t bits = s_bits[lane];
                const uint32_t own = (uint32_t)__popc(bits);
                uint32_t at = own;
                for (int d = 1; d < WAVE; d <<= 1) { const uint32_t y = (uint32_t)__shfl_up((int)at, d, WAVE); if ((int)lane >= d) at += y; }
                if (lane == WAVE - 1) s_found = at;
                for (at -= own; bits && at < DEEP + DI_FEW; bits &= bits - 1, ++at)
                    s_list[at] = (uint32_t)base + lane * 32 + (uint32_t)__ffs((int)bits) - 1;
            }
            __syncthreads();
            if (again || s_found <= DEEP) break;
            // too many to look at: those whose starts differ go
#pragma unroll 1
            for (uint32_t at = tid; at < SPAN; at += 256)
                if (((s_bits[at / 32] >> (at % 32)) & 1) && !alike<true>(tok, M, (uint32_t)base + at)) atomicAnd(&s_bits[at / 32], ~(1u << (at % 32)));
            __syncthreads();
        }
        const uint32_t found = s_found, look = min(found, DEEP);
        for (uint32_t q = wave; q < look; q += 4) {
            uint32_t at;
            const uint32_t what = look_deep(tok, M, s_list[q], DI_DEEP, at);
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
    __shared__ uint32_t s_best, s_list[DI_FEW + 1], s_at[DI_FEW], s_more, s_last;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) { s_best = DI_NONE; s_more = 0; }
    if (tid < DI_FEW) s_at[tid] = 0;
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
    for (uint32_t q = 0; q < found; ++q) {
        const uint32_t c = s_list[q];
        uint32_t at = 0;
#pragma unroll 4
        for (uint64_t i = (uint64_t)blockIdx.x * DI_THREADS + tid; i < c; i += (uint64_t)gridDim.x * DI_THREADS)
            at = tok[M - 2 * c + (uint32_t)i] != tok[M - c + (uint32_t)i] ? (uint32_t)i + 1 : at;
        at = wave_scan_max_u32(at);
        if (lane_id() == WAVE - 1 && at) atomicMax(&s_at[q], at);
    }
    __syncthreads();
    if (tid == 0) {
        for (uint32_t q = 0; q < found; ++q)
            if (s_at[q]) atomicMax(&S->at[q], s_at[q]);
        __threadfence();
        s_last = atomicAdd(&S->done, 1u) + 1 == gridDim.x ? 1u : 0u;
    }
    __syncthreads();
    if (s_last && tid == 0) {
        __threadfence();
        uint32_t p = best;
        for (uint32_t q = found; q-- > 0;) {
            const uint32_t at = atomicMax(&S->at[q], 0u);
            if (!at) p = s_list[q];
            S->places[2 * q] = M - s_list[q] + at - 1;
            S->places[2 * q + 1] = M - 2 * s_list[q] + at - 1;
        }
        if (s_more && p == best) {                         // (all DI_FEW of them differ)
            S->more = 1; S->top = min(best, M / 2);
            S->n_left = 0; S->checked = 0; S->candidate = DI_NONE; S->searched = 0;
            for (uint32_t q = 0; q < DI_LEFT; ++q) S->differs[q] = 0;
            for (int k = 0; k < 3; ++k) S->next[k] = S->ready[k] = 0;
        }
        *period = p == DI_NONE ? 0 : p;
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

// the workgroup's next `take` tiles (a counter for single waves took 0.2 ms: the chip adds to one address one after the other)
__device__ __forceinline__ uint32_t next_tiles(uint32_t *next, uint32_t take, uint32_t *s_next)
{
    __syncthreads();
    if (threadIdx.x == 0) *s_next = atomicAdd(next, take);
    __syncthreads();
    return *s_next;
}

// What is left: the distances that repeat what the DI_FEW did not, of which a few are compared by all workgroups.  Else the hashes:
// the totals of tiles of `tile` tokens (a multiple of DI_CHUNK), the hash of every prefix, the candidates; the last workgroup to
// finish checks the smallest.  A workgroup takes tiles from a counter, so what others wait for is held by one that runs
// already, and every wait ends.
__global__ __launch_bounds__(DI_THREADS) void k_detect_left(const uint64_t *__restrict__ tok, uint32_t M, uint32_t min_period,
                                                            uint32_t tile, uint32_t n_tiles, DiScratch *S, uint64_t *Q,
                                                            uint32_t *__restrict__ period)
{
    __shared__ uint32_t s_last, s_sum, s_next;
    if (!S->more) return;
    const uint32_t lane = threadIdx.x & (WAVE - 1), tid = threadIdx.x;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / WAVE));
    const bool vec = ((uintptr_t)tok & 15) == 0;
    const uint64_t last = tok[M - 1];
    uint32_t places[2 * DI_FEW];
    uint64_t tokens[2 * DI_FEW];
#pragma unroll
    for (uint32_t q = 0; q < 2 * DI_FEW; ++q) { places[q] = S->places[q]; tokens[q] = tok[places[q]]; }
    const uint32_t top = S->top, n_spans = (top - min_period) / DI_THREADS + 1;
    uint32_t mine = 0;
    for (uint32_t t0 = next_tiles(&S->next[0], 4, &s_next); t0 < n_spans; t0 = next_tiles(&S->next[0], 4, &s_next)) {
        for (uint32_t t = t0; t < min(n_spans, t0 + 4); ++t, mine += wave == 0) {
            const uint64_t p = (uint64_t)min_period + (uint64_t)t * DI_THREADS + tid;
            bool stays = p <= top && tok[M - 1 - (uint32_t)p] == last && ends_alike(tok, M, (uint32_t)p);
            if (stays) {
#pragma unroll
                for (uint32_t q = 0; q < 2 * DI_FEW; ++q) stays &= place_repeats(tok, M, (uint32_t)p, places[q], tokens[q]);
            }
            const uint64_t who = ballot(stays);
            if (!who) continue;
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&S->n_left, (uint32_t)__popcll(who));
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(who & ((1ull << lane) - 1));
            if (stays && at < DI_LEFT) S->left[at] = (uint32_t)p;
        }
    }
    wait_tiles(&S->ready[0], mine, n_spans, &s_sum);
    const uint32_t left = __hip_atomic_load(&S->n_left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (left <= DI_LEFT) {
        for (uint32_t q = 0; q < left; ++q) {
            const uint32_t c = S->left[q];
            bool bad = false;
#pragma unroll 4
            for (uint64_t i = (uint64_t)blockIdx.x * DI_THREADS + tid; i < c; i += (uint64_t)gridDim.x * DI_THREADS)
                bad |= tok[M - 2 * c + (uint32_t)i] != tok[M - c + (uint32_t)i];
            if (__syncthreads_or(bad ? 1 : 0) && tid == 0) atomicOr(&S->differs[q], 1u);
        }
        if (tid != 0) return;
        __threadfence();
        if (atomicAdd(&S->checked, 1u) + 1 != gridDim.x) return;
        __threadfence();
        uint32_t p = DI_NONE;
        for (uint32_t q = 0; q < left; ++q)
            if (!atomicOr(&S->differs[q], 0u)) p = min(p, S->left[q]);
        *period = p == DI_NONE ? 0 : p;
        return;
    }
    mine = 0;
    for (uint32_t t0 = next_tiles(&S->next[1], DI_WAVES, &s_next); t0 < n_tiles; t0 = next_tiles(&S->next[1], DI_WAVES, &s_next)) {
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
    wait_tiles(&S->ready[1], mine, n_tiles, &s_sum);
    mine = 0;
    for (uint32_t t0 = next_tiles(&S->next[2], DI_WAVES, &s_next); t0 < n_tiles; t0 = next_tiles(&S->next[2], DI_WAVES, &s_next)) {
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
    wait_tiles(&S->ready[2], mine, n_tiles, &s_sum);
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
        hipLaunchKernelGGL(k_detect_short, dim3(1), dim3(DI_THREADS), 0, st, tokens, M, min_period, period);
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
    hipLaunchKernelGGL(k_detect_left, dim3(blocks), dim3(DI_THREADS), 0, st, tokens, M, min_period, tile, nt, S, Q, period);
    return hipGetLastError();
}

}  // namespace lap
