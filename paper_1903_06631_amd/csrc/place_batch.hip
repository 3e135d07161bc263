// First-fit placement of every variable under many orderings (Section III-C), in batches: up to 64 variables of an ordering
// are placed at a time.
//
// One workgroup works on one ordering.  Its placed blocks are sorted by offset, as offset, end and lifetime (16 + 16 bits) in
// three arrays; the entries behind the last block have the highest offset and meet nothing.  The arrays lie in LDS up to
// 13 311 variables, else in global memory.
//
// A batch is the next variables in rank order.
//   ask      Each of them is taken by one wave, which goes through the blocks placed so far in rows of 512, eight entries a
//            lane: entries that do not meet the variable in time are masked, a prefix maximum of the remaining ends gives
//            the highest occupied address so far, and an entry whose offset leaves `size` free above it shows a hole.
//            The wave notes the first hole and the next one of the same row.  The answers do not know of each other.
//            Where the arrays lie in global memory, their rows come to the LDS some at a time, the next ones on their way
//            while these are looked at, and the variables of one lifetime share the question.
//   compare  Which others of the batch a variable meets in time, and whether an earlier one of them is in its way.
//   settle   One wave makes the answers what they would be one after the other.  An answer that nothing is in the way of
//            stands: more blocks take places away and never give one.  Where something is, everything below the answer stays
//            refused all the same, so the variable moves up behind the block in its way, as often as need be; if it still
//            ends inside the hole that it was shown, or else in the next one, that is its place.  The batch ends before
//            the first variable whose place is not known; the first one's always is.
//   insert   The blocks enter the three arrays together: where each belongs is searched for, then every entry moves up by
//            the number of new blocks below it, read by all waves, written by all waves, from the top down in as many
//            rounds as the registers need.
// Measured: 193 orderings of a residual chain of 9001 variables 4.9 ms (in registers, one variable a round of two barriers,
// 11.2), 256 of 3000 1.2 (2.4), of 13 000 8.3 (19.6), of 20 000 14.4 (38.2), of 32 767 32 (98), of 50 000 65 (848 by segment
// lists), 4096 of them 811 (1114).  Without the shared questions 50 000 took 77; in LDS sharing does not pay (9001: 9.9).
// What bounds it: the vector instructions of the questions, 60 for a row of 512 entries (two thirds of the time of 9001
// variables; at 50 000 a batch asks 1540 rows, of 2450 if every lifetime asked all of them, 38 of its 83 us), the waits where a
// chunk's lifetimes do not come out even over the waves (22 us), and one variable after the other where a batch is settled,
// 200 cycles each (half of the time where all variables of a step follow each other).  A second ordering on the compute unit
// fills those waits.  Rows that every wave reads for itself, four lifetimes at a time, took as long under one ordering a unit and
// read them 2.5 times over (4096 orderings: 5.3 TB/s; 948 ms).  Where holes take one variable each and sizes are few, an order
// that follows the trace fills a batch with 5 to 8 variables only, and the registers are faster (batches_lose).
#include "block_rows.h"
#include "lap_kernels.h"

namespace lap {

namespace {

constexpr uint32_t AHEAD = 2 * WAVE;           // ranks whose records are in LDS: the 64 that are being placed and the next 64
constexpr uint32_t BATCH_LDS = 4096;           // bytes of LDS beside the blocks, at most
constexpr uint32_t BATCH = WAVE;               // variables a batch: lanes stand for them
// Where a batch was cut short before that many variables, the next ones have no more, and each is shown further holes, of further
// rows as well
constexpr uint32_t FEW = 16, FEW_HOLES = BATCH / FEW;
constexpr int E = 8;                           // entries a lane of a row
constexpr uint32_t ROWE = E * WAVE;

struct BatchArgs {
    uint32_t n, cap;             // cap: entries of the three arrays
    const uint4 *vrec;           // [n] (first step, end of life, size in granules, -)
    const uint32_t *perm;        // [B][n]
    PlanHeader *hdr;
    uint32_t *blocks;            // [B][4 n] the three arrays where they do not fit the LDS
    uint64_t *offs;              // [B][n] in rank order
    uint64_t *fps;               // [B]
    uint64_t *ticks;             // [B] duration of every ordering in timer ticks
};

__device__ __forceinline__ uint32_t bound_of(uint32_t life) { return life_bound(life & 0xFFFFu, 0xFFFFu - (life >> 16)); }
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint32_t first_lane(uint64_t m) { return (uint32_t)__builtin_ctzll(m); }

// a lane's entries of a row, as Row (block_rows.h)
struct Entries {
    uint32_t off[E], end[E], life[E];
    __device__ __forceinline__ void load(const uint32_t *o, const uint32_t *e, const uint32_t *f, uint32_t row)
    {
        const uint32_t i = (row * WAVE + (uint32_t)lane_id()) * E;
#pragma unroll
        for (int j = 0; j < E; j += 4) {
            const uint4 x = *(const uint4 *)(o + i + j), y = *(const uint4 *)(e + i + j), z = *(const uint4 *)(f + i + j);
            off[j] = x.x; off[j + 1] = x.y; off[j + 2] = x.z; off[j + 3] = x.w;
            end[j] = y.x; end[j + 1] = y.y; end[j + 2] = y.z; end[j + 3] = y.w;
            life[j] = z.x; life[j + 1] = z.y; life[j + 2] = z.z; life[j + 3] = z.w;
        }
    }
    // arrays `stride` words apart, in which a row has the first half of every lane's entries before the second
    __device__ __forceinline__ void load_halves(const uint32_t *o, uint32_t stride, uint32_t row)
    {
        const uint32_t i = row * ROWE + (uint32_t)lane_id() * 4;
#pragma unroll
        for (int j = 0; j < E; j += 4) {
            const uint4 x = *(const uint4 *)(o + i + j * WAVE), y = *(const uint4 *)(o + stride + i + j * WAVE),
                        z = *(const uint4 *)(o + 2 * stride + i + j * WAVE);
            off[j] = x.x; off[j + 1] = x.y; off[j + 2] = x.z; off[j + 3] = x.w;
            end[j] = y.x; end[j + 1] = y.y; end[j + 2] = y.z; end[j + 3] = y.w;
            life[j] = z.x; life[j + 1] = z.y; life[j + 2] = z.z; life[j + 3] = z.w;
        }
    }
};

// the ends of the entries that meet the variable, and their inclusive prefix maximum over the lanes
__device__ __forceinline__ uint32_t batch_ends(const Entries &R, uint32_t bound, uint32_t (&e)[E])
{
    uint32_t m = 0;
#pragma unroll
    for (int j = 0; j < E; ++j) { e[j] = life_meets(R.life[j], bound) ? R.end[j] : 0u; m = max(m, e[j]); }
    return wave_scan_max_u32(m);
}

// as row_holes (block_rows.h)
__device__ __forceinline__ void batch_holes(const Entries &R, const uint32_t (&e)[E], uint32_t incl, uint32_t P,
                                                             uint32_t (&before)[E], uint32_t (&free_)[E])
{
    before[0] = max(P, shift_in_zero(incl));
#pragma unroll
    for (int j = 1; j < E; ++j) before[j] = max(before[j - 1], e[j - 1]);
#pragma unroll
    for (int j = 0; j < E; ++j) free_[j] = __builtin_elementwise_sub_sat(R.off[j], before[j]);
}

// the offset of the row's first neighbour at or above `from` (entries below a hole that starts at `at` start below at + s), or
// NOTHING
__device__ __forceinline__ uint32_t first_neighbour(const Entries &R, const uint32_t (&e)[E], uint32_t from)
{
    // offsets below `from` wrap to more than any above it
    uint32_t d = NOTHING;
#pragma unroll
    for (int j = 0; j < E; ++j) d = min(d, e[j] != 0 ? R.off[j] - from : NOTHING);
    const uint64_t any = ballot(d < 0u - from);
    return any ? from + read_lane(d, first_lane(any)) : NOTHING;
}

// The first hole of a row that shows one, and the next one of the row (end 0: there is none)
__device__ __forceinline__ void row_answer(const Entries &R, const uint32_t (&e)[E], const uint32_t (&before)[E],
                                           const uint32_t (&free_)[E], uint64_t any, uint32_t s, uint32_t &at, uint32_t &hole, uint2 &next)
{
    uint32_t x = before[E - 1];
#pragma unroll
    for (int j = E - 2; j >= 0; --j) x = pick(free_[j] >= s, before[j], x);
    at = read_lane(x, first_lane(any));
    // it ends at the first neighbour behind it, or at the row's last entry at least
    const uint32_t end = read_lane(R.off[E - 1], WAVE - 1);
    hole = min(first_neighbour(R, e, at + s), end);
    // the next one: a lane's highest address so far where it shows a hole behind the first
    x = NOTHING;
#pragma unroll
    for (int j = E - 1; j >= 0; --j) x = pick(free_[j] >= s && before[j] > at, before[j], x);
    const uint64_t more = ballot(x != NOTHING);
    if (more) {
        const uint32_t at2 = read_lane(x, first_lane(more));
        next = make_uint2(at2, min(first_neighbour(R, e, at2 + s), end));
    }
}

// NW waves an ordering, which move RPW rows of 256 each at once; NEAR: the three arrays lie in LDS, else in global memory
template <int NW, int RPW, bool NEAR>
__global__ __launch_bounds__(NW *WAVE, 4) void k_place_batch(BatchArgs A)
{
    // (read 16 bytes a lane: eight times slower where it only starts at a multiple of 8)
    extern __shared__ __attribute__((aligned(16))) uint32_t s_blocks[];
    __shared__ uint2 s_rec[AHEAD];                         // lifetime, size of the ranks ahead, at rank % AHEAD
    __shared__ uint4 s_ask[BATCH];                         // start of the hole, size, lifetime, end of the hole
    __shared__ uint2 s_next[BATCH];                        // start and end of the next holes (0: no further one)
    __shared__ uint64_t s_meets[BATCH];                    // the variables of the batch that meet this one; before: that have its lifetime, not answered
    __shared__ uint2 s_state[BATCH];                       // per lifetime: highest address so far, smallest size not answered
    __shared__ uint32_t s_open[2], s_done[4];              // bits: the first variable of every lifetime; those that are answered, by chunk
    // bits: the variables with an earlier one in their way, and those that are in the way
    __shared__ uint32_t s_hit[4], s_task, s_acc, s_fp;
    static_assert(sizeof(s_rec) + sizeof(s_ask) + sizeof(s_next) + sizeof(s_meets) + sizeof(s_hit) + sizeof(s_state) + sizeof(s_open) + sizeof(s_done) + 12 <= BATCH_LDS, "");
    static_assert((PLAN_BATCH_LDS_VARS / ROWE + 1) * ROWE * 12 + BATCH_LDS <= 160 * 1024, "");
    uint2 *const s_pos = s_next;                           // where a new block goes: entries below it, and its index

    const uint32_t b = blockIdx.x;
    if (!A.hdr->fast || A.hdr->mode1 || A.hdr->mode2 == 1) return;
    // the sweep, which comes after this and leaves only traces of fewer variables to others by itself, has to know
    if (A.n > PLAN_REG_MAX_VARS && b == 0 && threadIdx.x == 0) A.hdr->mode2 = 2;
    const long long t_begin = wall_clock64();
    const uint32_t n = A.n, sh = A.hdr->shift, cap = A.cap;
    uint32_t *s_off;
    if constexpr (NEAR) s_off = s_blocks;
    else s_off = A.blocks + (size_t)b * 4 * n;
    uint32_t *const s_end = s_off + cap, *const s_life = s_off + 2 * cap;
    const uint32_t l = (uint32_t)lane_id(), tid = threadIdx.x;
    const uint32_t wave = uniform(tid / WAVE);
    const uint32_t *perm = A.perm + (size_t)b * n;
    uint64_t *offs = A.offs + (size_t)b * n;

    for (uint32_t i = tid; i < cap; i += NW * WAVE) { s_off[i] = NOTHING; s_end[i] = NOTHING; s_life[i] = NOTHING; }
    if (tid < AHEAD && tid < n) {
        const uint4 v = A.vrec[perm[tid]];
        s_rec[tid] = make_uint2(life_word(v.x, v.y), v.z);
    }
    if (tid == 0) { s_fp = 0; s_task = NW; }
    if (tid < 4) s_hit[tid] = 0;
    if (tid < 2) s_open[tid] = 0;
    if (tid < 4) s_done[tid] = 0;
    // one wave fetches the records of the ranks to come: those of the next 64 and the variable numbers of the 64 after
    const bool fetches = wave == NW - 1;
    uint4 rec_next = make_uint4(0u, 1u, 1u, 0u);
    uint32_t v_next = 0;
    if (fetches) {
        if (l + 2 * WAVE < n) rec_next = A.vrec[perm[l + 2 * WAVE]];
        if (l + 3 * WAVE < n) v_next = perm[l + 3 * WAVE];
    }
    __syncthreads();

    constexpr uint32_t CHUNK = NW * WAVE * 4 / ROWE;       // rows that come to the LDS at a time: four entries a thread
    uint32_t fp = 0;
    uint32_t most = BATCH, few = 0, cut = 0;               // variables of the next batch; batches to come of few, cut short one after the other
    for (uint32_t r = 0, turn = 0; r < n; ++turn) {        // r ranks are placed
        const uint32_t lim = min(few ? FEW : most, n - r), others = few ? FEW_HOLES : 1u;
        // ---- ask
        if (!NEAR && !few) {
            // The rows come through the LDS, CHUNK at a time, the next ones on their way while these are looked at.  Variables of
            // one lifetime ask together; the lifetimes that are not answered yet are dealt to the waves anew for every chunk.
            const uint32_t last = r / ROWE;
            uint4 xo, xe, xl;
            auto fetch = [&](uint32_t c) {
                const uint32_t i = c * CHUNK * ROWE + 4 * tid;
                if (i < cap) { xo = *(const uint4 *)(s_off + i); xe = *(const uint4 *)(s_end + i); xl = *(const uint4 *)(s_life + i); }
            };
            auto put = [&](uint32_t c) {                   // (a lane's first and last four entries apart: no two lanes meet in a bank)
                uint4 *const to = (uint4 *)(s_blocks + c % 2 * 3 * CHUNK * ROWE) + tid / 128 * 128 + tid % 2 * 64 + tid % 128 / 2;
                to[0] = xo; to[CHUNK * ROWE / 4] = xe; to[2 * CHUNK * ROWE / 4] = xl;
            };
            fetch(0);
            const uint32_t life = l < lim ? s_rec[(r + l) % AHEAD].x : NOTHING;
            uint64_t first = 0;
#pragma unroll
            for (uint32_t q = 0; q < BATCH / NW; ++q) {
                if (q * NW >= lim) break;
                const uint32_t v = q * NW + wave;
                const uint64_t m = v < lim ? ballot(l < lim && life == read_lane(life, v)) : 0;
                if (l == v) { s_meets[v] = m; s_state[v] = make_uint2(0, 0); }
                first |= m && first_lane(m) == v ? 1ull << v : 0;
            }
            if (first && l < 2) atomicOr(&s_open[l], (uint32_t)(first >> (32 * l)));
            put(0);
            __syncthreads();
            uint64_t open = ((uint64_t)uniform(s_open[1]) << 32) | uniform(s_open[0]);
            for (uint32_t c = 0;; ++c) {
                const bool more = (c + 1) * CHUNK <= last;
                if (more) fetch(c + 1);
                const uint32_t *const buf = s_blocks + c % 2 * 3 * CHUNK * ROWE;
                uint64_t mine = ballot(((open >> l) & 1) && (uint32_t)__popcll(open & ((1ull << l) - 1)) % NW == wave);
                for (; mine; mine &= mine - 1) {
                    const uint32_t v = first_lane(mine), lf = uniform(s_rec[(r + v) % AHEAD].x), bound = bound_of(lf);
                    const uint64_t has = s_meets[v];
                    uint64_t left = ((uint64_t)uniform((uint32_t)(has >> 32)) << 32) | uniform((uint32_t)has);
                    const uint2 state = s_state[v];
                    uint32_t P = uniform(state.x), least = uniform(state.y);
                    const uint32_t rows = min(CHUNK, last + 1 - c * CHUNK);
                    for (uint32_t i = 0; i < rows && left; ++i) {
                        Entries R;
                        R.load_halves(buf, CHUNK * ROWE, i);
                        uint32_t e[E], before[E], free_[E];
                        const uint32_t incl = batch_ends(R, bound, e);
                        batch_holes(R, e, incl, P, before, free_);
                        uint32_t f = free_[0];
#pragma unroll
                        for (int j = 1; j < E; ++j) f = max(f, free_[j]);
                        if (ballot(f >= least)) {
                            // those whose size it takes are answered; the smallest size of the others
                            least = NOTHING;
                            for (uint64_t m = left; m; m &= m - 1) {
                                const uint32_t k = first_lane(m), s = uniform(s_rec[(r + k) % AHEAD].y);
                                const uint64_t any = ballot(f >= s);
                                if (any) {
                                    uint32_t at, hole;
                                    uint2 next = make_uint2(0, 0);
                                    row_answer(R, e, before, free_, any, s, at, hole, next);
                                    if (l == 0) { s_ask[k] = make_uint4(at, s, lf, hole); s_next[k] = next; }
                                    left &= ~(1ull << k);
                                } else least = min(least, s);
                            }
                        }
                        P = max(P, read_lane(incl, WAVE - 1));
                    }
                    if (l == 0) {
                        s_meets[v] = left;
                        s_state[v] = make_uint2(P, least);
                        if (!left) atomicOr(&s_done[c % 2 * 2 + v / 32], 1u << v % 32);
                    }
                }
                if (!more) break;
                put(c + 1);
                __syncthreads();
                // (the next chunk's go to the other two words, which all have read by now)
                open &= ~(((uint64_t)uniform(s_done[c % 2 * 2 + 1]) << 32) | uniform(s_done[c % 2 * 2]));
                if (!open) break;
            }
        } else
        for (uint32_t v = wave, v_after; v < lim; v = uniform(v_after)) {
            v_after = l == 0 ? atomicAdd(&s_task, 1u) : 0;
            const uint2 rec = s_rec[(r + v) % AHEAD];
            const uint32_t lf = uniform(rec.x), s = uniform(rec.y), bound = bound_of(lf);
            const uint32_t last = r / ROWE;                // the row of the first entry not in use, which shows a hole
            uint32_t P = 0, at = 0, at0 = 0, hole0 = 0;
            if (!few) {
                uint2 next = make_uint2(0, 0);
                for (uint32_t i = 0; i <= last; ++i) {
                    Entries R;
                    R.load(s_off, s_end, s_life, i);
                    uint32_t e[E], before[E], free_[E];
                    const uint32_t incl = batch_ends(R, bound, e);
                    batch_holes(R, e, incl, P, before, free_);
                    uint32_t f = free_[0];
#pragma unroll
                    for (int j = 1; j < E; ++j) f = max(f, free_[j]);
                    const uint64_t any = ballot(f >= s);
                    if (any) {
                        row_answer(R, e, before, free_, any, s, at0, hole0, next);
                        break;
                    }
                    P = max(P, read_lane(incl, WAVE - 1));
                }
                if (l == 0) s_next[v] = next;
            } else {
                uint32_t found = 0;
                bool open = false;                             // the end of the hole at `at` is not known yet
                for (uint32_t i = 0; i <= last; ++i) {
                    Entries R;
                    R.load(s_off, s_end, s_life, i);
                    uint32_t e[E], before[E], free_[E];
                    const uint32_t incl = batch_ends(R, bound, e);
                    batch_holes(R, e, incl, P, before, free_);
                    uint32_t f = free_[0];
#pragma unroll
                    for (int j = 1; j < E; ++j) f = max(f, free_[j]);
                    if (open || ballot(f >= s)) {
                        const uint32_t end = read_lane(R.off[E - 1], WAVE - 1);
                        for (bool ends = open;; ends = true) {
                            if (ends) {
                                // it ends at the first neighbour behind it, or at the row's last entry at least
                                const uint32_t to = first_neighbour(R, e, at + s);
                                open = to == NOTHING && i < last;
                                if (l == 0 && found > 1) s_next[v * others + found - 2] = make_uint2(at, min(to, end));
                                if (found == 1) hole0 = min(to, end);
                                if (open || found > others) break;
                            }
                            // the next one: a lane's highest address so far where it shows a hole behind the last
                            uint32_t x = NOTHING;
#pragma unroll
                            for (int j = E - 1; j >= 0; --j) x = pick(free_[j] >= s && (before[j] > at || !found), before[j], x);
                            const uint64_t more = ballot(x != NOTHING);
                            if (!more) break;
                            at = read_lane(x, first_lane(more));
                            if (!found) at0 = at;
                            ++found;
                        }
                        if (found > others) break;
                    }
                    P = max(P, read_lane(incl, WAVE - 1));
                }
                if (l >= found - 1 && l < others) s_next[v * others + l].y = 0;       // no further hole
            }
            if (l == 0) s_ask[v] = make_uint4(at0, s, lf, hole0);
        }
        __syncthreads();
        // ---- compare
        const uint4 mine = s_ask[l];
        {
            uint64_t hits = 0, ways = 0;
#pragma unroll
            for (uint32_t q = 0; q < BATCH / NW; ++q) {
                if (q * NW >= lim) break;
                const uint32_t v = q * NW + wave;
                const uint32_t av = read_lane(mine.x, v), ev = av + read_lane(mine.y, v), bound = bound_of(read_lane(mine.z, v));
                const uint64_t m = v < lim ? ballot(l != v && l < lim && life_meets(mine.z, bound)) : 0;
                const uint64_t before = m & ((1ull << v) - 1);
                const uint64_t way = before & ballot(mine.x < ev && av < mine.x + mine.y);
                if (l == v) s_meets[v] = m;
                hits |= way ? 1ull << v : 0;
                ways |= way;
            }
            if (hits && l < 4) atomicOr(&s_hit[l], (uint32_t)((l < 2 ? hits : ways) >> (l % 2 * 32)));
        }
        __syncthreads();
        // ---- settle: lane i has variable i.  Every batch another wave, so that those of the orderings on a compute unit
        // that settle are not all on one SIMD.
        if (wave == turn % NW) {
            uint64_t check = ((uint64_t)uniform(s_hit[1]) << 32) | uniform(s_hit[0]);
            uint32_t acc = lim, o = mine.x, e = mine.x + mine.y;
            if (check) {
                const uint64_t meets = l < lim ? s_meets[l] : 0;
                uint32_t h = mine.w, used = 0;             // the end of the hole it is in, and how many others it has left
                // in rank order: those that have something in their way, and those that are in others' way (no branch
                // but for the next hole: one variable is a chain of some 25 instructions)
                uint64_t todo = check | (((uint64_t)uniform(s_hit[3]) << 32) | uniform(s_hit[2]));
                do {
                    const uint32_t k = first_lane(todo);
                    const uint64_t self = 1ull << k;
                    if (ballot(e > h) & self) {        // behind its hole's end: to the next hole
                        const uint32_t q = read_lane(used, k);
                        const uint2 next = q < others ? s_next[k * others + q] : make_uint2(0, 0);
                        if (uniform(next.y) == 0) { acc = k; break; }
                        if (l == k) { o = next.x; e = o + mine.y; h = next.y; ++used; }
                    }
                    const uint32_t ok = read_lane(o, k), ek = read_lane(e, k);
                    const uint64_t ways = ballot((meets & self) != 0) & ballot(o < ek) & ballot(e > ok);
                    // what is in its way: behind that, every time higher up; else the later ones in whose way it is go
                    // behind it
                    const uint64_t before = ways & (self - 1);
                    const uint32_t to = read_lane(e, before ? 63u - (uint32_t)__builtin_clzll(before) : k);
                    const bool up = __builtin_amdgcn_inverse_ballot_w64(before ? self : ways);
                    o = up ? to : o;
                    e = o + mine.y;
                    todo = before ? todo : (todo | ways) & ~self;
                } while (todo);
            }
            if (l < acc) {
                s_ask[l].x = o;
                offs[r + l] = (uint64_t)o << sh;
                fp = max(fp, e);
            }
            if (l == 0) { s_acc = acc; s_task = NW; }
            if (l < 4) { s_hit[l] = 0; s_done[l] = 0; }
            if (l < 2) s_open[l] = 0;
        }
        __syncthreads();
        // ---- insert: lane k has the batch's block k.  First how many entries each has below it (or at the same offset):
        // steps of a search among 64 entries
        const uint32_t acc = uniform(s_acc);
        uint32_t no = NOTHING, ne = 0, nl = 0;
        if (l < acc) {
            const uint4 q = s_ask[l];
            no = q.x; ne = q.x + q.y; nl = q.z;
        }
        {
            // a wave takes every NW-th block, NW lanes each, that look at as many entries at a time
            const uint32_t k = l / NW * NW + wave, j = l % NW;
            const uint32_t nk = (uint32_t)__shfl((int)no, (int)k, WAVE);
            uint32_t rank = 0;
#pragma unroll
            for (uint32_t q = 0; q < BATCH / NW; ++q) {
                const uint32_t kq = q * NW + wave, nq = read_lane(no, kq);
                const uint32_t c = (uint32_t)__popcll(ballot(no < nq || (no == nq && l < kq)));
                rank = l / NW == q ? c : rank;
            }
            uint32_t from = 0, to = r;                     // the entries before `from` are not above the block, those from `to` on are
            for (uint32_t len = r; len; len /= NW + 1) {   // (the longest that can be left, the same for all)
                const uint32_t step = (to - from) / (NW + 1) + 1, i = from + (j + 1) * step - 1;
                const uint64_t m = ballot(i < to && s_off[min(i, to)] <= nk);
                const uint32_t c = (uint32_t)__popcll(m >> (l / NW * NW) & ((1ull << NW) - 1));
                to = min(to, from + (c + 1) * step - 1);
                from += c * step;
            }
            if (j == 0 && k < acc) s_pos[k] = make_uint2(from, from + rank);
        }
        __syncthreads();
        uint32_t pos = NOTHING, index = 0;
        if (l < acc) { const uint2 q = s_pos[l]; pos = q.x; index = q.y; }
        for (int top = (int)((max(r, 1u) - 1) / ROW);; top -= NW * RPW) {
            uint32_t x[RPW][EPL], xe[RPW][EPL], xl[RPW][EPL], up[RPW][EPL];
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int row = top - (q * NW + (int)wave);
                const bool moves = row >= 0 && ballot(pos < (uint32_t)(row + 1) * ROW) != 0;
#pragma unroll
                for (int c = 0; c < EPL; ++c) {
                    up[q][c] = 0;
                    if (!moves) continue;
                    const uint32_t base = (uint32_t)row * ROW + c * WAVE, i = base + l;
                    const uint64_t all = ballot(pos <= base), some = ballot(pos < base + WAVE);
                    if (!some) continue;
                    x[q][c] = s_off[i]; xe[q][c] = s_end[i]; xl[q][c] = s_life[i];
                    uint32_t u = (uint32_t)__popcll(all);
                    for (uint64_t m = some & ~all; m; m &= m - 1) u += i >= read_lane(pos, first_lane(m)) ? 1u : 0u;
                    up[q][c] = i < r ? u : 0;
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const uint32_t base = (uint32_t)(top - (q * NW + (int)wave)) * ROW + l;
#pragma unroll
                for (int c = 0; c < EPL; ++c)
                    if (up[q][c]) {
                        const uint32_t i = base + c * WAVE + up[q][c];
                        s_off[i] = x[q][c]; s_end[i] = xe[q][c]; s_life[i] = xl[q][c];
                    }
            }
            if (top < NW * RPW) break;
        }
        if (wave == 0 && l < acc) { s_off[index] = no; s_end[index] = ne; s_life[index] = nl; }
        // the 64 ranks after the next 64, once the batches have reached the next 64
        if (fetches && (r + acc) / WAVE != r / WAVE) {
            const uint32_t base = (r + acc) / WAVE * WAVE + WAVE;
            if (base + l < n) s_rec[(base + l) % AHEAD] = make_uint2(life_word(rec_next.x, rec_next.y), rec_next.z);
            if (base + WAVE + l < n) rec_next = A.vrec[v_next];
            if (base + 2 * WAVE + l < n) v_next = perm[base + 2 * WAVE + l];
        }
        r += acc;
        if (few) --few;
        else if ((cut = acc < lim && acc < FEW ? cut + 1 : 0) == 3) { few = FEW; cut = 0; }
        // half as many again as could be placed, where that was not all
        most = acc == lim ? min(BATCH, 2 * most) : min(BATCH, max(8u, acc + acc / 2));
        __syncthreads();
    }
    fp = wave_max32(fp);
    if (l == 0) atomicMax(&s_fp, fp);
    __syncthreads();
    if (tid == 0) {
        A.fps[b] = (uint64_t)s_fp << sh;
        A.ticks[b] = (uint64_t)(wall_clock64() - t_begin);
    }
}

template <int NW, int RPW, bool NEAR>
hipError_t launch_one(const BatchArgs &A, uint32_t B, hipStream_t st)
{
    hipLaunchKernelGGL((k_place_batch<NW, RPW, NEAR>), dim3(B), dim3(NW * WAVE), (size_t)(NEAR ? A.cap : 2 * NW * WAVE * 4) * 12, st, A);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_place_batch(uint32_t n, uint32_t B, const uint32_t *perm,
                              PlanHeader *hdr, const void *vrec, uint32_t *blocks, uint64_t *offs, uint64_t *fps,
                              uint64_t *ticks, hipStream_t st)
{
    const BatchArgs A{n, (n / ROWE + 1) * ROWE, (const uint4 *)vrec, perm, hdr, blocks, offs, fps, ticks};
    // 16 waves where an ordering has a compute unit to itself, else 8, two orderings to a unit; ms with 16 and with 8, of a
    // residual chain of 20 000 variables: 300 orderings 23.6 and 22.1, 1024 51.3 and 43.5; 4096 of 50 000 929 and 811 (with four
    // waves, four to a unit, 842; 512 of 33 000 53 with 8 and 81 with 4).
    if (n > PLAN_BATCH_LDS_VARS) return B <= 256 ? launch_one<16, 2, false>(A, B, st) : launch_one<8, 2, false>(A, B, st);
    // In LDS likewise (registers: 20 waves a unit); ms with 8
    // and with 16 waves, of a residual chain of 5000 variables: 256 orderings 2.49 and 2.25, 512 2.49 and 3.59, 1024
    // 4.78 and 6.39; of 6400, whose blocks take more than half of the LDS: 300 orderings 4.81 and 3.95, 1024 10.5 and 8.8.
    // (Four waves, four orderings to a unit: 1024 orderings of 3000 2.68 ms, 2.86 in registers, but random lifetimes and few
    // sizes 3.67 and 2.80.)
    if (B <= 256 || 2 * (A.cap * 12 + BATCH_LDS) > 160u * 1024) return launch_one<16, 2, true>(A, B, st);
    return launch_one<8, 2, true>(A, B, st);
}

}  // namespace lap
