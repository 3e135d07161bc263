// Placed blocks in registers: a row of 256, sorted by offset, held by one wave -- lane l has the
// entries 4 l .. 4 l + 3.  Entries not in use lie at the highest offset and meet nothing, so they
// always show a hole and a row needs no count.  Lifetimes have 16-bit steps.
#pragma once
#include "lap_dev.h"

namespace lap {

constexpr uint32_t NOTHING = 0xFFFFFFFFu;
constexpr int EPL = 4;                         // entries per lane and row
constexpr uint32_t ROW = EPL * WAVE;

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// A lifetime [a, f), f <= 65535, as (a, 65535 - f): it meets [va, vf) iff both halves are at most
// those of life_bound(va, vf), one packed maximum and one comparison.
__device__ __forceinline__ uint32_t life_word(uint32_t a, uint32_t f) { return a | ((0xFFFFu - f) << 16); }
__device__ __forceinline__ uint32_t life_bound(uint32_t va, uint32_t vf) { return (vf - 1) | ((0xFFFEu - va) << 16); }
__device__ __forceinline__ bool life_meets(uint32_t lf, uint32_t bound)
{
    const u16x2 m = __builtin_elementwise_max(__builtin_bit_cast(u16x2, lf), __builtin_bit_cast(u16x2, bound));
    return __builtin_bit_cast(uint32_t, m) == bound;
}

__device__ __forceinline__ uint32_t wave_max32(uint32_t v) { return read_lane(wave_scan_max_u32(v), WAVE - 1); }

struct Row {
    uint32_t off[EPL], end[EPL], life[EPL];
};

// the ends of the entries that meet the variable, and their inclusive prefix maximum over the lanes
__device__ __forceinline__ uint32_t row_ends(const Row &R, uint32_t bound, uint32_t (&e)[EPL])
{
#pragma unroll
    for (int j = 0; j < EPL; ++j) e[j] = life_meets(R.life[j], bound) ? R.end[j] : 0u;
    return wave_scan_max_u32(max(max(e[0], e[1]), max(e[2], e[3])));
}

// lane i receives lane i-1's value, lane 0 receives 0
__device__ __forceinline__ uint32_t shift_in_zero(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);
}

// a select that stays one (no branch)
__device__ __forceinline__ uint32_t pick(bool c, uint32_t a, uint32_t b)
{
    const uint32_t m = c ? 0xFFFFFFFFu : 0u;
    return (a & m) | (b & ~m);
}

// What is free below each entry, down to the highest end among the neighbours below it (0 if that is
// higher), and that end.  P: the highest end among the neighbours below the row.
__device__ __forceinline__ void row_holes(const Row &R, const uint32_t (&e)[EPL], uint32_t incl, uint32_t P,
                                          uint32_t (&before)[EPL], uint32_t (&free_)[EPL])
{
    before[0] = max(P, shift_in_zero(incl));
    before[1] = max(before[0], e[0]);
    before[2] = max(max(before[0], e[0]), e[1]);
    before[3] = max(max(before[1], e[1]), e[2]);
#pragma unroll
    for (int j = 0; j < EPL; ++j) free_[j] = __builtin_elementwise_sub_sat(R.off[j], before[j]);
}

// First-fit: the first entry that leaves s free below it, as the address where that hole starts
// (lowest lane, then lowest entry); false if there is none.
__device__ __forceinline__ bool row_first(const uint32_t (&before)[EPL], const uint32_t (&free_)[EPL], uint32_t s, uint32_t &at)
{
    const uint64_t any = ballot(max(max(free_[0], free_[1]), max(free_[2], free_[3])) >= s);
    if (!any) return false;
    const uint32_t mine = pick(free_[0] >= s, before[0], pick(free_[1] >= s, before[1], pick(free_[2] >= s, before[2], before[3])));
    at = read_lane(mine, __ffsll((unsigned long long)any) - 1);
    return true;
}

// Best-fit: the lane's smallest hole between two neighbours so far (the lowest of equally small ones:
// a lane sees them in ascending order)
__device__ __forceinline__ void row_best(const uint32_t (&e)[EPL], const uint32_t (&before)[EPL], const uint32_t (&free_)[EPL],
                                         uint32_t s, uint32_t &gap, uint32_t &at)
{
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
        const uint32_t g = e[j] != 0 && free_[j] >= s ? free_[j] : NOTHING;      // (a neighbour's end is never 0)
        at = pick(g < gap, before[j], at);
        gap = min(g, gap);
    }
}

// the smallest of the lanes' holes as (size << 32 | address), the lowest of equally small ones
__device__ __forceinline__ uint64_t wave_min_hole(uint32_t gap, uint32_t at)
{
    const uint32_t g = ~wave_max32(~gap);
    const uint32_t low = ~wave_max32(gap == g ? ~at : 0u);
    return ((uint64_t)g << 32) | low;
}

// Moves the row up by one entry behind offset o, where x = (xo, xe, xl) goes if its place is in
// this row; c: the last entry of the row below (offset 0 if there is none).
// FIRST: the row's first entry is compared with o as well.  No entry lies below that last one, so it changes no result and
// costs two instructions; what it changes is where the code behind it lies, 8 bytes further on, and the long loops of
// k_place_fast answer to that.  Best-fit with eight waves and the per-step words in LDS: 16 orderings of 120 000 variables
// 48.5 ms without and 47.2 with it, of 200 000 78.3 and 76.0 (16 of 200 000 with one s_nop in its place 76.1, two 76.3, three
// 73.4, but then both policies in one call 78.9 for 74.8; with all loops aligned to 32 or 64 bytes 77.4).  In the other forms
// it is the other way round: 600 best-fit orderings of 200 000 (four waves) 112.7 and 114.1, 100 of 150 000 over 900 steps
// (the words in memory) 66.8 and 67.3, 256 first-fit ones of 200 000 50.8 and 51.8.
template <bool FIRST = false>
__device__ __forceinline__ void row_insert(Row &R, uint32_t o, uint32_t xo, uint32_t xe, uint32_t xl, uint32_t co, uint32_t ce,
                                           uint32_t cl)
{
    const uint32_t po = lane_shift_up(R.off[3], co), pe = lane_shift_up(R.end[3], ce), pl = lane_shift_up(R.life[3], cl);
    if ((!FIRST || read_lane(R.off[0], 0) > o) && co > o) {        // all of it moves
#pragma unroll
        for (int j = EPL - 1; j > 0; --j) { R.off[j] = R.off[j - 1]; R.end[j] = R.end[j - 1]; R.life[j] = R.life[j - 1]; }
        R.off[0] = po; R.end[0] = pe; R.life[0] = pl;
        return;
    }
    // entry by entry: stays, or is the block's place, or takes over the entry below (offsets ascend,
    // so the new one is the median of the old one, the one below and o)
    const bool s0 = R.off[0] <= o, s1 = R.off[1] <= o, s2 = R.off[2] <= o, s3 = R.off[3] <= o, sp = po <= o;
    const uint32_t e3 = pick(s2, xe, R.end[2]), e2 = pick(s1, xe, R.end[1]), e1 = pick(s0, xe, R.end[0]), e0 = pick(sp, xe, pe);
    const uint32_t l3 = pick(s2, xl, R.life[2]), l2 = pick(s1, xl, R.life[1]), l1 = pick(s0, xl, R.life[0]), l0 = pick(sp, xl, pl);
    R.end[3] = pick(s3, R.end[3], e3); R.end[2] = pick(s2, R.end[2], e2); R.end[1] = pick(s1, R.end[1], e1); R.end[0] = pick(s0, R.end[0], e0);
    R.life[3] = pick(s3, R.life[3], l3); R.life[2] = pick(s2, R.life[2], l2); R.life[1] = pick(s1, R.life[1], l1); R.life[0] = pick(s0, R.life[0], l0);
    R.off[3] = max(R.off[2], min(R.off[3], xo));
    R.off[2] = max(R.off[1], min(R.off[2], xo));
    R.off[1] = max(R.off[0], min(R.off[1], xo));
    R.off[0] = max(po, min(R.off[0], xo));
}

}  // namespace lap
