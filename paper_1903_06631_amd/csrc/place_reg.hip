// Placement of every variable under many orderings (Section III-C), first-fit or best-fit, for
// traces of up to a few ten thousand variables: the placed blocks stay in registers.
//
// One workgroup of NW waves works on one ordering.  The placed blocks are kept sorted by offset, in
// rows of 256: row r * NW + w belongs to wave w, lane l holds entries 4 l .. 4 l + 3 of it as
// (offset, end, lifetime in 16 + 16 bits), twelve registers per row.  A variable asks row after
// row: entries that do not meet it in time are masked, a prefix maximum of the remaining ends over
// the row gives the highest occupied address so far, and an entry whose offset leaves `size` free
// above it shows a hole (first-fit: the first one ends the search; best-fit: the smallest of all rows
// wins).  The block is then inserted: the rows above it move up by one entry, each taking over the
// last entry of the row below.  Entries not yet in use lie at the highest offset and meet nothing, so
// they always show a hole and no row needs a count.
//
// With several waves a variable takes two workgroup barriers: every wave publishes its rows' highest
// ends and last entries; knowing those of all rows it looks for holes in its own; the lowest answer
// is the variable's, and every wave moves its own rows.
#include "lap_dev.h"
#include "lap_kernels.h"

namespace lap {

namespace {

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
__device__ __forceinline__ void row_insert(Row &R, uint32_t o, uint32_t xo, uint32_t xe, uint32_t xl, uint32_t co, uint32_t ce,
                                           uint32_t cl)
{
    const uint32_t po = lane_shift_up(R.off[3], co), pe = lane_shift_up(R.end[3], ce), pl = lane_shift_up(R.life[3], cl);
    if (read_lane(R.off[0], 0) > o && co > o) {          // all of it moves
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

// f(row number) for the rows I .. N-1 in ascending order, or N-1 .. I in descending, until it
// returns false.  The number is a constant of the compilation: rows are registers and have no address.
template <int V> struct RowNo { static constexpr int value = V; };
template <int I, int N, class F> __device__ __forceinline__ void rows_up(F &&f)
{
    if constexpr (I < N) {
        if (f(RowNo<I>{})) rows_up<I + 1, N>(f);
    }
}
template <int I, int N, class F> __device__ __forceinline__ void rows_down(F &&f)
{
    if constexpr (I < N) {
        if (f(RowNo<N - 1>{})) rows_down<I, N - 1>(f);
    }
}

struct RegArgs {
    uint32_t n;
    const uint4 *vrec;           // [n] (first step, end of life, size in granules, -)
    const uint32_t *perm;        // [B][n]
    const uint32_t *fits;        // [B]
    const PlanHeader *hdr;
    uint64_t *offs;              // [B][n] in rank order
    uint64_t *fps;               // [B]
    uint64_t *ticks;             // [B] duration of every ordering in timer ticks
};

template <int NW, int R>
__global__ __launch_bounds__(NW *WAVE) void k_place_reg(RegArgs A)
{
    constexpr int ROWS = NW * R;
    constexpr int RL = (ROWS + WAVE - 1) / WAVE;          // rows per lane where lanes stand for rows
    __shared__ uint4 s_row[2][RL * WAVE];                 // per row: its last entry, the highest end among the neighbours
    __shared__ uint32_t s_at[2];
    __shared__ unsigned long long s_hole[2];

    const uint32_t b = blockIdx.x;
    const bool best_fit = A.fits[b] != 0;
    if (!reg_places(A.hdr, A.n, best_fit)) return;
    const long long t_begin = wall_clock64();
    const uint32_t n = A.n, sh = A.hdr->shift;
    const int l = lane_id();
    const uint32_t wave = NW == 1 ? 0u : (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const uint32_t *perm = A.perm + (size_t)b * n;
    uint64_t *offs = A.offs + (size_t)b * n;

    Row row[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < EPL; ++j) { row[r].off[j] = NOTHING; row[r].end[j] = NOTHING; row[r].life[j] = NOTHING; }
    if constexpr (NW > 1) {
        if (threadIdx.x < 2) { s_at[threadIdx.x] = NOTHING; s_hole[threadIdx.x] = U64_MAX; }
        __syncthreads();
    }

    uint32_t cnt = 0, fp = 0;
    // the records of the ranks to come are fetched ahead: while 64 ranks are placed, the records
    // of the next 64 and the variable numbers of the 64 after are on their way
    uint4 rec_next = make_uint4(0u, 1u, 1u, 0u);
    uint32_t v_next = 0;
    if ((uint32_t)l < n) rec_next = A.vrec[perm[l]];
    if ((uint32_t)l + WAVE < n) v_next = perm[l + WAVE];
    for (uint32_t r0 = 0; r0 < n; r0 += WAVE) {
        const uint4 rec = rec_next;
        if (r0 + l + WAVE < n) rec_next = A.vrec[v_next];
        if (r0 + l + 2 * WAVE < n) v_next = perm[r0 + l + 2 * WAVE];
        const uint32_t wn = min((uint32_t)WAVE, n - r0);
        uint32_t res = 0;
        for (uint32_t p = 0; p < wn; ++p) {
            const uint32_t va = read_lane(rec.x, (int)p), vf = read_lane(rec.y, (int)p), s = read_lane(rec.z, (int)p);
            const uint32_t bound = life_bound(va, vf), lf = life_word(va, vf);
            const uint32_t used = cnt / ROW + 1;          // rows 0 .. used-1 hold the blocks and room for one more
            uint32_t o = NOTHING;
            if constexpr (NW == 1) {
                uint32_t P = 0;
                if (!best_fit) {
                    // two rows at a time: the one's prefix maximum fills the waits of the other's
                    rows_up<0, (R + 1) / 2>([&](auto no) -> bool {
                        constexpr int r = 2 * decltype(no)::value, r1 = r + 1 < R ? r + 1 : r;
                        uint32_t e[EPL], e1[EPL], before[EPL], free_[EPL];
                        const uint32_t incl = row_ends(row[r], bound, e);
                        const uint32_t incl1 = r1 > r ? row_ends(row[r1], bound, e1) : 0u;
                        row_holes(row[r], e, incl, P, before, free_);
                        P = max(P, read_lane(incl, WAVE - 1));
                        if (row_first(before, free_, s, o)) return false;
                        if constexpr (r1 > r) {
                            row_holes(row[r1], e1, incl1, P, before, free_);
                            P = max(P, read_lane(incl1, WAVE - 1));
                            return !row_first(before, free_, s, o);
                        }
                        return true;
                    });
                    o = min(o, P);                        // no hole: all R rows are full
                } else {
                    uint32_t gap = NOTHING, at = 0;
                    rows_up<0, R>([&](auto no) -> bool {
                        constexpr int r = decltype(no)::value;
                        if ((uint32_t)r >= used) return false;
                        uint32_t e[EPL], before[EPL], free_[EPL];
                        const uint32_t incl = row_ends(row[r], bound, e);
                        row_holes(row[r], e, incl, P, before, free_);
                        P = max(P, read_lane(incl, WAVE - 1));
                        row_best(e, before, free_, s, gap, at);
                        return true;
                    });
                    const uint64_t h = wave_min_hole(gap, at);
                    o = (uint32_t)(h >> 32) != NOTHING ? (uint32_t)h : P;
                }
                rows_down<0, R>([&](auto no) -> bool {
                    constexpr int r = decltype(no)::value;
                    if ((uint32_t)r >= used) return true;
                    uint32_t co = 0, ce = 0, cl = 0;
                    if constexpr (r > 0) {
                        co = read_lane(row[r - 1].off[EPL - 1], WAVE - 1);
                        ce = read_lane(row[r - 1].end[EPL - 1], WAVE - 1);
                        cl = read_lane(row[r - 1].life[EPL - 1], WAVE - 1);
                    }
                    row_insert(row[r], o, o, o + s, lf, co, ce, cl);
                    return co > o;                        // else the rows below stay as they are
                });
            } else {
                const uint32_t buf = cnt & 1u;
                constexpr int KEEP = R <= 4 ? R : 1;       // rows whose masked ends stay in registers between the steps
                uint32_t ends[KEEP][EPL], incls[KEEP];
                rows_up<0, R>([&](auto no) -> bool {
                    constexpr int r = decltype(no)::value;
                    const uint32_t id = r * NW + wave;
                    if (id >= used) return false;
                    constexpr int k = KEEP == R ? r : 0;
                    incls[k] = row_ends(row[r], bound, ends[k]);
                    if (l == WAVE - 1)
                        s_row[buf][id] = make_uint4(row[r].off[EPL - 1], row[r].end[EPL - 1], row[r].life[EPL - 1], incls[k]);
                    return true;
                });
                __syncthreads();
                if (threadIdx.x == 0) { s_at[buf ^ 1] = NOTHING; s_hole[buf ^ 1] = U64_MAX; }
                uint32_t below[RL], top = 0;               // prefix maximum of the rows' highest ends
#pragma unroll
                for (int q = 0; q < RL; ++q) {
                    const uint32_t x = (uint32_t)(q * WAVE + l) < used ? s_row[buf][q * WAVE + l].w : 0u;
                    below[q] = max(wave_scan_max_u32(x), top);
                    top = read_lane(below[q], WAVE - 1);
                }
                uint32_t gap = NOTHING, at = NOTHING;
                rows_up<0, R>([&](auto no) -> bool {
                    constexpr int r = decltype(no)::value;
                    const uint32_t id = r * NW + wave;
                    if (id >= used) return false;
                    uint32_t P = 0;
                    if (id > 0) {
                        P = read_lane(below[0], (int)((id - 1) & (WAVE - 1)));
                        if (RL > 1 && id > (uint32_t)WAVE) P = read_lane(below[RL - 1], (int)((id - 1) & (WAVE - 1)));
                    }
                    constexpr int k = KEEP == R ? r : 0;
                    if constexpr (KEEP != R) incls[k] = row_ends(row[r], bound, ends[k]);
                    uint32_t before[EPL], free_[EPL];
                    row_holes(row[r], ends[k], incls[k], P, before, free_);
                    if (!best_fit) {
                        if (row_first(before, free_, s, at)) {
                            if (l == 0) atomicMin(&s_at[buf], at);
                            return false;
                        }
                    } else {
                        row_best(ends[k], before, free_, s, gap, at);
                    }
                    return true;
                });
                if (best_fit) {
                    const uint64_t h = wave_min_hole(gap, at);
                    if (l == 0 && (uint32_t)(h >> 32) != NOTHING) atomicMin(&s_hole[buf], (unsigned long long)h);
                }
                __syncthreads();
                if (!best_fit) {
                    o = min((uint32_t)__builtin_amdgcn_readfirstlane((int)s_at[buf]), top);
                } else {
                    const uint64_t h = s_hole[buf];
                    o = (uint32_t)(h >> 32) != NOTHING ? (uint32_t)h : top;
                    o = (uint32_t)__builtin_amdgcn_readfirstlane((int)o);
                }
                rows_down<0, R>([&](auto no) -> bool {
                    constexpr int r = decltype(no)::value;
                    const uint32_t id = r * NW + wave;
                    if (id >= used) return true;
                    uint4 c = make_uint4(0u, 0u, 0u, 0u);
                    if (id > 0) c = s_row[buf][id - 1];
                    const uint32_t co = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.x);
                    row_insert(row[r], o, o, o + s, lf, co, c.y, c.z);
                    return co > o;                        // else this wave's rows below stay as they are
                });
            }
            ++cnt;
            fp = max(fp, o + s);
            if ((uint32_t)l == p) res = o;
        }
        if (wave == 0 && r0 + l < n) offs[r0 + l] = (uint64_t)res << sh;
    }
    if (threadIdx.x == 0) {
        A.fps[b] = (uint64_t)fp << sh;
        A.ticks[b] = (uint64_t)(wall_clock64() - t_begin);
    }
}

template <int NW, int R>
hipError_t launch_one(const RegArgs &A, uint32_t B, hipStream_t st)
{
    hipLaunchKernelGGL((k_place_reg<NW, R>), dim3(B), dim3(NW * WAVE), 0, st, A);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_place_reg(uint32_t n, uint32_t T, uint32_t B, const uint32_t *perm, const uint32_t *fits,
                            const PlanHeader *hdr, const void *vrec, uint64_t *offs, uint64_t *fps, uint64_t *ticks,
                            hipStream_t st)
{
    if (!reg_may_place(n, T)) return hipSuccess;
    const RegArgs A{n, (const uint4 *)vrec, perm, fits, hdr, offs, fps, ticks};
    const uint32_t rows = (n + ROW - 1) / ROW;
    // Up to 8 rows one wave is the fastest way through an ordering (1000 variables: 0.55 ms; 0.75 ms
    // with 16 waves).  Beyond, 16 waves are (3000 variables: 2.6 ms instead of 3.3 ms), as long as every
    // ordering has a compute unit to itself; where orderings share one, the same work done by fewer
    // waves is more (1024 orderings of 3000: 4.2 ms with one wave, 6.8 ms with 16; 600 orderings of
    // 6000: 13 ms with 4, 21 ms with 16).  More rows than fit fewer waves' registers need 16.
    const bool alone = B <= 256;
    if (rows <= 1) return launch_one<1, 1>(A, B, st);
    if (rows <= 2) return launch_one<1, 2>(A, B, st);
    if (rows <= 4) return launch_one<1, 4>(A, B, st);
    if (rows <= 8) return launch_one<1, 8>(A, B, st);
    if (rows <= 16) return alone ? launch_one<16, 1>(A, B, st) : launch_one<1, 16>(A, B, st);
    if (rows <= 40 && !alone) return launch_one<4, 10>(A, B, st);
    if (rows <= 48) return launch_one<16, 3>(A, B, st);
    return launch_one<16, 7>(A, B, st);
}

}  // namespace lap
