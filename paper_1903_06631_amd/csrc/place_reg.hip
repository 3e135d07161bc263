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
#include "block_rows.h"
#include "lap_kernels.h"

namespace lap {

namespace {

// f(row number) for the rows I .. N-1 in ascending order until it returns false.  The number is a constant of the compilation: rows are registers and have no address.
template <int V> struct RowNo { static constexpr int value = V; };
template <int I, int N, class F> __device__ __forceinline__ void rows_up(F &&f)
{
    if constexpr (I < N) {
        if (f(RowNo<I>{})) rows_up<I + 1, N>(f);
    }
}
// ... descending, for the rows that come before `used` only (I is one of them): one branch leaves half of the rows out
template <int I, int N, class F> __device__ __forceinline__ bool rows_down(uint32_t used, F &&f)
{
    if constexpr (N - I == 1) return f(RowNo<I>{});
    else {
        constexpr int M = (I + N) / 2;
        if (used > (uint32_t)M && !rows_down<M, N>(used, f)) return false;
        return rows_down<I, M>(used, f);
    }
}

struct RegArgs {
    uint32_t n, B;
    const uint4 *vrec;           // [n] (first step, end of life, size in granules, -)
    const uint32_t *perm;        // [B][n]
    const uint32_t *fits;        // [B]
    const PlanHeader *hdr;
    uint64_t *offs;              // [B][n] in rank order
    uint64_t *fps;               // [B]
    uint64_t *ticks;             // [B] duration of every ordering in timer ticks
};

// PACK: where one wave works on an ordering, a workgroup may hold several of them side by side; its waves share nothing.
// A constant of the compilation, since a workgroup of one that looks at what there is for a second one starts 1 us later
// (plan of 120 variables 68.0 and 69.1 us).
template <int NW, int R, int PACK>
__global__ __launch_bounds__(NW *PACK *WAVE) void k_place_reg(RegArgs A)
{
    constexpr int ROWS = NW * R;
    constexpr int RL = (ROWS + WAVE - 1) / WAVE;          // rows per lane where lanes stand for rows
    __shared__ uint4 s_row[2][RL * WAVE];                 // per row: its last entry, the highest end among the neighbours
    __shared__ uint32_t s_at[2];
    __shared__ unsigned long long s_hole[2];

    static_assert(NW == 1 || PACK == 1, "several waves of one ordering, or one of several");
    uint32_t b = blockIdx.x;
    if constexpr (PACK > 1) {
        b = b * PACK + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
        if (b >= A.B) return;
    }
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
                rows_down<0, R>(used, [&](auto no) -> bool {
                    constexpr int r = decltype(no)::value;
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
                // the rows' masked ends stay in registers between the steps where there is room
                constexpr int KEEP = R <= 5 ? R : 1;
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
                rows_down<0, R>(R, [&](auto no) -> bool {
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
    if (PACK > 1 ? l == 0 : threadIdx.x == 0) {
        A.fps[b] = (uint64_t)fp << sh;
        A.ticks[b] = (uint64_t)(wall_clock64() - t_begin);
    }
}

template <int NW, int R>
hipError_t launch_one(const RegArgs &A, uint32_t B, hipStream_t st)
{
    // Four one-wave orderings to a workgroup where a compute unit gets four of them and more: the waves of a workgroup go
    // to a unit's four SIMDs one by one, those of four workgroups need not (of 1024 workgroups 60 to 110 SIMDs were given
    // two and as many none, up to chance and to what ran before, and the launch then takes 1.3 times as long).  Whole
    // plans with one and with four to a workgroup: 800 and 1024 orderings of 500 variables 0.58 and 0.50, 0.65 and 0.56 ms,
    // of 640 0.72 and 0.60, 0.79 and 0.66; 1024 of 3000 4.23 and 3.27 (all offsets asked for), or 3.29 and 3.21; 2048 of
    // 2000 3.30 and 2.67.  Three to a unit spread well either way, and so do many rounds (4096 of 1500 3.41 and 3.44).
    constexpr int PACK = NW == 1 ? 4 : 1;
    if (PACK > 1 && B > 768 && B <= 2048)
        hipLaunchKernelGGL((k_place_reg<NW, R, PACK>), dim3((B - 1) / PACK + 1), dim3(NW * PACK * WAVE), 0, st, A);
    else
        hipLaunchKernelGGL((k_place_reg<NW, R, 1>), dim3(B), dim3(NW * WAVE), 0, st, A);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_place_reg(uint32_t n, uint32_t T, uint32_t B, const uint32_t *perm, const uint32_t *fits,
                            bool any_best, const PlanHeader *hdr, const void *vrec, uint64_t *offs, uint64_t *fps, uint64_t *ticks,
                            hipStream_t st)
{
    if (n > PLAN_REG_MAX_VARS || T > 0xFFFFu) return hipSuccess;
    const RegArgs A{n, B, (const uint4 *)vrec, perm, fits, hdr, offs, fps, ticks};
    const uint32_t rows = (n + ROW - 1) / ROW;
    // Up to 8 rows one wave is the fastest way through an ordering (1000 variables: 0.55 ms; 0.75 ms
    // with 16 waves).  Beyond, 12 or 16 waves are (193 orderings of 3000 variables: 2.57 ms with 12; 3.3 ms with one),
    // as long as every ordering has a compute unit to itself; where orderings share one, the same work done by fewer
    // waves is more: one wave up to 16 rows (1024 orderings of 3000: 3.0 ms, 4.6 with 4 waves and 5.2 with 8; 300 of
    // 4000 4.99 ms, 5.08 with 8 and 5.13 with 16), 8 waves up to 40 rows.  Of more than 24 rows, 8 waves (96 and 115
    // registers) leave a unit two orderings and 4 waves (154) three, so what 4 waves lose in a round they win where they
    // need one round and 8 waves two, from 513 to 768 orderings, and nowhere else (ms with 8 and with 4 waves, of
    //   6400:   512 orderings 9.7 and 12.6, 513 15.6 and 13.9, 768 15.7 and 14.3, 800 18.8 and 22.7, 1536 27.9 and 28.2
    //   8192:   512           13.5    18.0, 513 21.4     20.3, 768 21.7     20.7, 800 26.2     32.4, 1536 38.7     40.7
    //   10 000: 512           17.9    24.6, 513 28.4     27.7, 768 28.7     28.5, 800 34.7     44.0, 1536 51.3     55.6;
    // best-fit, 768 orderings of 6145 18.3 and 16.9, 7224 22.7 and 21.8, 8192 27.0 and 26.7, but 9000 31.0 and 31.2, 10 000
    // 36.2 and 37.1).  More rows than 40 need 16.
    // Rows that a trace cannot fill cost all the same (193 orderings of 9001: 11.5 ms with 12 waves of 3 rows, 11.8
    // with 16), and up to 5 rows a wave keeps their ends (100 of 15 000: 24 ms with 4 rows, 30 with 7).
    // First-fit calls of more than 1024 variables go to the batches (place_batch.hip); here come those of them whose
    // lifetimes cross and that have few sizes, and all with a best-fit ordering among them.
    const bool alone = B <= 256;
    if (rows <= 1) return launch_one<1, 1>(A, B, st);
    if (rows <= 2) return launch_one<1, 2>(A, B, st);
    if (rows <= 3) return launch_one<1, 3>(A, B, st);
    if (rows <= 4) return launch_one<1, 4>(A, B, st);
    if (rows <= 8) return launch_one<1, 8>(A, B, st);
    if (alone) {
        if (rows <= 12) return launch_one<12, 1>(A, B, st);
        if (rows <= 16) return launch_one<16, 1>(A, B, st);
        if (rows <= 24) return launch_one<12, 2>(A, B, st);
        if (rows <= 36) return launch_one<12, 3>(A, B, st);
    } else {
        if (rows <= 16) return launch_one<1, 16>(A, B, st);
        if (rows <= 24) return launch_one<8, 3>(A, B, st);
        if (rows <= (any_best ? 32u : 40u) && B > 512 && B <= 768) return launch_one<4, 10>(A, B, st);
        if (rows <= 32) return launch_one<8, 4>(A, B, st);
        if (rows <= 40) return launch_one<8, 5>(A, B, st);
    }
    if (rows <= 48) return launch_one<16, 3>(A, B, st);
    if (rows <= 64) return launch_one<16, 4>(A, B, st);
    if (rows <= 80) return launch_one<16, 5>(A, B, st);
    if (rows <= 112) return launch_one<16, 7>(A, B, st);
    // 64, 256 and 1024 orderings of a residual chain of 32 767: 98, 99 and 396 ms; 436, 469 and 711 by the sweep.  (All of
    // its 128 registers are in use and two values that wait for the end of 64 placements and of the ordering, the granule's
    // shift among them, are spilled: 12 bytes of scratch a lane.)
    return launch_one<16, 8>(A, B, st);
}

}  // namespace lap
