// Sums per step of variables that arrive in the order in which they are allocated.
#pragma once
#include "lap_dev.h"

namespace lap {

// inclusive prefix sum over the wave, without the LDS unit that shuffles go through
__device__ __forceinline__ uint64_t wave_scan_add_dpp(uint64_t v)
{
    auto from = [&](auto lo, auto hi) { return ((uint64_t)hi << 32) | lo; };
    v += from(dpp_mov<0x111>(0u, (uint32_t)v), dpp_mov<0x111>(0u, (uint32_t)(v >> 32)));
    v += from(dpp_mov<0x112>(0u, (uint32_t)v), dpp_mov<0x112>(0u, (uint32_t)(v >> 32)));
    v += from(dpp_mov<0x114>(0u, (uint32_t)v), dpp_mov<0x114>(0u, (uint32_t)(v >> 32)));
    v += from(dpp_mov<0x118>(0u, (uint32_t)v), dpp_mov<0x118>(0u, (uint32_t)(v >> 32)));
    v += from(dpp_mov<0x142, 0xA>(0u, (uint32_t)v), dpp_mov<0x142, 0xA>(0u, (uint32_t)(v >> 32)));
    v += from(dpp_mov<0x143, 0xC>(0u, (uint32_t)v), dpp_mov<0x143, 0xC>(0u, (uint32_t)(v >> 32)));
    return v;
}

// add(key, sum of v) for every run of neighbouring lanes with the same key, by the run's last lane; the key NO_KEY is
// left out.  All lanes of the wave take part.  Variables arrive in the order in which they are allocated, so most lanes
// of a wave meet the same step or two, and an atomic unit serves adds on one address one after the other: up to
// RUNS_MERGED runs are summed first (a scan), more are added as they are.
constexpr uint32_t NO_KEY = 0xFFFFFFFFu;
constexpr int RUNS_MERGED = 32;
template <class Add> __device__ __forceinline__ void wave_add_runs(uint32_t key, uint64_t v, Add add)
{
    const uint64_t heads = ballot(key != lane_shift_up(key, ~key));        // lane 0 starts a run whatever its key is
    if (__popcll(heads) > RUNS_MERGED) {
        if (key != NO_KEY) add(key, v);
        return;
    }
    const int l = lane_id();
    const uint64_t sum = wave_scan_add_dpp(v);
    const uint64_t upto = heads & (~0ull >> (WAVE - 1 - l));               // never zero: lane 0 is a head
    const int first = WAVE - 1 - __clzll((long long)upto);
    const uint64_t before = shfl64(sum, first ? first - 1 : 0);
    const bool last = l == WAVE - 1 || ((heads >> ((l + 1) & (WAVE - 1))) & 1ull);
    if (last && key != NO_KEY) add(key, first ? sum - before : sum);
}

}  // namespace lap
