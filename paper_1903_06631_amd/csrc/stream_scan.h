// A transfer stream that serves jobs one after the other, as a scan.  A stream that serves job j (ready r_j, duration
// d_j) after it is free at x is free again at max(x + d_j, r_j + d_j): such functions compose as (a, b) pairs.
#pragma once
#include "lap_dev.h"

namespace lap {

constexpr long long SC_NEG = -(1ll << 62), SC_POS = (1ll << 62);

struct Fn {
    long long a, b;
};
// OUT: f(x) = max(x + a, b), `then` applied after `first`
__device__ __forceinline__ Fn then_max(const Fn &first, const Fn &then)
{
    const long long t = first.b + then.a;
    return Fn{first.a + then.a, t > then.b ? t : then.b};
}
// IN: g(y) = min(y - a, b)
__device__ __forceinline__ Fn then_min(const Fn &first, const Fn &then)
{
    const long long t = first.b - then.a;
    return Fn{first.a + then.a, t < then.b ? t : then.b};
}

// inclusive over a workgroup of WAVES waves; carry is what came before and takes what comes after
template <bool OUT, int WAVES>
__device__ __forceinline__ Fn block_scan_fn(Fn v, Fn &carry, Fn *wtmp)
{
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        Fn o;
        o.a = (long long)shfl_up64((uint64_t)v.a, d);
        o.b = (long long)shfl_up64((uint64_t)v.b, d);
        if (lane >= d) v = OUT ? then_max(o, v) : then_min(o, v);
    }
    if (lane == WAVE - 1) wtmp[wave] = v;
    __syncthreads();
    Fn pre = carry, tot = carry;
    for (int q = 0; q < WAVES; ++q) {
        const Fn x = wtmp[q];
        if (q < wave) pre = OUT ? then_max(pre, x) : then_min(pre, x);
        tot = OUT ? then_max(tot, x) : then_min(tot, x);
    }
    __syncthreads();
    carry = tot;
    return OUT ? then_max(pre, v) : then_min(pre, v);
}

}  // namespace lap
