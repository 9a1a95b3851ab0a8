// Binning of mode powers by |n| in a workgroup's LDS histogram.
#pragma once

#include "pm_internal.h"

namespace pm {
namespace {

// floor(sqrt(v)) of an integer below 2^24 (three squared mode numbers of a
// mesh of at most 2048 per side): the float root is off by at most one.
__device__ __forceinline__ int isqrt24(int v)
{
    int b = (int)__builtin_sqrtf((float)v);
    b -= b * b > v ? 1 : 0;
    b += (b + 1) * (b + 1) <= v ? 1 : 0;
    return b;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    const long long u = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, false);
    return v + __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Inclusive sum over the lanes of a wavefront (row shifts by 1, 2, 4, 8, then
// the last lanes of rows 0/2 and of the first half broadcast onwards).
__device__ __forceinline__ double lane_prefix(double v)
{
    v = dpp_add<0x111, 0xf>(v);
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);
    return dpp_add<0x143, 0xc>(v);
}

// hist[bin] += v over a whole wavefront (every lane calls it; bin < 0: nothing).
// Lanes hold neighbouring modes, so runs of them share a bin, and LDS atomics on
// one address are taken one by one: each run instead adds its prefix sum's
// difference, two atomics per run.  next: the bin of the lane above.
__device__ __forceinline__ void bin_runs(double *hist, int bin, int next, bool last, double v)
{
    const double s = lane_prefix(v);
    if (last || next != bin) {
        if (bin >= 0) atomicAdd(hist + bin, s);
        if (!last && next >= 0) atomicAdd(hist + next, -s);
    }
}

// 1 / sinc^4(pi n / N) per axis (n = 0 .. N/2): the reciprocal of the
// cloud-in-cell window of a power.
__device__ __forceinline__ void window_table(double *tab, int n, int threads)
{
    for (int i = threadIdx.x; i <= n / 2; i += threads) {
        const double x = 3.141592653589793238 * i / n, s = i == 0 ? 1.0 : sin(x) / x;
        tab[i] = 1.0 / (s * s * s * s);
    }
}

}  // namespace
}  // namespace pm
