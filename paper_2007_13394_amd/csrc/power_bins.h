// Binning of mode powers by |n| in a workgroup's LDS histogram.
#pragma once

#include "pm_internal.h"

namespace pm {
namespace {

// floor(sqrt(v)) of an integer below 2^24 (three squared mode numbers of a
// mesh of at most 2048 per side): the float root (one instruction, one unit in the
// last place; a rounded one takes sixteen) is off by at most one.
__device__ __forceinline__ int isqrt24(int v)
{
    int b = (int)__builtin_amdgcn_sqrtf((float)v);
    b -= b * b > v ? 1 : 0;
    b += (b + 1) * (b + 1) <= v ? 1 : 0;
    return b;
}

// Runs of neighbouring lanes with one bin, as lane masks (scalar arithmetic): the
// runs' last lanes, and for each step of bin_runs' prefix sum the lanes whose run
// reaches back to the lane that the step takes its value from: 1, 2, 4 or 8 lanes
// below, the last lane of the row of 16 below, the last of the half below.
struct BinRuns {
    int bin;
    uint64_t end, reach[6];
};
__device__ __forceinline__ BinRuns bin_runs_of(int bin)
{
    BinRuns r;
    r.bin = bin;
    r.end = __ballot(__shfl_down(bin, 1) != bin) | 1ull << 63;
    uint64_t start = r.end << 1 | 1;
    r.reach[0] = ~start;
    r.reach[1] = r.reach[0] & r.reach[0] << 1;
    r.reach[2] = r.reach[1] & r.reach[1] << 2;
    r.reach[3] = r.reach[2] & r.reach[2] << 4;
    // starts spread to the lanes above them in their row, then from rows 0 and 2 over
    // the row above
    start |= start << 1 & 0xfffefffefffefffeull;
    start |= start << 2 & 0xfffcfffcfffcfffcull;
    start |= start << 4 & 0xfff0fff0fff0fff0ull;
    start |= start << 8 & 0xff00ff00ff00ff00ull;
    r.reach[4] = ~start & 0xffff0000ffff0000ull;
    const uint64_t below = start & 0x0000800000008000ull;
    r.reach[5] = ~(start | ((below << 17) - (below << 1))) & 0xffffffff00000000ull;
    return r;
}

// Lanes of `reach` add the value that CTRL brings them; what the others read is
// not used.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v, uint64_t reach)
{
    const long long u = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xf, 0xf, true);
    const double t = __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
    return __builtin_amdgcn_inverse_ballot_w64(reach) ? v + t : v;
}

// hist[bin] += v over a whole wavefront (every lane calls it; bin < 0: nothing).
// Lanes hold neighbouring modes, so runs of them share a bin, and LDS atomics on
// one address are taken one by one: each run instead adds its own sum, formed by
// a prefix sum that takes no value from before the run.  (Differences of one
// prefix sum over all lanes would give each bin the rounding of the largest power
// among its 64 neighbours, and an infinity to all behind it.)
__device__ __forceinline__ void bin_runs(double *hist, const BinRuns &r, double v)
{
    v = dpp_add<0x111>(v, r.reach[0]);
    v = dpp_add<0x112>(v, r.reach[1]);
    v = dpp_add<0x114>(v, r.reach[2]);
    v = dpp_add<0x118>(v, r.reach[3]);
    v = dpp_add<0x142>(v, r.reach[4]);
    v = dpp_add<0x143>(v, r.reach[5]);
    if (__builtin_amdgcn_inverse_ballot_w64(r.end) && r.bin >= 0) atomicAdd(hist + r.bin, v);
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
