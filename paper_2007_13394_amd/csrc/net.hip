// Learned force correction: kernels of the forward model and its reverse mode.
//
// Model (an addition to the method; the paper's introduction motivates
// learned corrections of fast particle-mesh codes): a radial filter
// g(k, a) = 1 + MLP(|k| / k_Nyq, a) on the potential spectrum, tabulated at
// NET_NB radial bins and interpolated linearly, and a 3-layer periodic 3^3
// CNN (1 -> 16 -> 16 -> 1 channels, SiLU) on the density contrast (read from
// the int64 mesh); the force is minus the spectral gradient of phi_f + cnn.
// Parameters: one flat FP32 array (offsets in pm_internal.h).  The CNN takes
// BF16 activations and weights and accumulates in FP32; the 16 -> 16 layer,
// 89 % of the network's arithmetic, runs on MFMA.  The CNN's reverse mode is in
// net_bwd.hip.
#include "net_common.h"

namespace pm {
namespace {

// sum + a.lo b.lo + a.hi b.hi for BF16 pairs, FP32 accumulation
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float sum)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2bf, a), __builtin_bit_cast(v2bf, b), sum, false);
}

inline unsigned grid_for(int64_t n, int block, int64_t cap = 65536LL * 16)
{
    int64_t b = (n + block - 1) / block;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (unsigned)b;
}

__device__ __forceinline__ float bin_kt(int b) { return (float)b * 1.7320508075688772f / (float)(NET_NB - 1); }

// ---------------------------------------------------------------- radial MLP table
// One workgroup per bin, one thread per hidden unit.
__global__ __launch_bounds__(128) void k_mlp_fwd(const float *__restrict__ th, float a, float *table)
{
    __shared__ float h[NET_H], red[128];
    const int b = blockIdx.x, j = threadIdx.x;
    const float kt = bin_kt(b);
    float z = 0.f;
    if (j < NET_H) h[j] = silu(th[NB0 + j] + th[NW0 + 2 * j] * kt + th[NW0 + 2 * j + 1] * a);
    __syncthreads();
#pragma unroll 1
    for (int l = 0; l < 2; l++) {
        const int W = l == 0 ? NW1 : NW2, B = l == 0 ? NB1 : NB2;
        if (j < NET_H) {
            z = th[B + j];
            for (int i = 0; i < NET_H; i++) z += th[W + j * NET_H + i] * h[i];
        }
        __syncthreads();
        if (j < NET_H) h[j] = silu(z);
        __syncthreads();
    }
    red[j] = j < NET_H ? th[NW3 + j] * h[j] : 0.f;
    __syncthreads();
    for (int s = 64; s >= 1; s >>= 1) {
        if (j < s) red[j] += red[j + s];
        __syncthreads();
    }
    if (j == 0) table[b] = 1.f + th[NB3] + red[0];
}

// dth += tbar[b] d table[b] / d th.  A workgroup takes MB_BINS bins in turn and
// keeps its share of the weights and of their gradients in registers: thread
// (j, q), q = 0..3, holds columns 24 q .. 24 q + 23 of row j of W1 and W2 and
// the same rows of their transposes, so that a bin is four short products
// between LDS vectors; the gradients go out as float atomics once per workgroup
// (18 600 of them; one workgroup per bin, eight times as many, took 480 us
// against 75).
constexpr int MB_BINS = 8, MB_Q = 4, MB_T = NET_H * MB_Q, MB_C = NET_H / MB_Q;
static_assert(NET_NB % MB_BINS == 0 && NET_H % MB_Q == 0 && MB_C % 4 == 0, "mlp_bwd shape");

// Sum over the columns of this thread's quarter, then over the four quarters.
__device__ __forceinline__ float quarter_dot(const float *w, const float *v)
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MB_C; i += 4) {
        const float4 x = *reinterpret_cast<const float4 *>(v + i);
        s += w[i] * x.x;
        s += w[i + 1] * x.y;
        s += w[i + 2] * x.z;
        s += w[i + 3] * x.w;
    }
    s += __shfl_xor(s, 1);
    return s + __shfl_xor(s, 2);
}

__global__ __launch_bounds__(MB_T) void k_mlp_bwd(const float *__restrict__ th, float a, const double *tbar, float *dth)
{
    __shared__ __align__(16) float h0[NET_H], h1[NET_H], d1[NET_H], d2[NET_H];
    const int j = threadIdx.x / MB_Q, c0 = (threadIdx.x % MB_Q) * MB_C;
    const bool lead = c0 == 0;
    float w1[MB_C], w2[MB_C], w1t[MB_C], w2t[MB_C], g1[MB_C], g2[MB_C];
#pragma unroll
    for (int i = 0; i < MB_C; i++) {
        w1[i] = th[NW1 + j * NET_H + c0 + i];
        w2[i] = th[NW2 + j * NET_H + c0 + i];
        w1t[i] = th[NW1 + (c0 + i) * NET_H + j];
        w2t[i] = th[NW2 + (c0 + i) * NET_H + j];
        g1[i] = g2[i] = 0.f;
    }
    const float b0 = th[NB0 + j], wa = th[NW0 + 2 * j], wb = th[NW0 + 2 * j + 1], b1 = th[NB1 + j], b2 = th[NB2 + j],
                w3 = th[NW3 + j];
    float gb0 = 0.f, gwa = 0.f, gwb = 0.f, gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f;
#pragma unroll 1
    for (int b = blockIdx.x * MB_BINS; b < (blockIdx.x + 1) * MB_BINS; b++) {
        const float g = (float)tbar[b];
        if (g == 0.f) continue;   // uniform over the workgroup
        const float kt = bin_kt(b);
        const float z0 = b0 + wa * kt + wb * a;
        __syncthreads();   // the last bin's vectors have been read
        if (lead) h0[j] = silu(z0);
        __syncthreads();
        const float z1 = b1 + quarter_dot(w1, h0 + c0);
        if (lead) h1[j] = silu(z1);
        __syncthreads();
        const float z2 = b2 + quarter_dot(w2, h1 + c0);
        const float e2 = g * w3 * dsilu(z2);
        gb3 += g;
        gw3 += g * silu(z2);
        gb2 += e2;
        if (lead) d2[j] = e2;
#pragma unroll
        for (int i = 0; i < MB_C; i++) g2[i] += e2 * h1[c0 + i];
        __syncthreads();
        const float e1 = quarter_dot(w2t, d2 + c0) * dsilu(z1);
        gb1 += e1;
        if (lead) d1[j] = e1;
#pragma unroll
        for (int i = 0; i < MB_C; i++) g1[i] += e1 * h0[c0 + i];
        __syncthreads();
        const float e0 = quarter_dot(w1t, d1 + c0) * dsilu(z0);
        gb0 += e0;
        gwa += e0 * kt;
        gwb += e0 * a;
    }
#pragma unroll
    for (int i = 0; i < MB_C; i++) {
        atomicAdd(dth + NW1 + j * NET_H + c0 + i, g1[i]);
        atomicAdd(dth + NW2 + j * NET_H + c0 + i, g2[i]);
    }
    if (lead) {
        atomicAdd(dth + NB0 + j, gb0);
        atomicAdd(dth + NW0 + 2 * j, gwa);
        atomicAdd(dth + NW0 + 2 * j + 1, gwb);
        atomicAdd(dth + NB1 + j, gb1);
        atomicAdd(dth + NB2 + j, gb2);
        atomicAdd(dth + NW3 + j, gw3);
        if (j == 0) atomicAdd(dth + NB3, gb3);
    }
}

// ---------------------------------------------------------------- spectral parts
// Natural-order half spectra [n][n][nhp]; mode t -> wave vector in grid units.
struct Mode {
    float k0, k1, k2, kk;
    bool pad, nyq0, nyq1, nyq2;
    int kz;
};
__device__ __forceinline__ Mode mode_of(int64_t t, int64_t nhp, int n)
{
    Mode m;
    const int kz = (int)(t % nhp);
    const int64_t r = t / nhp;
    const int i1 = (int)(r % n), i0 = (int)(r / n);
    const float sc = 6.28318530717958648f / (float)n;
    m.k0 = sc * (i0 <= n / 2 ? i0 : i0 - n);
    m.k1 = sc * (i1 <= n / 2 ? i1 : i1 - n);
    m.k2 = sc * kz;
    m.kk = m.k0 * m.k0 + m.k1 * m.k1 + m.k2 * m.k2;
    m.pad = kz > n / 2;
    m.nyq0 = i0 == n / 2;
    m.nyq1 = i1 == n / 2;
    m.nyq2 = kz == n / 2;
    m.kz = kz;
    return m;
}


// out = g(|k|) coef / k^2 in (k = 0 and padding -> 0).
__global__ void k_spec_filter(const float2 *in, float2 *out, int64_t nhp, int n, const float *table, float coef)
{
    __shared__ float tab[NET_NB];
    for (int i = threadIdx.x; i < NET_NB; i += blockDim.x) tab[i] = table[i];
    __syncthreads();
    const int64_t tot = (int64_t)n * n * nhp;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
        const Mode m = mode_of(t, nhp, n);
        float2 o = make_float2(0.f, 0.f);
        if (!m.pad && m.kk > 0.f) {
            int b;
            float w;
            const float g = table_at(tab, sqrtf(m.kk) * 0.31830988618379067f, b, w) * coef / m.kk;
            const float2 v = in[t];
            o = make_float2(g * v.x, g * v.y);
        }
        out[t] = o;
    }
}

// tbar[b] += sum over modes of the bin weights times Re[coef / k^2 dk conj(pf)],
// each half-spectrum mode standing for its conjugate too (weight 2) except on
// the planes kz = 0 and kz = n/2.
__global__ __launch_bounds__(256) void k_spec_filter_bwd(const float2 *dk, const float2 *pf, int64_t nhp, int n,
                                                         float coef, double *tbar)
{
    __shared__ double hist[NET_NB];
    for (int i = threadIdx.x; i < NET_NB; i += blockDim.x) hist[i] = 0.0;
    __syncthreads();
    const int64_t tot = (int64_t)n * n * nhp;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
        const Mode m = mode_of(t, nhp, n);
        if (m.pad || m.kk == 0.f) continue;
        const float2 a = dk[t], c = pf[t];
        const float mult = (m.kz == 0 || m.nyq2) ? 1.f : 2.f;
        const float dg = mult * coef / m.kk * (a.x * c.x + a.y * c.y);
        int b;
        float w;
        const float kt = sqrtf(m.kk) * 0.31830988618379067f;
        const float tt = kt * (float)(NET_NB - 1) / 1.7320508075688772f;
        b = (int)floorf(tt);
        if (b > NET_NB - 2) b = NET_NB - 2;
        w = tt - (float)b;
        atomicAdd(&hist[b], (double)((1.f - w) * dg));
        atomicAdd(&hist[b + 1], (double)(w * dg));
    }
    __syncthreads();
    for (int i = threadIdx.x; i < NET_NB; i += blockDim.x)
        if (hist[i] != 0.0) atomicAdd(tbar + i, hist[i]);
}

// F_d = -i k_d phi scale (field 0 holds phi on entry; fields fs apart).
__global__ void k_grad3(float2 *F, int64_t nhp, int64_t fs, int n, float scale)
{
    const int64_t tot = (int64_t)n * n * nhp;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
        const Mode m = mode_of(t, nhp, n);
        const float2 v = F[t];
        const float f0 = (m.pad || m.nyq0) ? 0.f : m.k0 * scale, f1 = (m.pad || m.nyq1) ? 0.f : m.k1 * scale,
                    f2 = (m.pad || m.nyq2) ? 0.f : m.k2 * scale;
        F[t] = make_float2(f0 * v.y, -f0 * v.x);
        F[fs + t] = make_float2(f1 * v.y, -f1 * v.x);
        F[2 * fs + t] = make_float2(f2 * v.y, -f2 * v.x);
    }
}

// F_d = -i k_d (A + B) scale for the sum of two spectra A (field 1) and B
// (field 2), written to fields 0, 1, 2 (fields fs apart); zero on the
// Nyquist plane of d.
__global__ void k_grad3_sum(float2 *F, int64_t nhp, int64_t fs, int n, float scale)
{
    const int64_t tot = (int64_t)n * n * nhp;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
        const Mode m = mode_of(t, nhp, n);
        const float2 a = F[fs + t], b = F[2 * fs + t];
        const float2 v = make_float2(a.x + b.x, a.y + b.y);
        const float f0 = (m.pad || m.nyq0) ? 0.f : m.k0 * scale, f1 = (m.pad || m.nyq1) ? 0.f : m.k1 * scale,
                    f2 = (m.pad || m.nyq2) ? 0.f : m.k2 * scale;
        F[t] = make_float2(f0 * v.y, -f0 * v.x);
        F[fs + t] = make_float2(f1 * v.y, -f1 * v.x);
        F[2 * fs + t] = make_float2(f2 * v.y, -f2 * v.x);
    }
}

// Transpose: phibar = sum_d i k_d Fbar_d scale into field 0.
__global__ void k_grad3_t(float2 *F, int64_t nhp, int64_t fs, int n, float scale)
{
    const int64_t tot = (int64_t)n * n * nhp;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tot; t += (int64_t)gridDim.x * blockDim.x) {
        const Mode m = mode_of(t, nhp, n);
        const float f0 = (m.pad || m.nyq0) ? 0.f : m.k0 * scale, f1 = (m.pad || m.nyq1) ? 0.f : m.k1 * scale,
                    f2 = (m.pad || m.nyq2) ? 0.f : m.k2 * scale;
        const float2 a = F[t], b = F[fs + t], c = F[2 * fs + t];
        const float sx = f0 * a.x + f1 * b.x + f2 * c.x, sy = f0 * a.y + f1 * b.y + f2 * c.y;
        F[t] = make_float2(-sy, sx);
    }
}

// ---------------------------------------------------------------- convolutions
// Voxel v = (i0 n + i1) n + i2; tap t = (t0 3 + t1) 3 + t2, offset t_e - 1.
constexpr int C2X = 16, C2Y = 8, C2HX = C2X + 2, C2HY = C2Y + 2;

// ---- inference path: no pre-activations kept, a1 never leaves LDS
// conv1 + conv2 on v_mfma_f32_16x16x32_bf16 (K = 32; lane l holds
// A[row l % 16][k 8 (l / 16) + j], B[k 8 (l / 16) + j][col l % 16] and
// D[row 4 (l / 16) + r][col l % 16]).  The 16 x 8 x IZ output tile of conv2
// needs a1 on the tile and its one-voxel halo (IHALO voxels); conv1 computes
// those from delta on a two-voxel halo staged in LDS as BF16, one MFMA per 16
// halo voxels: D[co][vox] = W1[co][tap] U[tap][vox] over 32 taps (27 real,
// weights zero past 26).  a1 sits in LDS as two planes of 8 channels (16 bytes
// per voxel), so the 16 lanes of a K group read 256 contiguous bytes.  conv2
// takes two taps per MFMA: k = 8 kg + j is tap 2 p + kg / 2, channel
// 8 (kg % 2) + j, so 14 MFMAs cover 27 taps (the 28th has zero weights); the
// 14 weight fragments live in registers.  Only a2 (BF16) is written.
#ifndef INF_Z
#define INF_Z 8
#endif
// Inference tile: 16 x 8 x IZ outputs on IZ wavefronts (one per z plane of
// conv2's output); the deeper the tile, the less of conv1's two-voxel halo is
// recomputed (2.1x the tile's voxels at IZ = 4, 1.76x at IZ = 8).
constexpr int IZ = INF_Z, INF_T = 64 * IZ, IHZ = IZ + 2, IHALO = C2HX * C2HY * IHZ;
constexpr int U1X = C2X + 4, U1Y = C2Y + 4, U1Z = IZ + 4, U1N = U1X * U1Y * U1Z;
constexpr int NG1 = (IHALO + 15) / 16, NPAIR = 14;
// Inference weights repacked once per call (byte offsets in wpk): conv2 as
// MFMA A fragments [pair][co][kg][8] BF16, conv1 [co][32 taps] BF16, conv3
// [t][ci] BF16.
constexpr int WPK_W2 = 0, WPK_W1 = NPAIR * NET_C * 4 * 8 * 2, WPK_W3 = WPK_W1 + NET_C * 32 * 2,
              WPK_END = WPK_W3 + 27 * NET_C * 2;
// The training forward's weights (k_pack_wf) around the same conv3 rows.
constexpr int WPK_W2F = 0, WPK_W1F = ((WPK_END + 63) / 64) * 64;
static_assert(WPK_END <= NET_WPK_BYTES && WPK_W1 % 16 == 0 && WPK_W3 % 16 == 0, "packed weight layout");
static_assert(27 * NET_C * NET_C * 2 <= WPK_W3 && WPK_W1F + 27 * NET_C * 4 <= NET_WPK_BYTES, "training weights");

// A grid of PACK_BLOCKS workgroups (one would wait on its strided weight
// reads for 32 rounds).
constexpr int PACK_BLOCKS = 32;
__global__ __launch_bounds__(256) void k_pack_w(const float *__restrict__ th, uint16_t *wpk)
{
    uint16_t *w2 = wpk + WPK_W2 / 2, *w1 = wpk + WPK_W1 / 2, *w3 = wpk + WPK_W3 / 2;
    const int e0 = blockIdx.x * 256 + threadIdx.x, es = PACK_BLOCKS * 256;
    for (int e = e0; e < NPAIR * NET_C * 4 * 8; e += es) {
        const int pr = e / (NET_C * 32), co = (e / 32) % NET_C, kg = (e / 8) % 4, j = e % 8;
        const int t = 2 * pr + kg / 2, ci = 8 * (kg % 2) + j;
        w2[e] = t < 27 ? to_bf16(th[NC2W + (co * NET_C + ci) * 27 + t]) : (uint16_t)0;
    }
    for (int e = e0; e < NET_C * 32; e += es) {
        const int co = e / 32, t = e % 32;
        w1[e] = t < 27 ? to_bf16(th[NC1W + co * 27 + t]) : (uint16_t)0;
    }
    for (int e = e0; e < 27 * NET_C; e += es) {
        const int t = e / NET_C, ci = e % NET_C;
        w3[e] = to_bf16(th[NC3W + ci * 27 + t]);
    }
}

__device__ __forceinline__ int u1_off(int t) { return ((t / 9) * U1Y + (t / 3) % 3) * U1X + t % 3; }
__device__ __forceinline__ int x_off(int t) { return ((t / 9) * C2HY + (t / 3) % 3) * C2HX + t % 3; }

// SRC int64_t: the fixed-point density, delta = q qs - 1 formed here; SRC
// float: the density contrast as the tile paint stores it (the same value).
template <typename SRC>
__global__ __launch_bounds__(INF_T) void k_cnn12_inf(const SRC *__restrict__ q, double qs, int n,
                                                   const float *__restrict__ th, const uint16_t *__restrict__ wpk,
                                                   uint16_t *a2)
{
    __shared__ __align__(16) uint16_t U[U1N];
    __shared__ __align__(16) uint4 X[2 * IHALO];   // channel planes 0-7 and 8-15
    const int tid = threadIdx.x;
    const int ntx = n / C2X, nty = n / C2Y;
    const int tile = blockIdx.x;
    const int tx = tile % ntx, ty = (tile / ntx) % nty, tz = tile / (ntx * nty);
    const int x0 = tx * C2X, y0 = ty * C2Y, z0 = tz * IZ, m = n - 1;
    const int lane = tid & 63, wave = tid >> 6;
    constexpr int NW = INF_T / 64;   // wavefronts
    const int col = lane & 15, kg = lane >> 4;
    // weight fragments straight from the packed buffer (L2-resident)
    const v8bf w1 = *reinterpret_cast<const v8bf *>(wpk + WPK_W1 / 2 + col * 32 + 8 * kg);
    v8bf wa[NPAIR];
#pragma unroll
    for (int pr = 0; pr < NPAIR; pr++)
        wa[pr] = *reinterpret_cast<const v8bf *>(wpk + WPK_W2 / 2 + ((pr * NET_C + col) * 4 + kg) * 8);
    {
        // every load of the halo fill issued before the first LDS store (one
        // memory round trip per tile rather than one per round); indices past
        // the end are clamped, and the empty asm keeps the loads from being
        // sunk into the guarded stores
        constexpr int NU = (U1N + INF_T - 1) / INF_T;
        SRC qv[NU];
#pragma unroll
        for (int k = 0; k < NU; k++) {
            const int e = min(tid + INF_T * k, U1N - 1);
            const int eq = Div24<U1X, U1N>::div(e), uz = Div24<U1Y, U1N / U1X>::div(eq);
            const int ux = e - __mul24(eq, U1X), uy = eq - __mul24(uz, U1Y);
            qv[k] = q[vox_index((z0 + uz - 2) & m, (y0 + uy - 2) & m, (x0 + ux - 2) & m, n)];
        }
#pragma unroll
        for (int k = 0; k < NU; k++) asm volatile("" : "+v"(qv[k]));
#pragma unroll
        for (int k = 0; k < NU; k++) {
            const int e = tid + INF_T * k;
            if constexpr (std::is_same<SRC, int64_t>::value) {
                if (e < U1N) U[e] = delta_bf16(qv[k], qs);
            } else {
                if (e < U1N) U[e] = to_bf16(qv[k]);
            }
        }
    }
    __syncthreads();
    {
        // taps 27..31 read a real voxel (tap 26's) against zero weights, so
        // every lane's eight reads are unconditional (no exec-mask branches)
        int ou[8];
#pragma unroll
        for (int j = 0; j < 8; j++) ou[j] = u1_off(8 * kg + j < 27 ? 8 * kg + j : 26);
        float bias[4];
#pragma unroll
        for (int r = 0; r < 4; r++) bias[r] = th[NC1B + 4 * kg + r];
        for (int g = wave; g < NG1; g += NW) {
            const int hv = g * 16 + col;
            const int hc = hv < IHALO ? hv : IHALO - 1;
            const int hq = Div24<C2HX, IHALO>::div(hc), hz = Div24<C2HY, IHALO / C2HX>::div(hq);
            const int hx = hc - __mul24(hq, C2HX), hy = hq - __mul24(hz, C2HY);
            const int base = __mul24(__mul24(hz, U1Y) + hy, U1X) + hx;
            v8bf b;
#pragma unroll
            for (int j = 0; j < 8; j++) b[j] = __builtin_bit_cast(__bf16, U[base + ou[j]]);
            v4f acc = {0.f, 0.f, 0.f, 0.f};
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, b, acc, 0, 0, 0);
            // lane holds D[co = 4 kg + r][vox = col]: channels 4 kg .. 4 kg + 3
            if (hv < IHALO) {
                uint16_t aa[4];
#pragma unroll
                for (int r = 0; r < 4; r++) aa[r] = to_bf16(silu(acc[r] + bias[r]));
                reinterpret_cast<uint2 *>(X + (kg >> 1) * IHALO + hv)[kg & 1] =
                    make_uint2((uint32_t)aa[0] | ((uint32_t)aa[1] << 16), (uint32_t)aa[2] | ((uint32_t)aa[3] << 16));
            }
        }
    }
    __syncthreads();
    int ox[NPAIR];
#pragma unroll
    for (int pr = 0; pr < NPAIR; pr++) {
        const int t = 2 * pr + (kg >> 1);
        ox[pr] = x_off(t < 27 ? t : 26);   // the 28th tap reads real data against zero weights
    }
    // wavefront w computes the output rows y = w of every z plane: with the
    // loop unrolled, a row's LDS offsets are the loop-invariant lane offsets
    // plus an immediate, and the output pointer steps by one plane
    static_assert(NW == C2Y, "one wavefront per output row of a plane");
    const uint4 *Xp = X + (kg & 1) * IHALO + wave * C2HX + col;
    float bias[4];
#pragma unroll
    for (int r = 0; r < 4; r++) bias[r] = th[NC2B + 4 * kg + r];
    uint16_t *out = a2 + ((((int64_t)z0 * n + (y0 + wave)) * n + (x0 + col)) * NET_C + 4 * kg);
    const int64_t plane_step = (int64_t)n * n * NET_C;
#pragma unroll
    for (int rz = 0; rz < IZ; rz++) {
        const uint4 *xr = Xp + rz * (C2HY * C2HX);
        v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int pr = 0; pr < NPAIR; pr++) {
            const v8bf xb = __builtin_bit_cast(v8bf, xr[ox[pr]]);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[pr], xb, acc, 0, 0, 0);
        }
        uint16_t aa[4];
#pragma unroll
        for (int r = 0; r < 4; r++) aa[r] = to_bf16(silu(acc[r] + bias[r]));
        *reinterpret_cast<uint2 *>(out) =
            make_uint2((uint32_t)aa[0] | ((uint32_t)aa[1] << 16), (uint32_t)aa[2] | ((uint32_t)aa[3] << 16));
        out += plane_step;
    }
}

// conv3 fused with the combination: out = phi_f + b3 + conv3(a2) on
// real rows of stride rs.  Tile 16 x 16 x 4 with a2's one-voxel halo in LDS;
// a thread owns a column of 4 voxels along axis 0, so each halo voxel it reads
// feeds up to three taps.
// Tile 16 x TY x TZ with a2's one-voxel halo in LDS; 256 threads, each owning
// ZPT consecutive voxels along axis 0 of one (axis 1, axis 2) column, so each
// halo voxel it reads feeds up to three taps.
template <int TY, int TZ, int ZPT>
__global__ __launch_bounds__(256) void k_conv3_inf(const uint16_t *__restrict__ a2, int n,
                                                   const float *__restrict__ th, const uint16_t *__restrict__ wpk,
                                                   const float *__restrict__ phif, int64_t rs, float *out)
{
    static_assert(16 * TY * (TZ / ZPT) == 256 && TZ % ZPT == 0, "conv3 tile shape");
    constexpr int HX = 18, HY = TY + 2, HZ = TZ + 2, HALO = HX * HY * HZ;
    // channel halves of each halo voxel in two planes: 16-byte rows, no bank conflicts
    // + one slot per lane after the two planes (stores of idle fill tasks)
    __shared__ __align__(16) uint4 X[2 * HALO + 64];
    __shared__ __align__(16) uint32_t W[27 * NET_C / 2];   // BF16 pairs [t][ci / 2]
    const int tid = threadIdx.x;
    const int ntx = n / 16, nty = n / TY;
    const int tile = blockIdx.x;
    const int tx = tile % ntx, ty = (tile / ntx) % nty, tz = tile / (ntx * nty);
    const int x0 = tx * 16, y0 = ty * TY, z0 = tz * TZ, m = n - 1;
    const int lx = tid % 16, ly = (tid / 16) % TY, zg = tid / (16 * TY);
    // phi_f of the thread's voxels, loaded now rather than after the sums
    float pf[ZPT];
#pragma unroll
    for (int z = 0; z < ZPT; z++)
        pf[z] = phif ? phif[((int64_t)(z0 + zg * ZPT + z) * n + (y0 + ly)) * rs + (x0 + lx)] : 0.f;
    {
        // Every load of the halo fill is issued before the first LDS store
        // (one memory round trip per tile, not one per round).  Indices past
        // the end are clamped, and those lanes store to their own slot after
        // the tile, so no store is guarded (a guarded store would let the
        // compiler sink its load into the guard).
        constexpr int NX = (HALO * 2 + 255) / 256;
        uint4 xv[NX];
#pragma unroll
        for (int k = 0; k < NX; k++) {
            const int e = min(tid + 256 * k, HALO * 2 - 1);
            const int hv = e >> 1, half = e & 1;
            const int hq = Div24<HX, HALO>::div(hv), hz = Div24<HY, HALO / HX>::div(hq);
            const int hx = hv - __mul24(hq, HX), hy = hq - __mul24(hz, HY);
            const int64_t g = vox_index((z0 + hz - 1) & m, (y0 + hy - 1) & m, (x0 + hx - 1) & m, n);
            xv[k] = reinterpret_cast<const uint4 *>(a2 + g * NET_C)[half];
        }
        // the conv3 weights, one 16-byte row per thread, unconditional like
        // the halo (lanes past the last row store to their slot after the tile)
        constexpr int NW = 27 * NET_C / 8;
        static_assert(NW <= 256, "one weight row per thread");
        const uint4 wv = reinterpret_cast<const uint4 *>(wpk + WPK_W3 / 2)[min(tid, NW - 1)];
        *(tid < NW ? reinterpret_cast<uint4 *>(W) + tid : X + 2 * HALO + (tid & 63)) = wv;
#pragma unroll
        for (int k = 0; k < NX; k++) {
            const int e = tid + 256 * k;
            X[e < HALO * 2 ? (e & 1) * HALO + (e >> 1) : 2 * HALO + (tid & 63)] = xv[k];
        }
    }
    __syncthreads();
    const float b = th[NC3B];
    float acc[ZPT];
#pragma unroll
    for (int z = 0; z < ZPT; z++) acc[z] = b;
#pragma unroll 1
    for (int t2 = 0; t2 < 9; t2++) {
        const int dy = t2 / 3, dx = t2 % 3;
        uint32_t w[3][NET_C / 2];
#pragma unroll
        for (int dz = 0; dz < 3; dz++)
#pragma unroll
            for (int k = 0; k < NET_C / 2; k++) w[dz][k] = W[(dz * 9 + t2) * (NET_C / 2) + k];
        const int h0 = (zg * ZPT * HY + ly + dy) * HX + lx + dx;
#pragma unroll
        for (int j = 0; j < ZPT + 2; j++) {
            const int hv = h0 + j * HY * HX;
            const uint4 q0 = X[hv], q1 = X[HALO + hv];
            const uint32_t xv[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
#pragma unroll
            for (int dz = 0; dz < 3; dz++) {
                const int lz = j - dz;
                if (lz < 0 || lz >= ZPT) continue;
                float sum = acc[lz];
#pragma unroll
                for (int k = 0; k < NET_C / 2; k++) sum = dot2_bf16(w[dz][k], xv[k], sum);
                acc[lz] = sum;
            }
        }
    }
#pragma unroll
    for (int z = 0; z < ZPT; z++) {
        const int64_t o = ((int64_t)(z0 + zg * ZPT + z) * n + (y0 + ly)) * rs + (x0 + lx);
        out[o] = pf[z] + acc[z];
    }
}

// Measured at 256^3 (one MI355X): 16 x 8 x 4 with two voxels per thread
// (35 KB of LDS, four workgroups per CU) 306 us; 16 x 16 x 4 with four per
// thread (63 KB, two per CU) 418 us; one voxel per thread 360 us.
constexpr int C3TY = 8, C3TZ = 4, C3ZPT = 2;

// ---- training forward: z1, a1, z2 and a2 are stored for the reverse mode.  The
// activations are rounded to BF16, so a pre-activation that moves by an FP32
// rounding can move its activation by 2^-8: the sums keep one fixed order
// (conv1: the taps in turn, from the bias; conv2: one 16x16x16 product per tap
// in turn, then the bias).
//
// conv1: tile 16 x 8 x 4 with delta's halo in LDS, two voxels per thread; the
// weights are wave-uniform, so a tap is one FMA with a scalar operand per
// channel (432 per voxel).  Bound by the writes of z1 and a1 (96 bytes per voxel).
constexpr int T1Y = 8, T1Z = 4;
template <typename SRC>
__global__ __launch_bounds__(256) void k_conv1_fwd(const SRC *__restrict__ q, double qs, int n,
                                                   const float *__restrict__ th, const uint16_t *__restrict__ wpk,
                                                   float *z1, uint16_t *a1)
{
    constexpr int HX = 18, HY = T1Y + 2, HZ = T1Z + 2, NH = HX * HY * HZ, NU = (NH + 255) / 256;
    __shared__ float U[NH];
    const int tid = threadIdx.x, m = n - 1;
    const int tile = xcd_tile(blockIdx.x, gridDim.x), ntx = n / 16, nty = n / T1Y;
    const int x0 = (tile % ntx) * 16, y0 = ((tile / ntx) % nty) * T1Y, z0 = (tile / (ntx * nty)) * T1Z;
    SRC qv[NU];
#pragma unroll
    for (int k = 0; k < NU; k++) {
        const int e = min(tid + 256 * k, NH - 1);
        const int hq = Div24<HX, NH>::div(e), hz = Div24<HY, HY * HZ>::div(hq), hx = e - hq * HX, hy = hq - hz * HY;
        qv[k] = q[vox_index((z0 + hz - 1) & m, (y0 + hy - 1) & m, (x0 + hx - 1) & m, n)];
    }
#pragma unroll
    for (int k = 0; k < NU; k++) {
        uint16_t d;
        if constexpr (std::is_same<SRC, int64_t>::value) d = delta_bf16(qv[k], qs);
        else d = to_bf16(qv[k]);
        if (tid + 256 * k < NH) U[tid + 256 * k] = from_bf16(d);
    }
    __syncthreads();
    const int lx = tid & 15, ly = (tid >> 4) & 7, lz = (tid >> 7) * 2;
    float z[2][NET_C];
#pragma unroll
    for (int c = 0; c < NET_C; c++) z[0][c] = z[1][c] = th[NC1B + c];
    const float *w = reinterpret_cast<const float *>(wpk + WPK_W1F / 2);
#pragma unroll 3
    for (int t = 0; t < 27; t++) {
        const float *u = U + ((lz + t / 9) * HY + ly + (t / 3) % 3) * HX + lx + t % 3;
        const float u0 = u[0], u1 = u[HY * HX];
#pragma unroll
        for (int c = 0; c < NET_C; c++) {
            const float wc = w[t * NET_C + c];
            z[0][c] = fmaf(wc, u0, z[0][c]);
            z[1][c] = fmaf(wc, u1, z[1][c]);
        }
    }
#pragma unroll
    for (int p = 0; p < 2; p++) {
        const int64_t v = vox_index(z0 + lz + p, y0 + ly, x0 + lx, n) * NET_C;
#pragma unroll
        for (int c = 0; c < NET_C; c += 4) {
            *reinterpret_cast<float4 *>(z1 + v + c) = make_float4(z[p][c], z[p][c + 1], z[p][c + 2], z[p][c + 3]);
            const uint32_t lo = (uint32_t)to_bf16(silu(z[p][c])) | ((uint32_t)to_bf16(silu(z[p][c + 1])) << 16);
            const uint32_t hi = (uint32_t)to_bf16(silu(z[p][c + 2])) | ((uint32_t)to_bf16(silu(z[p][c + 3])) << 16);
            *reinterpret_cast<uint2 *>(a1 + v + c) = make_uint2(lo, hi);
        }
    }
}

// conv2: tile 16 x 8 x 4 with a1's halo in LDS, the 27 weight fragments in
// registers.  Per 16-voxel row and tap D[co][vox] += W_t[co][ci] X_t[ci][vox]
// (lane l holds A[co = l % 16][ci = 4 (l / 16) + r], B[ci = 4 (l / 16) + r][vox =
// l % 16] and D[co = 4 (l / 16) + r][vox = l % 16]); two rows in flight.  Bound by
// the writes of z2 and a2 and the read of a1.
__global__ __launch_bounds__(256, 2) void k_conv2_fwd(const uint16_t *__restrict__ a1, int n,
                                                     const float *__restrict__ th, const uint16_t *__restrict__ wpk,
                                                     float *z2, uint16_t *a2)
{
    constexpr int HX = 18, HY = 10, HZ = 6, NH = HX * HY * HZ, NX = (2 * NH + 255) / 256;
    __shared__ __align__(16) uint4 X[2 * NH];
    const int tid = threadIdx.x, m = n - 1;
    const int tile = xcd_tile(blockIdx.x, gridDim.x), ntx = n / 16, nty = n / 8;
    const int x0 = (tile % ntx) * 16, y0 = ((tile / ntx) % nty) * 8, z0 = (tile / (ntx * nty)) * 4;
    uint4 xv[NX];
#pragma unroll
    for (int k = 0; k < NX; k++) {
        const int e = min(tid + 256 * k, 2 * NH - 1), hv = e >> 1;
        const int hq = Div24<HX, NH>::div(hv), hz = Div24<HY, HY * HZ>::div(hq), hx = hv - hq * HX, hy = hq - hz * HY;
        xv[k] = reinterpret_cast<const uint4 *>(
            a1 + vox_index((z0 + hz - 1) & m, (y0 + hy - 1) & m, (x0 + hx - 1) & m, n) * NET_C)[e & 1];
    }
    const int lane = tid & 63, wave = tid >> 6, col = lane & 15, kg = lane >> 4;
    v4s w[27];
#pragma unroll
    for (int t = 0; t < 27; t++)
        w[t] = *reinterpret_cast<const v4s *>(wpk + WPK_W2F / 2 + (t * NET_C + col) * NET_C + 4 * kg);
    float bias[4];
#pragma unroll
    for (int r = 0; r < 4; r++) bias[r] = th[NC2B + 4 * kg + r];
#pragma unroll
    for (int k = 0; k < NX; k++)
        if (tid + 256 * k < 2 * NH) X[tid + 256 * k] = xv[k];
    __syncthreads();
    // wavefront w takes the rows (y = 2 w, 2 w + 1) of each plane
    const v4s *Xp = reinterpret_cast<const v4s *>(X) + (2 * wave * HX + col) * 4 + kg;
#pragma unroll 1
    for (int z = 0; z < 4; z++) {
        v4f acc[2] = {};
#pragma unroll
        for (int t = 0; t < 27; t++) {
            const v4s *p = Xp + (((z + t / 9) * HY + (t / 3) % 3) * HX + t % 3) * 4;
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[t], p[0], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[t], p[4 * HX], acc[1], 0, 0, 0);
        }
#pragma unroll
        for (int y = 0; y < 2; y++) {
            const int64_t v = vox_index(z0 + z, y0 + 2 * wave + y, x0 + col, n) * NET_C + 4 * kg;
            float zz[4];
            uint16_t aa[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                zz[r] = acc[y][r] + bias[r];
                aa[r] = to_bf16(silu(zz[r]));
            }
            *reinterpret_cast<float4 *>(z2 + v) = make_float4(zz[0], zz[1], zz[2], zz[3]);
            *reinterpret_cast<uint2 *>(a2 + v) =
                make_uint2((uint32_t)aa[0] | ((uint32_t)aa[1] << 16), (uint32_t)aa[2] | ((uint32_t)aa[3] << 16));
        }
    }
}

// Weights of the training forward: conv1 [t][co] FP32 (BF16-rounded), conv2
// [t][co][ci] BF16, conv3 [t][ci] BF16 where the inference layout has it.
__global__ __launch_bounds__(256) void k_pack_wf(const float *__restrict__ th, uint16_t *wpk)
{
    float *w1 = reinterpret_cast<float *>(wpk + WPK_W1F / 2);
    uint16_t *w2 = wpk + WPK_W2F / 2, *w3 = wpk + WPK_W3 / 2;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < 27 * NET_C * NET_C) {
        const int t = e / (NET_C * NET_C), co = (e / NET_C) % NET_C, ci = e % NET_C;
        w2[e] = to_bf16(th[NC2W + (co * NET_C + ci) * 27 + t]);
    }
    if (e < 27 * NET_C) {
        w1[e] = bf16r(th[NC1W + (e % NET_C) * 27 + e / NET_C]);
        w3[e] = to_bf16(th[NC3W + (e % NET_C) * 27 + e / NET_C]);
    }
}

// ---- loss and optimiser
// red[0] += sum (acc - target)^2, red[1] += sum target^2; acc -= target.
__global__ __launch_bounds__(256) void k_force_loss(float *acc, const float *target, int64_t n3, double *red)
{
    __shared__ double sa[256], sb[256];
    double a = 0.0, b = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n3; i += (int64_t)gridDim.x * blockDim.x) {
        const float d = acc[i] - target[i];
        a += (double)d * d;
        b += (double)target[i] * target[i];
        acc[i] = d;
    }
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s) {
            sa[threadIdx.x] += sa[threadIdx.x + s];
            sb[threadIdx.x] += sb[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomicAdd(red, sa[0]);
        atomicAdd(red + 1, sb[0]);
    }
}

// Adam with bias correction (FP32 master weights).
__global__ void k_adam(float *th, float *m, float *v, const float *g, int64_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

__global__ void k_zero_f64(double *p, int n)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0.0;
}

}  // namespace

hipError_t launch_mlp_fwd(const float *th, double a, float *table, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_fwd, dim3(NET_NB), dim3(128), 0, s, th, (float)a, table);
    return hipGetLastError();
}

hipError_t launch_mlp_bwd(const float *th, double a, const double *tbar, float *dth, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_bwd, dim3(NET_NB / MB_BINS), dim3(MB_T), 0, s, th, (float)a, tbar, dth);
    return hipGetLastError();
}

hipError_t launch_spec_filter(const float2 *in, float2 *out, int64_t nhp, int n, const float *table, double coef,
                              hipStream_t s)
{
    const int64_t tot = (int64_t)n * n * nhp;
    hipLaunchKernelGGL(k_spec_filter, dim3(grid_for(tot, 256, 4096)), dim3(256), 0, s, in, out, nhp, n, table,
                       (float)coef);
    return hipGetLastError();
}

hipError_t launch_spec_filter_bwd(const float2 *dk, const float2 *pf, int64_t nhp, int n, double coef, double *tbar,
                                  hipStream_t s)
{
    const int64_t tot = (int64_t)n * n * nhp;
    hipLaunchKernelGGL(k_zero_f64, dim3(1), dim3(256), 0, s, tbar, NET_NB);
    hipLaunchKernelGGL(k_spec_filter_bwd, dim3(grid_for(tot, 256, 1024)), dim3(256), 0, s, dk, pf, nhp, n,
                       (float)coef, tbar);
    return hipGetLastError();
}

hipError_t launch_grad3_sum(float2 *F, int64_t nhp, int64_t fs, int n, double scale, hipStream_t s)
{
    const int64_t tot = (int64_t)n * n * nhp;
    hipLaunchKernelGGL(k_grad3_sum, dim3(grid_for(tot, 256)), dim3(256), 0, s, F, nhp, fs, n, (float)scale);
    return hipGetLastError();
}

hipError_t launch_grad3(float2 *F, int64_t nhp, int64_t fs, int n, double scale, bool transpose, hipStream_t s)
{
    const int64_t tot = (int64_t)n * n * nhp;
    if (transpose)
        hipLaunchKernelGGL(k_grad3_t, dim3(grid_for(tot, 256)), dim3(256), 0, s, F, nhp, fs, n, (float)scale);
    else
        hipLaunchKernelGGL(k_grad3, dim3(grid_for(tot, 256)), dim3(256), 0, s, F, nhp, fs, n, (float)scale);
    return hipGetLastError();
}

hipError_t launch_cnn_inf(const int64_t *q, double qs, const float *delta, const float *phif, int64_t rs, int n,
                          const float *th, uint16_t *wpk, uint16_t *a2, float *out, hipStream_t s)
{
    if (n < 16 || n % 16 || n > 4096) return hipErrorInvalidValue;
    const int64_t M = (int64_t)n * n * n;
    const dim3 grid((unsigned)(M / (C2X * C2Y * IZ)));
    hipLaunchKernelGGL(k_pack_w, dim3(PACK_BLOCKS), dim3(256), 0, s, th, wpk);
    if (delta)
        hipLaunchKernelGGL(k_cnn12_inf<float>, grid, dim3(INF_T), 0, s, delta, qs, n, th, wpk, a2);
    else
        hipLaunchKernelGGL(k_cnn12_inf<int64_t>, grid, dim3(INF_T), 0, s, q, qs, n, th, wpk, a2);
    hipLaunchKernelGGL((k_conv3_inf<C3TY, C3TZ, C3ZPT>), dim3((unsigned)(M / (16 * C3TY * C3TZ))), dim3(256), 0, s, a2,
                       n, th, wpk, phif, rs, out);
    return hipGetLastError();
}

hipError_t launch_cnn_fwd(const int64_t *q, double qs, const float *delta, const float *phif, int64_t rs, int n,
                          const float *th, uint16_t *wpk, float *z1, uint16_t *a1, float *z2, uint16_t *a2, float *out, hipStream_t s)
{
    if (n < 16 || n % 16 || n > 4096) return hipErrorInvalidValue;
    const int64_t M = (int64_t)n * n * n;
    hipLaunchKernelGGL(k_pack_wf, dim3(27), dim3(256), 0, s, th, wpk);
    const dim3 g1((unsigned)(M / (16 * T1Y * T1Z))), g2((unsigned)(M / (16 * 8 * 4)));
    if (delta)
        hipLaunchKernelGGL(k_conv1_fwd<float>, g1, dim3(256), 0, s, delta, qs, n, th, wpk, z1, a1);
    else
        hipLaunchKernelGGL(k_conv1_fwd<int64_t>, g1, dim3(256), 0, s, q, qs, n, th, wpk, z1, a1);
    hipLaunchKernelGGL(k_conv2_fwd, g2, dim3(256), 0, s, a1, n, th, wpk, z2, a2);
    hipLaunchKernelGGL((k_conv3_inf<C3TY, C3TZ, C3ZPT>), dim3((unsigned)(M / (16 * C3TY * C3TZ))), dim3(256), 0, s, a2,
                       n, th, wpk, phif, rs, out);
    return hipGetLastError();
}

hipError_t launch_zero_f64(double *p, int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_f64, dim3(1), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_force_loss(float *acc, const float *target, int64_t n3, double *red, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_f64, dim3(1), dim3(64), 0, s, red, 2);
    hipLaunchKernelGGL(k_force_loss, dim3(grid_for(n3, 256, 2048)), dim3(256), 0, s, acc, target, n3, red);
    return hipGetLastError();
}

hipError_t launch_adam(float *th, float *m, float *v, const float *g, int64_t n, double lr, double b1, double b2,
                       double eps, int t, hipStream_t s)
{
    const float c1 = (float)(1.0 - pow(b1, t)), c2 = (float)(1.0 - pow(b2, t));
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n, 256)), dim3(256), 0, s, th, m, v, g, n, (float)lr, (float)b1,
                       (float)b2, (float)eps, c1, c2);
    return hipGetLastError();
}

}  // namespace pm
