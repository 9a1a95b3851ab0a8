// Reverse mode of the learned correction's CNN on the matrix cores.
//
// Cotangents are FP32, activations and weights BF16.  An FP32 value is the
// exact sum of three BF16 values (its significand's 24 bits in three groups of
// eight), so every product of a cotangent with an activation or a weight is
// three exact BF16 products, accumulated in FP32 by v_mfma_f32_16x16x32_bf16:
// the arithmetic of an FP32 product-sum at a third of the BF16 rate.
//
// Three kernels and a reduction, each walking tiles of the mesh:
//   k_conv3_bwd    g2 = SiLU'(z2) W3^T phibar, and dW3, db3
//   k_conv2_bwd_w  dW2, db2 from a1 and g2
//   k_conv2_bwd_d  g1 = SiLU'(z1) W2^T g2, and dW1, db1 from g1 and delta; g1
//                  itself is never stored
// Workgroups keep their share of a weight gradient in accumulator registers
// over all their tiles and write it once to a partial buffer; k_bwd_reduce
// adds the partials in a fixed order.
//
// Fragment layouts (lane l, col = l % 16, kg = l / 16): A[row col][k 8 kg + j],
// B[k 8 kg + j][column col], D[row 4 kg + r][column col].  Where the summed
// index is the voxel, the channel-contiguous LDS rows are read transposed
// (ds_read_b64_tr_b16: each group of 16 lanes reads four rows of 16 channels,
// eight bytes per lane, and lane i receives channel i of the four rows).
//
// At 256^3 (one training step's reverse mode, us): k_conv3_bwd 615 (two
// kernels of FP32 loops over LDS before: 8640), k_conv2_bwd_w 766 (108700),
// k_conv2_bwd_d 1230 (two kernels: 7220).  Against 64-bit sums of the same
// BF16 inputs at 16^3 the weight gradients are off by 1.6e-7 to 2.5e-7 (FP32
// loops: 3.9e-7 to 5.3e-7).
#include "net_common.h"

namespace pm {
namespace {

typedef __attribute__((address_space(3))) v4s lds_v4s;

// Four values of one channel from four consecutive LDS rows; p is this lane's
// eight bytes of row (l % 16) / 4.
__device__ __forceinline__ v4s read_tr(const void *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)p);
}
__device__ __forceinline__ v8bf join(v4s a, v4s b)
{
    return __builtin_bit_cast(v8bf, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// a = h + m + l and b likewise, h, m and l the successive 8-bit groups of the
// significand (truncated, so no group can overflow), packed in pairs.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
    const float ra = a - __uint_as_float(ua & 0xffff0000u), rb = b - __uint_as_float(ub & 0xffff0000u);
    const uint32_t va = __float_as_uint(ra), vb = __float_as_uint(rb);
    const float sa = ra - __uint_as_float(va & 0xffff0000u), sb = rb - __uint_as_float(vb & 0xffff0000u);
    h = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
    m = __builtin_amdgcn_perm(vb, va, 0x07060302u);
    l = __builtin_amdgcn_perm(__float_as_uint(sb), __float_as_uint(sa), 0x07060302u);
}
__device__ __forceinline__ void split8(const float v[8], v8bf s[3])
{
    uint32_t u[3][4];
#pragma unroll
    for (int j = 0; j < 4; j++) split_pair(v[2 * j], v[2 * j + 1], u[0][j], u[1][j], u[2][j]);
#pragma unroll
    for (int i = 0; i < 3; i++) s[i] = __builtin_bit_cast(v8bf, make_uint4(u[i][0], u[i][1], u[i][2], u[i][3]));
}

__device__ __forceinline__ v4f mfma32(v8bf a, v8bf b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Sum over the four 16-lane groups: every lane holds its column's sum.
__device__ __forceinline__ double sum_groups(double v)
{
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// ---------------------------------------------------------------- conv3
// Tile 16 x 8 x 8 (x, y, z), four wavefronts.  P holds, per split and halo row
// (z, y), the triples phibar(x - 1 .. x + 1) of the 16 voxels as four BF16
// (the fourth zero): one eight-byte read is a row of three taps, for g2
// directly (k = taps) and transposed for dW3 (k = voxels).  71 KB of LDS, two
// workgroups per CU; bound by the reads of z2 and a2 and the write of g2.
constexpr int B3Y = 8, B3Z = 8, B3HY = B3Y + 2, B3ROWS = B3HY * (B3Z + 2);
constexpr int DW3_N = NET_C * 27 + 1;   // a workgroup's partial: [ci][27] then db3

__global__ __launch_bounds__(256, 2) void k_conv3_bwd(const float *__restrict__ phibar, int64_t rs, int n,
                                                     const float *__restrict__ th, const float *__restrict__ z2,
                                                     const uint16_t *__restrict__ a2, float *__restrict__ g2,
                                                     float *part)
{
    __shared__ __align__(16) uint2 P[3][B3ROWS * 16];
    __shared__ __align__(16) uint4 A[16 * B3Y * B3Z * 2];
    __shared__ float red[NET_C * 48 + 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, kg = lane >> 4, m = n - 1;
    const int ntx = n / 16, nty = n / B3Y, ntiles = ntx * nty * (n / B3Z);
    // B[k = taps][ci] of g2: tap row 2 kg + j / 4, dx = j % 4, of the mirrored
    // weights; w8: the ninth row in k < 4, zero elsewhere (a 16x16x16 product
    // would do, but where the compiler chained it with 16x16x32 ones through
    // the accumulator, its last two rows were read before they were written)
    v8bf w, w8;
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int t = (2 * kg + (j >> 2)) * 3 + (j & 3);
        w[j] = (__bf16)((j & 3) < 3 ? th[NC3W + col * 27 + 26 - t] : 0.f);
    }
#pragma unroll
    for (int j = 0; j < 8; j++) w8[j] = (__bf16)(kg == 0 && j < 3 ? th[NC3W + col * 27 + 2 - j] : 0.f);
    // halo row offsets (in 16-voxel rows) of this lane's tap rows
    const int r0 = 2 * kg, r1 = 2 * kg + 1;
    const int o0 = (r0 / 3) * B3HY + r0 % 3, o1 = (r1 / 3) * B3HY + r1 % 3, o8 = 2 * B3HY + 2;
    int ot[3];   // dW3, column tile c: tap row 4 c + lane % 4 (rows past the ninth repeat it, unused)
#pragma unroll
    for (int c = 0; c < 3; c++) {
        const int r = min(4 * c + (col & 3), 8);
        ot[c] = (r / 3) * B3HY + r % 3;
    }
    v4f acc[3] = {};
    double db = 0.0;
    for (int tile = xcd_tile(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const int x0 = (tile % ntx) * 16, y0 = ((tile / ntx) % nty) * B3Y, z0 = (tile / (ntx * nty)) * B3Z;
        {
            // all loads before the first LDS store: one memory round trip
            constexpr int NP = (B3ROWS * 16 + 255) / 256, NA = 16 * B3Y * B3Z * 2 / 256;
            float pv[NP][3];
            uint4 av[NA];
#pragma unroll
            for (int k = 0; k < NP; k++) {
                const int e = min(tid + 256 * k, B3ROWS * 16 - 1);
                const int row = e >> 4, x = e & 15, hz = Div24<B3HY, B3ROWS>::div(row), hy = row - hz * B3HY;
                const float *src = phibar + ((int64_t)((z0 + hz - 1) & m) * n + ((y0 + hy - 1) & m)) * rs;
                pv[k][0] = src[(x0 + x - 1) & m];
                pv[k][1] = src[x0 + x];
                pv[k][2] = src[(x0 + x + 1) & m];
            }
#pragma unroll
            for (int k = 0; k < NA; k++) {
                const int e = tid + 256 * k, row = e >> 5, y = row % B3Y, z = row / B3Y;
                av[k] = reinterpret_cast<const uint4 *>(a2 + vox_index(z0 + z, y0 + y, x0, n) * NET_C)[e & 31];
            }
#pragma unroll
            for (int k = 0; k < NP; k++) {
                const int e = tid + 256 * k;
                if (e < B3ROWS * 16) {
                    const int row = e >> 4, hz = Div24<B3HY, B3ROWS>::div(row), hy = row - hz * B3HY;
                    uint2 h, mm, l;
                    split_pair(pv[k][0], pv[k][1], h.x, mm.x, l.x);
                    split_pair(pv[k][2], 0.f, h.y, mm.y, l.y);
                    P[0][e] = h;
                    P[1][e] = mm;
                    P[2][e] = l;
                    if (hz >= 1 && hz <= B3Z && hy >= 1 && hy <= B3Y) db += pv[k][1];
                }
            }
#pragma unroll
            for (int k = 0; k < NA; k++) A[tid + 256 * k] = av[k];
        }
        __syncthreads();
        for (int c = wave; c < B3Y * B3Z / 2; c += 4) {
            const int z = c / (B3Y / 2), y = 2 * (c % (B3Y / 2));
            float zz[2][4];
#pragma unroll
            for (int q = 0; q < 2; q++)
#pragma unroll
                for (int r = 0; r < 4; r++)
                    zz[q][r] = z2[vox_index(z0 + z, y0 + y + q, x0 + 4 * kg + r, n) * NET_C + col];
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const int base = z * B3HY + y + q;
                v4f d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 2; s >= 0; s--) {
                    const uint2 p0 = P[s][(base + o0) * 16 + col], p1 = P[s][(base + o1) * 16 + col],
                                p8 = P[s][(base + o8) * 16 + col];
                    d = mfma32(__builtin_bit_cast(v8bf, make_uint4(p8.x, p8.y, p8.x, p8.y)), w8, d);
                    d = mfma32(__builtin_bit_cast(v8bf, make_uint4(p0.x, p0.y, p1.x, p1.y)), w, d);
                }
#pragma unroll
                for (int r = 0; r < 4; r++)
                    g2[vox_index(z0 + z, y0 + y + q, x0 + 4 * kg + r, n) * NET_C + col] = d[r] * dsilu(zz[q][r]);
            }
            // dW3: k = voxel 8 (kg % 2) + j of row y + kg / 2
            const int yk = y + (kg >> 1), xk = 8 * (kg & 1) + (col >> 2);
            const uint2 *ap = reinterpret_cast<const uint2 *>(A) + ((z * B3Y + yk) * 16 + xk) * 4 + (col & 3);
            const v8bf av = join(read_tr(ap), read_tr(ap + 16));
#pragma unroll
            for (int t = 0; t < 3; t++) {
                const int at = (z * B3HY + yk + ot[t]) * 16 + xk;
#pragma unroll
                for (int s = 2; s >= 0; s--)
                    acc[t] = mfma32(av, join(read_tr(&P[s][at]), read_tr(&P[s][at + 4])), acc[t]);
            }
        }
        __syncthreads();
    }
    // D[ci = 4 kg + r][column]: tap row 4 t + col / 4, dx = col % 4
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) db += __shfl_xor(db, off);
    if (lane == 0) red[NET_C * 48 + wave] = (float)db;
    for (int v = 0; v < 4; v++) {
        if (wave == v)
#pragma unroll
            for (int t = 0; t < 3; t++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    float *p = red + (4 * kg + r) * 48 + t * 16 + col;
                    *p = v == 0 ? acc[t][r] : *p + acc[t][r];
                }
        __syncthreads();
    }
    float *out = part + (int64_t)blockIdx.x * DW3_N;
    for (int e = tid; e < NET_C * 27; e += 256) {
        const int ci = e / 27, t = 26 - e % 27, row = t / 3, dx = t % 3;   // phibar(v - o(t)): the mirrored tap
        out[e] = red[ci * 48 + row * 4 + dx];
    }
    if (tid == 0) out[NET_C * 27] = (red[NET_C * 48] + red[NET_C * 48 + 1]) + (red[NET_C * 48 + 2] + red[NET_C * 48 + 3]);
}

// ---------------------------------------------------------------- conv2 weights
// dW2[co][ci][t] = sum_v g2[v][co] a1[v + o(t)][ci].  Tile 16 x 8 x 8 with
// a1's halo in LDS (58 KB, two workgroups per CU); a wavefront takes 32 voxels
// (two rows) per MFMA chain, its g2 straight from HBM and split in registers,
// and keeps all 27 tap gradients in 108 accumulator registers: 81 MFMAs and 54
// transposed reads per 32 voxels.
constexpr int W2X = 18, W2Y = 10, W2Z = 10;
constexpr int DW2_N = NET_C * NET_C * 27 + NET_C;   // a workgroup's partial: [t][co][ci] then db2

__global__ __launch_bounds__(256, 2) void k_conv2_bwd_w(const uint16_t *__restrict__ a1,
                                                       const float *__restrict__ g2, int n, float *part)
{
    __shared__ __align__(16) uint4 X[W2X * W2Y * W2Z * 2];
    __shared__ float bred[4][NET_C];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, kg = lane >> 4, m = n - 1;
    const int ntx = n / 16, nty = n / 8, ntiles = ntx * nty * (n / 8);
    v4f acc[27] = {};
    double db = 0.0;
    for (int tile = xcd_tile(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const int x0 = (tile % ntx) * 16, y0 = ((tile / ntx) % nty) * 8, z0 = (tile / (ntx * nty)) * 8;
        {
            // all loads before the first LDS store, as above
            constexpr int NE = W2X * W2Y * W2Z * 2, NX = (NE + 255) / 256;
            uint4 v[NX];
#pragma unroll
            for (int k = 0; k < NX; k++) {
                const int e = min(tid + 256 * k, NE - 1);
                const int hv = e >> 1, hq = Div24<W2X, W2X * W2Y * W2Z>::div(hv), hz = Div24<W2Y, W2Y * W2Z>::div(hq);
                const int hx = hv - hq * W2X, hy = hq - hz * W2Y;
                v[k] = reinterpret_cast<const uint4 *>(
                    a1 + vox_index((z0 + hz - 1) & m, (y0 + hy - 1) & m, (x0 + hx - 1) & m, n) * NET_C)[e & 1];
            }
#pragma unroll
            for (int k = 0; k < NX; k++)
                if (tid + 256 * k < NE) X[tid + 256 * k] = v[k];
        }
        __syncthreads();
        for (int c = wave; c < 32; c += 4) {
            // k = voxel 8 (kg % 2) + j of row y + kg / 2
            const int z = c >> 2, y = 2 * (c & 3) + (kg >> 1), x = 8 * (kg & 1);
            const float *gp = g2 + vox_index(z0 + z, y0 + y, x0 + x, n) * NET_C + col;
            float g[8];
#pragma unroll
            for (int j = 0; j < 8; j++) g[j] = gp[j * NET_C];
            v8bf gs[3];
            split8(g, gs);
            db += ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7]));
            const uint2 *xp = reinterpret_cast<const uint2 *>(X) + ((z * W2Y + y) * W2X + x + (col >> 2)) * 4 + (col & 3);
#pragma unroll
            for (int t = 0; t < 27; t++) {
                const uint2 *p = xp + (((t / 9) * W2Y + (t / 3) % 3) * W2X + t % 3) * 4;
                const v8bf b = join(read_tr(p), read_tr(p + 16));
                acc[t] = mfma32(gs[2], b, acc[t]);
                acc[t] = mfma32(gs[1], b, acc[t]);
                acc[t] = mfma32(gs[0], b, acc[t]);
            }
        }
        __syncthreads();
    }
    // the four wavefronts' sums, in order, through the tile's LDS: [t][co][ci]
    float *red = reinterpret_cast<float *>(X);
    static_assert(sizeof(X) >= 27 * 256 * sizeof(float), "the reduction fits the tile");
    for (int v = 0; v < 4; v++) {
        if (wave == v)
#pragma unroll
            for (int t = 0; t < 27; t++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    float *p = red + t * 256 + (4 * kg + r) * 16 + col;
                    *p = v == 0 ? acc[t][r] : *p + acc[t][r];
                }
        __syncthreads();
    }
    db = sum_groups(db);
    if (kg == 0) bred[wave][col] = (float)db;
    __syncthreads();
    float *out = part + (int64_t)blockIdx.x * DW2_N;
    for (int e = tid; e < 27 * 256; e += 256) out[e] = red[e];
    if (tid < NET_C) out[27 * 256 + tid] = (bred[0][tid] + bred[1][tid]) + (bred[2][tid] + bred[3][tid]);
}

// ---------------------------------------------------------------- conv2 data, conv1 weights
// Tile 16 x D2R x 4, D2R wavefronts.  g2's halo lies in LDS as its three
// splits, eight channels per 16-byte row, so the 16 lanes of a K group read
// 256 contiguous bytes (104 KB, one workgroup per CU).  Wavefront w takes the
// rows y = w of all four planes: a halo fragment (two taps of a plane x 16
// channels) is read once and feeds the up to three output planes it reaches.
// g1 comes out with the channel as the column, which is the A operand of dW1:
// two planes' rows make K = 32 voxels against delta's taps as columns.
constexpr int D2R = 8, D2Z = 4, D2HZ = D2Z + 2, D2X = 18, D2Y = D2R + 2, D2HALO = D2X * D2Y * D2HZ, D2T = 64 * D2R;
constexpr int D2W_BYTES = 3 * 5 * NET_C * 4 * 8 * 2;
constexpr int DW1_N = NET_C * 27 + NET_C;   // a workgroup's partial: [co][27] then db1

// W2 as MFMA B operands: [dz][pair][ci][kg][j], tap 2 pair + kg / 2 of the
// plane's nine (the tenth zero), channel co = 8 (kg % 2) + j, taps mirrored.
__global__ __launch_bounds__(256) void k_pack_w2t(const float *__restrict__ th, uint16_t *wpk)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= D2W_BYTES / 2) return;
    const int j = e % 8, kg = (e / 8) % 4, ci = (e / 32) % NET_C, pr = (e / (32 * NET_C)) % 5, dz = e / (32 * NET_C * 5);
    const int q = 2 * pr + kg / 2, co = 8 * (kg % 2) + j;
    wpk[e] = q < 9 ? to_bf16(th[NC2W + (co * NET_C + ci) * 27 + 26 - (dz * 9 + q)]) : (uint16_t)0;
}

// SRC int64_t: the fixed-point density, delta = q qs - 1; float: delta itself.
template <typename SRC>
__global__ __launch_bounds__(D2T, 2) void k_conv2_bwd_d(const SRC *__restrict__ q, double qs,
                                                       const float *__restrict__ g2, int n,
                                                       const uint16_t *__restrict__ wpk,
                                                       const float *__restrict__ z1, float *part)
{
    __shared__ __align__(16) uint4 G[3][2][D2HALO];
    __shared__ __align__(16) uint16_t D3[3][D2HZ * D2Y * 16];   // delta(x + dx - 1) per dx
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, kg = lane >> 4, m = n - 1;
    const int ntx = n / 16, nty = n / D2R, ntiles = ntx * nty * (n / D2Z);
    v8bf w[3][5];
#pragma unroll
    for (int dz = 0; dz < 3; dz++)
#pragma unroll
        for (int p = 0; p < 5; p++)
            w[dz][p] = *reinterpret_cast<const v8bf *>(wpk + (((dz * 5 + p) * NET_C + col) * 4 + kg) * 8);
    int ox[5];
#pragma unroll
    for (int p = 0; p < 5; p++) {
        const int t = min(2 * p + (kg >> 1), 8);   // the tenth tap reads real data against zero weights
        ox[p] = (t / 3) * D2X + t % 3;
    }
    int od[2];   // dW1's columns: tap 16 c + col (columns past the 27th repeat it, unused)
#pragma unroll
    for (int c = 0; c < 2; c++) {
        const int t = min(16 * c + col, 26);
        od[c] = (t % 3) * (D2HZ * D2Y * 16) + ((t / 9) * D2Y + (t / 3) % 3) * 16;
    }
    v4f dw[2] = {};
    double db = 0.0;
    for (int tile = xcd_tile(blockIdx.x, gridDim.x); tile < ntiles; tile += gridDim.x) {
        const int x0 = (tile % ntx) * 16, y0 = ((tile / ntx) % nty) * D2R, z0 = (tile / (ntx * nty)) * D2Z;
        // every load before the first LDS store, as above (loading a tile
        // ahead, behind the products, gained nothing)
        constexpr int NG = (D2HALO * 4 + D2T - 1) / D2T, ND = (D2HALO + D2T - 1) / D2T;
        float4 gv[NG];
        SRC qv[ND];
#pragma unroll
        for (int k = 0; k < NG; k++) {
            const int e = min(tid + D2T * k, D2HALO * 4 - 1);
            const int hv = e >> 2, hq = Div24<D2X, D2HALO>::div(hv), hz = Div24<D2Y, D2Y * D2HZ>::div(hq);
            const int hx = hv - hq * D2X, hy = hq - hz * D2Y;
            gv[k] = reinterpret_cast<const float4 *>(
                g2 + vox_index((z0 + hz - 1) & m, (y0 + hy - 1) & m, (x0 + hx - 1) & m, n) * NET_C)[e & 3];
        }
#pragma unroll
        for (int k = 0; k < ND; k++) {
            const int e = min(tid + D2T * k, D2HALO - 1);
            const int hq = Div24<D2X, D2HALO>::div(e), hz = Div24<D2Y, D2Y * D2HZ>::div(hq);
            const int hx = e - hq * D2X, hy = hq - hz * D2Y;
            qv[k] = q[vox_index((z0 + hz - 1) & m, (y0 + hy - 1) & m, (x0 + hx - 1) & m, n)];
        }
#pragma unroll
        for (int k = 0; k < NG; k++) {
            const int e = tid + D2T * k, hv = e >> 2, c4 = e & 3;
            if (e < D2HALO * 4) {
                uint2 h, mm, l;
                split_pair(gv[k].x, gv[k].y, h.x, mm.x, l.x);
                split_pair(gv[k].z, gv[k].w, h.y, mm.y, l.y);
                reinterpret_cast<uint2 *>(&G[0][c4 >> 1][hv])[c4 & 1] = h;
                reinterpret_cast<uint2 *>(&G[1][c4 >> 1][hv])[c4 & 1] = mm;
                reinterpret_cast<uint2 *>(&G[2][c4 >> 1][hv])[c4 & 1] = l;
            }
        }
#pragma unroll
        for (int k = 0; k < ND; k++) {
            const int e = tid + D2T * k, hq = Div24<D2X, D2HALO>::div(min(e, D2HALO - 1)), hx = e - hq * D2X;
            if (e < D2HALO) {
                uint16_t d;
                if constexpr (std::is_same<SRC, int64_t>::value) d = delta_bf16(qv[k], qs);
                else d = to_bf16(qv[k]);
#pragma unroll
                for (int dx = 0; dx < 3; dx++)
                    if (hx - dx >= 0 && hx - dx < 16) D3[dx][hq * 16 + hx - dx] = d;
            }
        }
        float zz[D2Z][4];
#pragma unroll
        for (int z = 0; z < D2Z; z++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                zz[z][r] = z1[vox_index(z0 + z, y0 + wave, x0 + 4 * kg + r, n) * NET_C + col];
        __syncthreads();
        v4f acc[D2Z] = {};
#pragma unroll
        for (int hz = 0; hz < D2HZ; hz++)
#pragma unroll
            for (int p = 0; p < 5; p++) {
                const int hv = (hz * D2Y + wave) * D2X + col + ox[p];
#pragma unroll
                for (int s = 2; s >= 0; s--) {
                    const v8bf g = __builtin_bit_cast(v8bf, G[s][kg & 1][hv]);
#pragma unroll
                    for (int dz = 0; dz < 3; dz++)
                        if (hz - dz >= 0 && hz - dz < D2Z) acc[hz - dz] = mfma32(g, w[dz][p], acc[hz - dz]);
                }
            }
        // D[voxel 4 kg + r][ci = col]; dW1: k = 8 kg + j is voxel 4 kg + j % 4 of plane z + j / 4
#pragma unroll
        for (int z = 0; z < D2Z; z += 2) {
            float g[8];
#pragma unroll
            for (int j = 0; j < 8; j++) {
                g[j] = acc[z + (j >> 2)][j & 3] * dsilu(zz[z + (j >> 2)][j & 3]);
            }
            db += ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7]));
            v8bf gs[3];
            split8(g, gs);
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const uint16_t *dp = &D3[0][0] + od[c] + (z * D2Y + wave) * 16 + 4 * kg;
                const uint2 d0 = *reinterpret_cast<const uint2 *>(dp), d1 = *reinterpret_cast<const uint2 *>(dp + D2Y * 16);
                const v8bf dv = __builtin_bit_cast(v8bf, make_uint4(d0.x, d0.y, d1.x, d1.y));
#pragma unroll
                for (int s = 2; s >= 0; s--) dw[c] = mfma32(gs[s], dv, dw[c]);
            }
        }
        __syncthreads();
    }
    // [co][32 taps] per wavefront, then the workgroup's sum in order
    float *red = reinterpret_cast<float *>(G);
    constexpr int RS = NET_C * 32 + NET_C;
    db = sum_groups(db);
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int r = 0; r < 4; r++) red[wave * RS + (4 * kg + r) * 32 + 16 * c + col] = dw[c][r];
    if (kg == 0) red[wave * RS + NET_C * 32 + col] = (float)db;
    __syncthreads();
    float *out = part + (int64_t)blockIdx.x * DW1_N;
    for (int e = tid; e < DW1_N; e += D2T) {
        const int at = e < NET_C * 27 ? (e / 27) * 32 + e % 27 : NET_C * 32 + e - NET_C * 27;
        float s = 0.f;
#pragma unroll
        for (int v = 0; v < D2T / 64; v++) s += red[v * RS + at];
        out[e] = s;
    }
}

// dst[map(e)] += sum over np partials of part[i][e], e < ne: 16 values per
// workgroup, 16 strided sums each, added in order.  Weights come first, in
// the order of the parameter array, then the biases at dst + bias; conv2's
// weights (t_major) are stored [t][co][ci].
__global__ __launch_bounds__(256) void k_bwd_reduce(const float *__restrict__ part, int np, int ne, int nw,
                                                    int64_t bias, int t_major, float *dst)
{
    __shared__ double sh[16][17];
    const int c = threadIdx.x & 15, g = threadIdx.x >> 4, e = blockIdx.x * 16 + c;
    double s = 0.0;
    if (e < ne)
        for (int i = g; i < np; i += 16) s += (double)part[(int64_t)i * ne + e];
    sh[g][c] = s;
    __syncthreads();
    if (g == 0 && e < ne) {
        for (int i = 1; i < 16; i++) s += sh[i][c];
        const int64_t at = e >= nw ? bias + (e - nw) : (t_major ? (int64_t)(e % 256) * 27 + e / 256 : (int64_t)e);
        dst[at] += (float)s;
    }
}

}  // namespace

// Partials of one weight gradient fit the g1 buffer of n^3 x 16 floats: at
// most one workgroup per tile of 512 voxels (8192 floats of it, a partial has
// fewer), and enough to fill the chip.
static unsigned bwd_grid(int64_t tiles, unsigned most) { return (unsigned)(tiles < most ? tiles : most); }

hipError_t launch_cnn_bwd(const int64_t *q, double qs, const float *delta, const float *phibar, int64_t rs, int n,
                          const float *th, const float *z1, const uint16_t *a1, const float *z2, const uint16_t *a2, float *part,
                          float *g2, uint16_t *wpk, float *dth, hipStream_t s)
{
    static_assert(DW2_N <= 1024 * NET_C && DW3_N <= 1024 * NET_C && DW1_N <= 16 * D2R * D2Z * NET_C, "a tile's share of the buffer");
    static_assert(D2W_BYTES <= NET_WPK_BYTES, "packed weights");
    if (n < 16 || n % 16 || n > 4096) return hipErrorInvalidValue;
    const int64_t M = (int64_t)n * n * n;
    const unsigned g3 = bwd_grid(M / 1024, 512), gw = bwd_grid(M / 1024, 512), gd = bwd_grid(M / (16 * D2R * D2Z), 256);
    auto reduce = [&](unsigned np, int ne, int nw, int w, int b, int t_major) {
        hipLaunchKernelGGL(k_bwd_reduce, dim3((ne + 15) / 16), dim3(256), 0, s, part, (int)np, ne, nw, (int64_t)(b - w),
                           t_major, dth + w);
    };
    hipLaunchKernelGGL(k_conv3_bwd, dim3(g3), dim3(256), 0, s, phibar, rs, n, th, z2, a2, g2, part);
    reduce(g3, DW3_N, NET_C * 27, NC3W, NC3B, 0);
    hipLaunchKernelGGL(k_conv2_bwd_w, dim3(gw), dim3(256), 0, s, a1, g2, n, part);
    reduce(gw, DW2_N, NET_C * NET_C * 27, NC2W, NC2B, 1);
    hipLaunchKernelGGL(k_pack_w2t, dim3((D2W_BYTES / 2 + 255) / 256), dim3(256), 0, s, th, wpk);
    if (delta)
        hipLaunchKernelGGL(k_conv2_bwd_d<float>, dim3(gd), dim3(D2T), 0, s, delta, qs, g2, n, wpk, z1, part);
    else
        hipLaunchKernelGGL(k_conv2_bwd_d<int64_t>, dim3(gd), dim3(D2T), 0, s, q, qs, g2, n, wpk, z1, part);
    reduce(gd, DW1_N, NET_C * 27, NC1W, NC1B, 0);
    return hipGetLastError();
}

}  // namespace pm
