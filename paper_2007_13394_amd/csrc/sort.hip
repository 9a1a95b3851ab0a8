// Counting sort of particles by mesh tile, done at the start of every step
// so that the paint and the readout can work tile by tile out of LDS.
//
// Key of a particle = 8 * tile + face flags: tile is the Morton index of the
// TILE^3-cell block holding floor(u); bit d of the flags is set when floor(u_d) is the last
// cell of the tile along axis d (its +1 cloud-in-cell corner then lies in the
// next tile).  Counting: one atomic per distinct key per wavefront (lanes
// sharing a key are grouped by ballot) or, in the form for large sets, per chunk of
// 2048 particles (gathered in an LDS hash table), so lattice-ordered CDM, where
// most of a wavefront falls in one tile, costs few atomics.  Offsets come from an
// exclusive scan of the counts, which also leaves a copy of them as per-key
// cursors; the scatter recomputes each particle's key from its position,
// takes its slot from the cursor (one returning atomic per key and wavefront or
// chunk), and writes the position record (with the segment tag), the momentum and
// the optional id there.  The order of particles within a key depends on the
// order of the atomics.
#include "pm_internal.h"

namespace pm {
namespace {

inline unsigned grid_for(int64_t n, int block, int64_t cap = 65536LL * 16)
{
    int64_t b = (n + block - 1) / block;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (unsigned)b;
}


// Each workgroup takes a chunk of consecutive particles, workgroups numbered so
// that each XCD owns a contiguous run of chunks (the scatter of a nearly
// sorted state then writes whole cache lines from one L2).
//
// Two forms: one particle per thread, grouped by key within a wavefront, and
// chunks of WG_R per thread, grouped within the workgroup.  Chunks bring a
// key's atomics down and cost a chain of eight rounds (15 us at least), so they pay
// where atomics to one key queue up: with many particles per key, sooner in
// canonical order, where a key's particles lie scattered over the launch.
// Wavefront form / chunks, us, by particles and @ particles per key.
//   count and scatter, canonical order: chunks from 2^18 with 512 per key and from
//   2^20.  Evolved state (initial conditions): 69 k @134 36/32 (13/27); 267 k @521
//   64/44 (23/28); 298 k @582 85/49 (24/30), @73 37/37 (17/29); 549 k @1072 214/90
//   (37/36), @134 79/61 (23/31), @17 65/63; 803 k @196 108/83, @25 84/91; 2.4 M @582
//   158/125 (40/53), @73 141/114 (47/60); 19 M @582 970/684 (285/258), @73 1059/768
//   (339/298).
//   scatter of a step: chunks from 2^18 with 640 per key, from 2^20 with 128 and
//   from 2^26.  69 k @1072 17.1/15.0, @134 7.8/15.3; 298 k @582 14.2/15.8; 406 k @792
//   21.8/18.0; 549 k @1072 29.8/20.2, @134 15.0/18.8; 803 k @1568 44.3/22.8, @196
//   21.5/19.8; 2.4 M @582 58/29, @73 35/40, @9 32/44; 4.4 M @134 80/64, @17 58/72; 19 M
//   @582 410/244, @73 237/247, @9 242/278; 153 M @73 1530/1460.
constexpr int SORT_T = 256;

inline bool by_chunks(int64_t P, int n, bool sorted)
{
    const int64_t nt = n / TILE, keys = 8 * nt * nt * nt;
    if (P >= (sorted ? 1 << 26 : 1 << 20)) return true;
    const int64_t per_key = !sorted ? 512 : P < 1 << 20 ? 640 : 128;
    return P >= 1 << 18 && P >= per_key * keys;
}

__global__ __launch_bounds__(SORT_T) void k_sort_count(const float *__restrict__ x, int64_t P, int n, int *cnt)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * SORT_T + threadIdx.x;
    const bool live = i < P;
    const int k = live ? tile_key(x[i], x[P + i], x[2 * P + i], n) : -1;
    uint64_t group;
    int leader;
    key_group(live, k, group, leader);
    if (live && lane == leader) atomicAdd(cnt + k, __popcll(group));
}

// The same for large particle sets: a workgroup of WG_R x SORT_T particles first
// gathers its counts per key in an LDS hash table (open addressing, twice as
// many slots as particles, so that a probe always ends), then adds each key
// once.  Device-wide atomics do not combine across the eight L2s and set the pace of
// the sort: a chunk of lattice-ordered CDM has about 150 keys, its 32 wavefronts
// 600.  19 M particles on 512^3: count 381 -> 234 us,
// scatter of a sorted state 404 -> 248 us, of canonical order 604 -> 458 us
// (with indices).
constexpr int WG_R = 8, HASH = 2 * WG_R * SORT_T;

__device__ __forceinline__ int hash_slot(int *keys, int key)
{
    static_assert(HASH == 4096, "12 hash bits");
    unsigned h = ((unsigned)key * 2654435761u) >> 20;
    for (;;) {
        int old = __hip_atomic_load(keys + h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (old == -1) old = atomicCAS(keys + h, -1, key);
        if (old == -1 || old == key) return (int)h;
        h = (h + 1) & (HASH - 1);
    }
}

__device__ __forceinline__ void hash_clear(int *keys, int *cnt)
{
    for (int i = threadIdx.x; i < HASH; i += SORT_T) {
        keys[i] = -1;
        cnt[i] = 0;
    }
}

// One of a wavefront's runs of neighbouring lanes with one key: its first lane, and
// the lane behind its last.
struct KeyRun {
    int first, end;
};
__device__ __forceinline__ KeyRun key_run(int key)
{
    const int lane = threadIdx.x & 63, below = __shfl_up(key, 1);
    const uint64_t starts = __ballot(lane == 0 || below != key), upto = ~0ull >> (63 - lane);
    const uint64_t above = starts & ~upto;
    return KeyRun{63 - __clzll((long long)(starts & upto)), above ? __ffsll((unsigned long long)above) - 1 : 64};
}

__global__ __launch_bounds__(SORT_T) void k_sort_count_wg(const float *__restrict__ x, int64_t P, int n, int *cnt)
{
    __shared__ int hkey[HASH], hcnt[HASH];
    const int64_t c0 = (int64_t)blockIdx.x * (WG_R * SORT_T);
    float a0[WG_R], a1[WG_R], a2[WG_R];
#pragma unroll
    for (int r = 0; r < WG_R; r++) {
        const int64_t i = c0 + threadIdx.x + r * SORT_T, ic = i < P ? i : P - 1;
        a0[r] = x[ic];
        a1[r] = x[P + ic];
        a2[r] = x[2 * P + ic];
    }
    hash_clear(hkey, hcnt);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < WG_R; r++) {
        const bool live = c0 + threadIdx.x + r * SORT_T < P;
        const int key = live ? tile_key(a0[r], a1[r], a2[r], n) : -1;
        const KeyRun run = key_run(key);
        if (live && (int)(threadIdx.x & 63) == run.first) atomicAdd(hcnt + hash_slot(hkey, key), run.end - run.first);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < HASH; i += SORT_T)
        if (hcnt[i] > 0) atomicAdd(cnt + hkey[i], hcnt[i]);
}

// Exclusive scan of up to SCAN_ONE counts by one workgroup, all loads in
// flight at once: out[i] = sum of in[0 .. i), out[n - 1] the total (in[n - 1],
// past the last key, is not read; n - 1 is a multiple of four).  A thread takes
// four consecutive values of each of R rows; the rows' and wavefronts' totals
// are scanned by the first wavefront.  clear: zero the counts behind the scan
// (the next readout adds to them), else out2 may be the counts' own array.  At
// 32 768 keys (256^3) 8.6 us against 10.3 us and two launches more for the blocked
// form below.
constexpr int SCAN_ONE = 32768, ONE_T = 1024;

__device__ __forceinline__ int wave_inclusive(int v, int lane)
{
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int t = __shfl_up(v, off);
        if (lane >= off) v += t;
    }
    return v;
}

template <int R>
__global__ __launch_bounds__(ONE_T) void k_scan_one(int *in, int *out, int n, int *out2, int clear)
{
    constexpr int NW = ONE_T / 64;
    __shared__ int tot[R * NW + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = n - 1;
    int4 v[R];
    int incl[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = 4 * (r * ONE_T + tid);
        v[r] = i < m ? *reinterpret_cast<const int4 *>(in + i) : make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        incl[r] = wave_inclusive(v[r].x + v[r].y + v[r].z + v[r].w, lane);
        if (lane == 63) tot[r * NW + wave] = incl[r];
    }
    __syncthreads();
    if (wave == 0) {
        static_assert(R * NW <= 128, "two totals per lane");
        const int a = 2 * lane < R * NW ? tot[2 * lane] : 0, b = 2 * lane + 1 < R * NW ? tot[2 * lane + 1] : 0;
        const int e = wave_inclusive(a + b, lane) - a - b;
        if (2 * lane < R * NW) tot[2 * lane] = e;
        if (2 * lane + 1 < R * NW) tot[2 * lane + 1] = e + a;
        if (lane == 63) tot[R * NW] = e + a + b;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int i = 4 * (r * ONE_T + tid);
        if (i < m) {
            const int e = tot[r * NW + wave] + incl[r] - (v[r].x + v[r].y + v[r].z + v[r].w);
            const int4 o = make_int4(e, e + v[r].x, e + v[r].x + v[r].y, e + v[r].x + v[r].y + v[r].z);
            *reinterpret_cast<int4 *>(out + i) = o;
            if (clear) *reinterpret_cast<int4 *>(in + i) = make_int4(0, 0, 0, 0);
            if (out2) *reinterpret_cast<int4 *>(out2 + i) = o;
        }
    }
    if (tid == 0) {
        out[m] = tot[R * NW];
        if (clear) in[m] = 0;
        if (out2) out2[m] = tot[R * NW];
    }
}

// Exclusive scan in blocks of SCAN_B = 2048 values (256 threads x 8).
constexpr int SCAN_T = 256, SCAN_PER = 8, SCAN_B = SCAN_T * SCAN_PER;

__device__ __forceinline__ int block_exclusive_scan(int v, int *sh)
{
    // sh: SCAN_T ints; returns the exclusive prefix of v over the block, total in sh[SCAN_T - 1] + last v
    const int tid = threadIdx.x;
    sh[tid] = v;
    __syncthreads();
    for (int off = 1; off < SCAN_T; off <<= 1) {
        const int t = tid >= off ? sh[tid - off] : 0;
        __syncthreads();
        sh[tid] += t;
        __syncthreads();
    }
    const int incl = sh[tid];
    __syncthreads();
    return incl - v;
}

__global__ __launch_bounds__(SCAN_T) void k_scan_blocks(int *in, int *out, int64_t n, int *block_sums, int clear)
{
    __shared__ int sh[SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * SCAN_B + (int64_t)threadIdx.x * SCAN_PER;
    int v[SCAN_PER], s = 0;
#pragma unroll
    for (int j = 0; j < SCAN_PER; j++) {
        v[j] = base + j < n ? in[base + j] : 0;
        s += v[j];
    }
    const int pre = block_exclusive_scan(s, sh);
    int run = pre;
#pragma unroll
    for (int j = 0; j < SCAN_PER; j++) {
        if (base + j < n) {
            out[base + j] = run;
            if (clear) in[base + j] = 0;
        }
        run += v[j];
    }
    if (threadIdx.x == SCAN_T - 1) block_sums[blockIdx.x] = run;
}

// Single block: exclusive scan of up to SCAN_B * 4 block sums, in place.
__global__ __launch_bounds__(SCAN_T) void k_scan_sums(int *sums, int nb)
{
    __shared__ int sh[SCAN_T];
    int carry = 0;
    for (int start = 0; start < nb; start += SCAN_B) {
        const int base = start + threadIdx.x * SCAN_PER;
        int v[SCAN_PER], s = 0;
#pragma unroll
        for (int j = 0; j < SCAN_PER; j++) {
            v[j] = base + j < nb ? sums[base + j] : 0;
            s += v[j];
        }
        const int pre = block_exclusive_scan(s, sh);
        int run = carry + pre;
#pragma unroll
        for (int j = 0; j < SCAN_PER; j++) {
            if (base + j < nb) sums[base + j] = run;
            run += v[j];
        }
        // total of this chunk = inclusive value of the last thread
        if (threadIdx.x == SCAN_T - 1) sh[0] = run;
        __syncthreads();
        carry = sh[0];
        __syncthreads();
    }
}

// out2 (optional): a second copy of the result.
__global__ void k_scan_add(int *out, int64_t n, const int *sums, int *out2)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int v = out[i] + sums[i / SCAN_B];
        out[i] = v;
        if (out2) out2[i] = v;
    }
}

// Scatter into float4 records: one 16-byte store for the position and the
// segment tag, one for the momentum, so a particle that moves far in the
// order costs two stores instead of seven partial ones.  The optional arrays
// are template flags (HI 1: the caller's ids, 2: the particle's index).  The
// pointers do not alias (caller arrays in, workspace records out).
template <bool HP, bool HT, int HI>
__global__ __launch_bounds__(SORT_T) void k_sort_scatter(const float *__restrict__ x, const float *__restrict__ p,
                                                         const uint8_t *__restrict__ tag_in, int64_t P, int nseg,
                                                         const int64_t *__restrict__ seg_off, int n, int *cursor,
                                                         float4 *__restrict__ xs, Mom3 *__restrict__ ps,
                                                         const uint32_t *__restrict__ ids_in,
                                                         uint32_t *__restrict__ ids_out)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * SORT_T + threadIdx.x, ic = i < P ? i : P - 1;
    const bool live = i < P;
    const float a0 = x[ic], a1 = x[P + ic], a2 = x[2 * P + ic];
    Mom3 b{0.f, 0.f, 0.f};
    if constexpr (HP) b = Mom3{p[ic], p[P + ic], p[2 * P + ic]};
    int t = 0;
    if constexpr (HT) {
        t = tag_in[ic];
    } else {   // canonical order: segment from the offsets
        for (int g = 1; g < nseg; g++) t += (ic >= seg_off[g]) ? 1 : 0;
    }
    uint32_t id = 0;
    if constexpr (HI == 1) id = ids_in[ic];
    if constexpr (HI == 2) id = (uint32_t)ic;
    const int k = live ? tile_key(a0, a1, a2, n) : -1;
    uint64_t group;
    int leader, base = 0;
    key_group(live, k, group, leader);
    if (live && lane == leader) base = atomicAdd(cursor + k, __popcll(group));
    const int64_t d = (int64_t)__shfl(base, leader) + __popcll(group & ((1ull << lane) - 1));
    if (live && d < P) {   // d >= P only with counts that do not match x (k_sort_verify reports it)
        xs[d] = make_float4(a0, a1, a2, __int_as_float(t));
        if constexpr (HP) ps[d] = b;
        if constexpr (HI) ids_out[d] = id;
    }
}

constexpr int CHUNK_RUN = 32;
__device__ __forceinline__ int run_tile(int b, int nb)
{
    // full rounds of 8 x CHUNK_RUN chunks, the rest in plain order
    const int round = 8 * CHUNK_RUN, full = nb / round * round;
    if (b >= full) return b;
    const int x = b % 8, i = b / 8;
    return (i / CHUNK_RUN) * round + x * CHUNK_RUN + i % CHUNK_RUN;
}

// The scatter with a chunk's slots taken key by key (see k_sort_count_wg): all of
// a thread's particles are loaded at once and ranked within the chunk, each
// key's cursor is advanced once, then the records are stored.
template <bool HP, bool HT, int HI>
__device__ __forceinline__ void scatter_wg(int *hkey, int *hcnt, int64_t c0, const float *__restrict__ x,
                                           const float *__restrict__ p, const uint8_t *__restrict__ tag_in, int64_t P,
                                           int nseg, const int64_t *__restrict__ seg_off, int n, int *cursor,
                                           float4 *__restrict__ xs, Mom3 *__restrict__ ps,
                                           const uint32_t *__restrict__ ids_in, uint32_t *__restrict__ ids_out)
{
    float a0[WG_R], a1[WG_R], a2[WG_R], b0[WG_R], b1[WG_R], b2[WG_R];
    int t[WG_R];
    uint32_t id[WG_R];
#pragma unroll
    for (int r = 0; r < WG_R; r++) {
        const int64_t i = c0 + threadIdx.x + r * SORT_T, ic = i < P ? i : P - 1;
        a0[r] = x[ic];
        a1[r] = x[P + ic];
        a2[r] = x[2 * P + ic];
        if constexpr (HT) t[r] = tag_in[ic];
        if constexpr (HI == 1) id[r] = ids_in[ic];
    }
    hash_clear(hkey, hcnt);
    __syncthreads();
    int at[WG_R];   // slot and rank within the chunk's particles of the key
#pragma unroll
    for (int r = 0; r < WG_R; r++) {
        const bool live = c0 + threadIdx.x + r * SORT_T < P;
        const int key = live ? tile_key(a0[r], a1[r], a2[r], n) : -1, lane = threadIdx.x & 63;
        const KeyRun run = key_run(key);
        int slot = 0;
        if (live && lane == run.first) {
            const int h = hash_slot(hkey, key);
            slot = (h << 16) | atomicAdd(hcnt + h, run.end - run.first);
        }
        at[r] = __shfl(slot, run.first) + lane - run.first;
    }
    if constexpr (HP) {
#pragma unroll
        for (int r = 0; r < WG_R; r++) {
            const int64_t i = c0 + threadIdx.x + r * SORT_T, ic = i < P ? i : P - 1;
            b0[r] = p[ic];
            b1[r] = p[P + ic];
            b2[r] = p[2 * P + ic];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < HASH; i += SORT_T)
        if (hcnt[i] > 0) hcnt[i] = atomicAdd(cursor + hkey[i], hcnt[i]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < WG_R; r++) {
        const int64_t i = c0 + threadIdx.x + r * SORT_T;
        const int64_t d = (int64_t)hcnt[at[r] >> 16] + (at[r] & 0xffff);
        if (i < P && d < P) {   // d >= P only with counts that do not match x (k_sort_verify reports it)
            int g = 0;
            if constexpr (HT) {
                g = t[r];
            } else {   // canonical order: segment from the offsets
                for (int k = 1; k < nseg; k++) g += (i >= seg_off[k]) ? 1 : 0;
            }
            xs[d] = make_float4(a0[r], a1[r], a2[r], __int_as_float(g));
            if constexpr (HP) ps[d] = Mom3{b0[r], b1[r], b2[r]};
            if constexpr (HI == 1) ids_out[d] = id[r];
            if constexpr (HI == 2) ids_out[d] = (uint32_t)i;
        }
    }
}

template <bool HP, bool HT, int HI>
__global__ __launch_bounds__(SORT_T) void k_sort_scatter_wg(const float *__restrict__ x, const float *__restrict__ p,
                                                            const uint8_t *__restrict__ tag_in, int64_t P, int nseg,
                                                            const int64_t *__restrict__ seg_off, int n, int *cursor,
                                                            float4 *xs, Mom3 *ps, const uint32_t *ids_in,
                                                            uint32_t *ids_out)
{
    __shared__ int hkey[HASH], hcnt[HASH];
    // Sorted input (tags): contiguous runs of chunks per XCD, whose stores meet in
    // one L2.  Canonical order: runs of CHUNK_RUN chunks dealt to the XCDs in
    // turn, else the last of them gets all the neutrinos, the slowest chunks.
    const int b = HT ? xcd_tile(blockIdx.x, gridDim.x) : run_tile(blockIdx.x, gridDim.x);
    const int64_t c0 = (int64_t)b * (WG_R * SORT_T);
    scatter_wg<HP, HT, HI>(hkey, hcnt, c0, x, p, tag_in, P, nseg, seg_off, n, cursor, xs, ps, ids_in, ids_out);
}

// After a scatter from counts computed elsewhere (the previous readout):
// every key's cursor must have reached the next key's offset, else the
// counts did not describe x and FLAG_STALE is raised, for the kernels queued
// behind and for the host.
__global__ __launch_bounds__(256) void k_sort_verify(const int *__restrict__ cursor, const int *__restrict__ koff,
                                                     int64_t K, int *stale, int *host_stale)
{
    bool bad = false;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += (int64_t)gridDim.x * blockDim.x)
        bad |= cursor[k] != koff[k + 1];
    if (__any(bad) && (threadIdx.x & 63) == 0) {
        raise(stale);
        raise(host_stale);
    }
}

}  // namespace

hipError_t launch_sort_verify(const int *cursor, const int *koff, int64_t K, int *stale, int *host_stale, hipStream_t s)
{
    hipLaunchKernelGGL(k_sort_verify, dim3(grid_for(K, 256, 65536)), dim3(256), 0, s, cursor, koff, K, stale, host_stale);
    return hipGetLastError();
}

hipError_t launch_sort_count(const float *x, int64_t P, int n, bool sorted, int *cnt, hipStream_t s)
{
    const bool chunks = by_chunks(P, n, sorted);
    const int64_t ch = chunks ? WG_R * SORT_T : SORT_T, nb = (P + ch - 1) / ch;
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(nb > 0 ? nb : 1));
    if (chunks)
        hipLaunchKernelGGL(k_sort_count_wg, grid, dim3(SORT_T), 0, s, x, P, n, cnt);
    else
        hipLaunchKernelGGL(k_sort_count, grid, dim3(SORT_T), 0, s, x, P, n, cnt);
    return hipGetLastError();
}

hipError_t launch_scan(int *in, int *out, int64_t n, int *block_sums, hipStream_t s, int *out2, bool clear)
{
    if (clear && (out2 == in || out == in)) return hipErrorInvalidValue;
    if (n - 1 <= SCAN_ONE && (n - 1) % 4 == 0 &&
        ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(out2)) & 15) == 0) {
        if (n - 1 <= 4 * ONE_T)
            hipLaunchKernelGGL(k_scan_one<1>, dim3(1), dim3(ONE_T), 0, s, in, out, (int)n, out2, clear ? 1 : 0);
        else
            hipLaunchKernelGGL(k_scan_one<8>, dim3(1), dim3(ONE_T), 0, s, in, out, (int)n, out2, clear ? 1 : 0);
        return hipGetLastError();
    }
    const int64_t nb = (n + SCAN_B - 1) / SCAN_B;
    if (nb > (int64_t)SCAN_B * 4096) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)nb), dim3(SCAN_T), 0, s, in, out, n, block_sums, clear ? 1 : 0);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(SCAN_T), 0, s, block_sums, (int)nb);
    hipLaunchKernelGGL(k_scan_add, dim3(grid_for(n, 256)), dim3(256), 0, s, out, n, block_sums, out2);
    return hipGetLastError();
}

hipError_t launch_sort_scatter(const float *x, const float *p, const uint8_t *tag_in, int64_t P, int nseg,
                               const int64_t *seg_off, int n, int *cursor, float4 *xs, Mom3 *ps,
                               const uint32_t *ids_in, uint32_t *ids_out, hipStream_t s)
{
    const bool chunks = by_chunks(P, n, tag_in != nullptr);
    const int64_t ch = chunks ? WG_R * SORT_T : SORT_T, nb = (P + ch - 1) / ch;
    if (nb > 0x7fffffff || (ids_in && !ids_out)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(nb > 0 ? nb : 1));
    const int hi = ids_in ? 1 : (ids_out ? 2 : 0);
#define SCATTER_K(HP, HT, HI)                                                                         \
    {                                                                                                \
        if (chunks)                                                                                  \
            hipLaunchKernelGGL((k_sort_scatter_wg<HP, HT, HI>), grid, dim3(SORT_T), 0, s, x, p, tag_in, P, nseg, seg_off, \
                               n, cursor, xs, ps, ids_in, ids_out);                                  \
        else                                                                                         \
            hipLaunchKernelGGL((k_sort_scatter<HP, HT, HI>), grid, dim3(SORT_T), 0, s, x, p, tag_in, P, nseg, seg_off, \
                               n, cursor, xs, ps, ids_in, ids_out);                                  \
    }
#define SCATTER_I(HP, HT)                                                                             \
    {                                                                                                \
        if (hi == 0) SCATTER_K(HP, HT, 0)                                                            \
        else if (hi == 1) SCATTER_K(HP, HT, 1)                                                       \
        else SCATTER_K(HP, HT, 2)                                                                    \
    }
    if (p) {
        if (tag_in) SCATTER_I(true, true)
        else SCATTER_I(true, false)
    } else {
        if (tag_in) SCATTER_I(false, true)
        else SCATTER_I(false, false)
    }
#undef SCATTER_I
#undef SCATTER_K
    return hipGetLastError();
}

}  // namespace pm
