// Tree construction on the GPU (Section 3.1: an octree-like tree over the
// sources with per-node aggregate weight and centre of mass; the summed
// dipole w*n is added for the winding kernel).
//
// Pipeline, every step a kernel on the caller's stream:
//   1. root cube: per-axis min/max, side = largest extent, inv_side =
//      fl32(1/side) (correctly rounded), plus an input validity flag;
//   2. Morton code: cell_a = min(2^20-1, (u32) fl32(fl32(x_a - lo_a) *
//      inv_side) * 2^20), bits of x/y/z interleaved into 60 bits;
//   3. stable LSD radix sort of (code, index), 10-bit digits, over the codes'
//      top bits with the few equal ones put in order after; up to 8192 points
//      in one workgroup;
//   4. topology in two passes over the sorted codes.  A node at level l is a
//      maximal run of equal (bits*l)-bit prefix; it is split iff count >
//      leaf_size and l < max.  Which levels have a node that starts at point
//      i, and which of those are internal, follows from the codes within
//      leaf_size points of i alone, so the first pass counts nodes and
//      internal nodes per level and block of points, the host reads the level
//      totals once, and the second pass writes every node, in breadth-first
//      order (Morton order within a level), with the leaves' aggregates;
//   5. the internal nodes' aggregates bottom-up, written with every node's
//      slot in its parent's child block.
// The build synchronises once for the sizes and once at its end.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "sbh_internal.hpp"

namespace sbh {

// ---------------------------------------------------------------------------
// 1. Root cube and validation
// ---------------------------------------------------------------------------
struct float3v {
    float x, y, z;
};
// a point's three floats in one 12-byte load
__device__ __forceinline__ float3v load3(const float* __restrict__ p, int64_t i)
{
    float3v v;
    __builtin_memcpy(&v, p + 3 * i, sizeof(v));
    return v;
}

constexpr int kBboxThreads = 256;

__global__ void __launch_bounds__(kBboxThreads) k_bbox_partial(const float* __restrict__ src,
                                                               const float* __restrict__ w,
                                                               const float* __restrict__ nrm, int64_t n,
                                                               float* __restrict__ partial)
{
    float mn0 = INFINITY, mn1 = INFINITY, mn2 = INFINITY;
    float mx0 = -INFINITY, mx1 = -INFINITY, mx2 = -INFINITY;
    int bad = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float3v p = load3(src, i);
        const float x = p.x, y = p.y, z = p.z;
        const float wi = w[i];
        bad |= !(__builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z));
        bad |= !(wi > 0.0f && __builtin_isfinite(wi));
        if (nrm) {
            const float3v m = load3(nrm, i);
            bad |= !(__builtin_isfinite(m.x) && __builtin_isfinite(m.y) && __builtin_isfinite(m.z));
        }
        mn0 = fminf(mn0, x); mn1 = fminf(mn1, y); mn2 = fminf(mn2, z);
        mx0 = fmaxf(mx0, x); mx1 = fmaxf(mx1, y); mx2 = fmaxf(mx2, z);
    }
    for (int o = 32; o > 0; o >>= 1) {
        mn0 = fminf(mn0, __shfl_xor(mn0, o)); mn1 = fminf(mn1, __shfl_xor(mn1, o)); mn2 = fminf(mn2, __shfl_xor(mn2, o));
        mx0 = fmaxf(mx0, __shfl_xor(mx0, o)); mx1 = fmaxf(mx1, __shfl_xor(mx1, o)); mx2 = fmaxf(mx2, __shfl_xor(mx2, o));
        bad |= __shfl_xor(bad, o);
    }
    __shared__ float sh[kBboxThreads / 64][7];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        sh[wv][0] = mn0; sh[wv][1] = mn1; sh[wv][2] = mn2;
        sh[wv][3] = mx0; sh[wv][4] = mx1; sh[wv][5] = mx2; sh[wv][6] = (float)bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kBboxThreads / 64; ++k) {
            for (int a = 0; a < 3; ++a) {
                sh[0][a] = fminf(sh[0][a], sh[k][a]);
                sh[0][3 + a] = fmaxf(sh[0][3 + a], sh[k][3 + a]);
            }
            sh[0][6] = fmaxf(sh[0][6], sh[k][6]);
        }
        for (int a = 0; a < 7; ++a) partial[blockIdx.x * 8 + a] = sh[0][a];
    }
}

// params: lo[3], side, inv_side, bad, and a cleared word.  One workgroup: each thread folds a
// stride of the partials, then the wavefronts and the workgroup combine
// (min and max are exact, so the order does not change the result).
__global__ void __launch_bounds__(kBboxThreads) k_bbox_final(const float* __restrict__ partial, int nb,
                                                             float* __restrict__ params)
{
    float mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    float bad = 0.0f;
    for (int b = threadIdx.x; b < nb; b += kBboxThreads) {
        for (int a = 0; a < 3; ++a) {
            mn[a] = fminf(mn[a], partial[b * 8 + a]);
            mx[a] = fmaxf(mx[a], partial[b * 8 + 3 + a]);
        }
        bad = fmaxf(bad, partial[b * 8 + 6]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        for (int a = 0; a < 3; ++a) {
            mn[a] = fminf(mn[a], __shfl_xor(mn[a], o));
            mx[a] = fmaxf(mx[a], __shfl_xor(mx[a], o));
        }
        bad = fmaxf(bad, __shfl_xor(bad, o));
    }
    __shared__ float sh[kBboxThreads / 64][7];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        for (int a = 0; a < 3; ++a) {
            sh[wv][a] = mn[a];
            sh[wv][3 + a] = mx[a];
        }
        sh[wv][6] = bad;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < kBboxThreads / 64; ++k) {
        for (int a = 0; a < 3; ++a) {
            mn[a] = fminf(mn[a], sh[k][a]);
            mx[a] = fmaxf(mx[a], sh[k][3 + a]);
        }
        bad = fmaxf(bad, sh[k][6]);
    }
    float side = 0.0f;
    for (int a = 0; a < 3; ++a) {
        const float e = __fsub_rn(mx[a], mn[a]);
        side = e > side ? e : side;
    }
    if (side == 0.0f) side = 1.0f;
    params[0] = mn[0]; params[1] = mn[1]; params[2] = mn[2];
    params[3] = side;
    params[4] = __fdiv_rn(1.0f, side);
    params[5] = bad;
    params[6] = 0.0f;   // set by k_rs_finish
}

static hipError_t launch_bbox(const float* src, const float* w, const float* nrm, int64_t n, float* params_dev,
                       float* partial_dev, int nblocks, hipStream_t s)
{
    k_bbox_partial<<<nblocks, kBboxThreads, 0, s>>>(src, w, nrm, n, partial_dev);
    k_bbox_final<<<1, kBboxThreads, 0, s>>>(partial_dev, nblocks, params_dev);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 2. Morton codes
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t spread_bits3(uint32_t v)
{
    // bit k of v (k < 21) moves to bit 3k
    uint64_t x = v & 0x1FFFFFu;
    x = (x | (x << 32)) & 0x001F00000000FFFFull;
    x = (x | (x << 16)) & 0x001F0000FF0000FFull;
    x = (x | (x << 8)) & 0x100F00F00F00F00Full;
    x = (x | (x << 4)) & 0x10C30C30C30C30C3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

__device__ __forceinline__ uint32_t quantize(float x, float lo, float inv_side)
{
    float u = __fsub_rn(x, lo);
    u = __fmul_rn(u, inv_side);
    u = __fmul_rn(u, 1048576.0f);
    uint32_t c = (uint32_t)u;  // truncation; u >= 0
    return c > 1048575u ? 1048575u : c;
}

__device__ __forceinline__ uint64_t morton_code(float3v x, const float* __restrict__ params)
{
    const float inv = params[4];
    return spread_bits3(quantize(x.x, params[0], inv)) | (spread_bits3(quantize(x.y, params[1], inv)) << 1) |
           (spread_bits3(quantize(x.z, params[2], inv)) << 2);
}

__device__ __forceinline__ float4 point_dipole(float3v m, float w) { return make_float4(w * m.x, w * m.y, w * m.z, 0.0f); }

// Codes, and each point as one record of 16 bytes (x, y, z, w), or 32 with its
// dipole: the sort's permutation then reads one record per point instead of
// one line from each of the input arrays (2^22 points with normals: the gather
// 263 -> 99 us, this kernel 50).
__global__ void k_morton(const float* __restrict__ src, const float* __restrict__ w, const float* __restrict__ nrm,
                         int64_t n, const float* __restrict__ params, uint64_t* __restrict__ keys,
                         float4* __restrict__ rec)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float3v x = load3(src, i);
    const float wi = w[i];
    keys[i] = morton_code(x, params);
    const float4 p = make_float4(x.x, x.y, x.z, wi);
    if (nrm) {
        rec[2 * i] = p;
        rec[2 * i + 1] = point_dipole(load3(nrm, i), wi);
    } else {
        rec[i] = p;
    }
}

// the sorted points from their records
__global__ void k_gather_points(const float4* __restrict__ rec, const uint32_t* __restrict__ perm, int64_t n,
                                float4* __restrict__ pts, float4* __restrict__ pdip)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const int64_t i = perm[s];
    if (pdip) {
        const float4 p = rec[2 * i], d = rec[2 * i + 1];
        pts[s] = p;
        pdip[s] = d;
    } else {
        pts[s] = rec[i];
    }
}

// ---------------------------------------------------------------------------
// 3. Stable LSD radix sort of (uint64 code, uint32 index) in 10-bit digits.
// The passes run over the codes' top bits alone (four of the six digits, three
// in k_sort_small): few codes share these, and a pass over the result puts
// such short runs in order.  Where a longer run is out of order, as in a cloud
// of clusters far smaller than its cube, the six passes over all bits follow
// (a build of 2^22 points 0.97 ms, of as many in clumps a 2^-15th of the cube
// wide 1.35).  A workgroup owns a tile of 8192 consecutive keys, its wavefront v the v-th sixteenth, which it walks in
// eight chunks of 64 in order: a key's rank among the tile's equal digits is
// (wavefronts before) + (chunks of this wavefront before) + (lanes of the
// chunk before), the last from one ballot per digit bit.  A pass is three
// kernels: the tiles' histograms; their prefix sums over a chunk of tiles,
// with the chunk's totals; and the scatter, which adds up the chunks before
// its own, sorts the tile in LDS and writes each digit's keys as one run.
// Memory traffic and the scatter's latency bound it: 47 us a pass for 2^22
// keys (the scatter 34, 2.9 TB/s; 45 with one workgroup a CU).  Eight passes of
// 8-bit digits whose scatter wrote every key on its own took 657 us, six passes
// 345, four and the runs 205; k_sort_small with 5,003 points 61 over all bits,
// 37 now.
// ---------------------------------------------------------------------------
constexpr int kRsBits = 10;
constexpr int kRsBins = 1 << kRsBits;
constexpr int kRsPasses = 6;
constexpr int kRsThreads = 1024;
constexpr int kRsWaves = kRsThreads / 64;
constexpr int kRsItems = 8;
constexpr int kRsTile = kRsThreads * kRsItems;
constexpr int kRsTopPasses = 4;        // 40 bits: 13 levels of the octree
constexpr int kRsTopPassesSmall = 3;   // of at most kRsTile codes
constexpr int kRsRun = 16;             // longest run of equal top bits that is put in order by one thread
// Points of a surface fill some 4^13 cells of the top bits, so that runs stay
// short up to this many: 2^26 points 10.1 ms of kernels a build against 11.2 over
// all bits (2^26 in a volume 8.7 against 10.3).  Beyond, a surface gains less (2^27
// 20.9 against 22.5, 2^28 43.3 against 43.6), and a run that is too long costs the
// passes over the top bits on top of all six.
constexpr int64_t kRsTopMax = (int64_t)1 << 26;
constexpr int kRsMaxChunks = 64;   // chunks of tiles (every scatter workgroup reads a row of each)
static_assert(kRsPasses * kRsBits >= 60 && kRsPasses % 2 == 0 && kRsTopPasses % 2 == 0 && kRsBins == kRsThreads, "radix sort layout");

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, int lane)
{
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// exclusive scan over the workgroup's 1024 threads; ws: one word per wavefront (reused by the next call)
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* ws)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t incl = wave_inclusive_scan(v, lane);
    if (lane == 63) ws[wv] = incl;
    __syncthreads();
    uint32_t run = incl - v;
    for (int k = 0; k < wv; ++k) run += ws[k];
    __syncthreads();
    return run;
}

__device__ __forceinline__ uint32_t rs_digit(uint64_t key, int shift) { return (uint32_t)(key >> shift) & (kRsBins - 1); }

// Ranks of the tile's keys within their wavefront's equal digits, and, once all
// have them, the tile-local position of the first key of each (wavefront,
// digit): start[digit] + wcnt[wavefront][digit].  cnt: keys of the tile.
struct RsLds {
    uint16_t wcnt[kRsWaves][kRsBins];
    uint32_t start[kRsBins];
    uint32_t ws[kRsWaves];
};
__device__ __forceinline__ void rs_rank(RsLds& S, const uint64_t (&kk)[kRsItems], uint32_t (&rank)[kRsItems], int cnt,
                                        int shift)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int w = 0; w < kRsWaves; ++w) S.wcnt[w][threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {
        const bool valid = wv * (64 * kRsItems) + c * 64 + lane < cnt;
        const uint32_t d = rs_digit(kk[c], shift);
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRsBits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        const uint32_t base = S.wcnt[wv][d];
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) S.wcnt[wv][d] = (uint16_t)(base + (uint32_t)__popcll(m));
        __builtin_amdgcn_wave_barrier();
        rank[c] = base + below;
    }
    __syncthreads();
    uint32_t run = 0u;   // this thread's digit: the wavefronts' counts become what is before each
    for (int w = 0; w < kRsWaves; ++w) {
        const uint32_t t = S.wcnt[w][threadIdx.x];
        S.wcnt[w][threadIdx.x] = (uint16_t)run;
        run += t;
    }
    S.start[threadIdx.x] = block_exclusive_scan(run, S.ws);
    __syncthreads();
}

// tile of a workgroup: consecutive tiles on one die, whose L2 then joins their neighbouring runs
__device__ __forceinline__ int rs_tile(int b, int tiles)
{
    const int per = (tiles + 7) >> 3;
    return (b & 7) * per + (b >> 3);
}

__global__ void __launch_bounds__(kRsThreads) k_rs_hist(const uint64_t* __restrict__ keys, int64_t n, int shift,
                                                        uint32_t* __restrict__ hist, int tiles)
{
    __shared__ uint32_t h[kRsBins];
    const int tile = rs_tile(blockIdx.x, tiles);
    if (tile >= tiles) return;
    h[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t base = (int64_t)tile * kRsTile + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kRsItems; ++k) {
        const int64_t i = base + k * kRsThreads;
        if (i < n) atomicAdd(&h[rs_digit(keys[i], shift)], 1u);
    }
    __syncthreads();
    hist[(int64_t)tile * kRsBins + threadIdx.x] = h[threadIdx.x];
}

// per digit: exclusive prefix sums of the histograms of chunk blockIdx.y's tiles, in place, and its total
__global__ void __launch_bounds__(256) k_rs_prefix(uint32_t* __restrict__ hist, int tiles, int per,
                                                   uint32_t* __restrict__ ctot)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    const int t0 = blockIdx.y * per, t1 = min(tiles, t0 + per);
    uint32_t run = 0u;
    for (int t = t0; t < t1; t += 8) {
        uint32_t v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = t + k < t1 ? hist[(int64_t)(t + k) * kRsBins + b] : 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (t + k < t1) hist[(int64_t)(t + k) * kRsBins + b] = run;
            run += v[k];
        }
    }
    ctot[(int64_t)blockIdx.y * kRsBins + b] = run;
}

// vin == nullptr: the first pass, where a key's value is its index
__global__ void __launch_bounds__(kRsThreads, 8) k_rs_scatter(const uint64_t* __restrict__ keys,
                                                           const uint32_t* __restrict__ vin, int64_t n, int shift,
                                                           const uint32_t* __restrict__ hist, int tiles, int per,
                                                           int chunks, const uint32_t* __restrict__ ctot,
                                                           uint64_t* __restrict__ kout, uint32_t* __restrict__ vout)
{
    // the ranks' counts, then the tile's keys in digit order, then its values: two workgroups fit a CU
    __shared__ union {
        RsLds rank;
        uint64_t key[kRsTile];
        uint32_t val[kRsTile];
    } U;
    __shared__ uint32_t gbase[kRsBins];
    RsLds& S = U.rank;
    const int tile = rs_tile(blockIdx.x, tiles);
    if (tile >= tiles) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t base = (int64_t)tile * kRsTile;
    const int cnt = (int)((n - base) < kRsTile ? (n - base) : kRsTile);
    uint64_t kk[kRsItems];
    uint32_t rank[kRsItems];
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {
        const int p = wv * (64 * kRsItems) + c * 64 + lane;
        kk[c] = p < cnt ? keys[base + p] : 0ull;
    }
    // where this tile's keys of digit threadIdx.x go
    uint32_t total = 0u, before = hist[(int64_t)tile * kRsBins + threadIdx.x];
    const int mine = tile / per;
    for (int c = 0; c < chunks; ++c) {
        const uint32_t t = ctot[(int64_t)c * kRsBins + threadIdx.x];
        before += c < mine ? t : 0u;
        total += t;
    }
    const uint32_t first = block_exclusive_scan(total, S.ws);
    rs_rank(S, kk, rank, cnt, shift);
    gbase[threadIdx.x] = first + before - S.start[threadIdx.x];
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {   // a key's rank becomes its place in the tile
        const uint32_t d = rs_digit(kk[c], shift);
        rank[c] += S.start[d] + S.wcnt[wv][d];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kRsItems; ++c)
        if (wv * (64 * kRsItems) + c * 64 + lane < cnt) U.key[rank[c]] = kk[c];
    __syncthreads();
    uint32_t vv[kRsItems];   // (loaded only here, when the keys' registers are free)
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {
        const int p = wv * (64 * kRsItems) + c * 64 + lane;
        vv[c] = p < cnt ? (vin ? vin[base + p] : (uint32_t)(base + p)) : 0u;
    }
    uint32_t gpos[kRsItems];
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {
        const int p = c * kRsThreads + threadIdx.x;
        if (p < cnt) {
            const uint64_t key = U.key[p];
            gpos[c] = gbase[rs_digit(key, shift)] + (uint32_t)p;
            kout[gpos[c]] = key;
        }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kRsItems; ++c)
        if (wv * (64 * kRsItems) + c * 64 + lane < cnt) U.val[rank[c]] = vv[c];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {
        const int p = c * kRsThreads + threadIdx.x;
        if (p < cnt) vout[gpos[c]] = U.val[p];
    }
}

// Codes sorted by their bits from `shift` up, equals in input order: puts the run of equal such bits
// that starts at i in full order if it has at most kRsRun codes, and returns true where a longer
// run descends at i.  Other threads reorder their own runs meanwhile, which changes no code's top
// bits, and nothing but these decides where a run ends.
template <class V>
__device__ __forceinline__ bool rs_finish_run(uint64_t* keys, V* vals, int64_t n, int64_t i, int shift)
{
    const uint64_t k = keys[i], top = k >> shift;
    const uint64_t p = i > 0 ? keys[i - 1] : ~0ull, q = i + 1 < n ? keys[i + 1] : ~0ull;   // (a code has 60 bits)
    if ((p >> shift) != top) {
        if ((q >> shift) != top) return false;   // most codes
        int len = 2;
        while (len <= kRsRun && i + len < n && (keys[i + len] >> shift) == top) ++len;
        if (len > kRsRun) return false;
        for (int a = 1; a < len; ++a) {
            const uint64_t x = keys[i + a];
            int b = a;
            while (b > 0 && keys[i + b - 1] > x) --b;
            if (b == a) continue;
            const V v = vals[i + a];
            for (int c = a; c > b; --c) {
                keys[i + c] = keys[i + c - 1];
                vals[i + c] = vals[i + c - 1];
            }
            keys[i + b] = x;
            vals[i + b] = v;
        }
        return false;
    }
    if (k >= p) return false;
    int len = 1;
    for (int64_t j = i; len <= kRsRun && j > 0 && (keys[j - 1] >> shift) == top; --j) ++len;
    for (int64_t j = i + 1; len <= kRsRun && j < n && (keys[j] >> shift) == top; ++j) ++len;
    return len > kRsRun;
}

// again: set to 1 where the passes over all bits have to follow
__global__ void k_rs_finish(uint64_t* __restrict__ keys, uint32_t* __restrict__ vals, int64_t n, int shift,
                            float* __restrict__ again)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && rs_finish_run(keys, vals, n, i, shift)) *again = 1.0f;
}

// At most one tile: codes, the whole sort in LDS and the gather in one
// workgroup, where the passes' launches would cost more than their work.
__global__ void __launch_bounds__(kRsThreads) k_sort_small(const float* __restrict__ src, const float* __restrict__ w,
                                                           const float* __restrict__ nrm, int n,
                                                           const float* __restrict__ params,
                                                           uint64_t* __restrict__ codes, uint32_t* __restrict__ perm,
                                                           float4* __restrict__ pts, float4* __restrict__ pdip)
{
    __shared__ RsLds S;
    __shared__ uint64_t kbuf[kRsTile];
    __shared__ uint16_t vbuf[kRsTile];
    __shared__ int again;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint64_t kk[kRsItems];
    uint32_t vv[kRsItems], rank[kRsItems];
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {
        const int p = wv * (64 * kRsItems) + c * 64 + lane;
        kk[c] = p < n ? morton_code(load3(src, p), params) : 0ull;
        vv[c] = (uint32_t)p;
    }
    bool all = false;
    for (int pass = kRsPasses - kRsTopPassesSmall; pass < kRsPasses; ++pass) {
        const int shift = pass * kRsBits;
        rs_rank(S, kk, rank, n, shift);
#pragma unroll
        for (int c = 0; c < kRsItems; ++c) {
            const int p = wv * (64 * kRsItems) + c * 64 + lane;
            const uint32_t d = rs_digit(kk[c], shift);
            const uint32_t l = S.start[d] + S.wcnt[wv][d] + rank[c];
            if (p < n) {
                kbuf[l] = kk[c];
                vbuf[l] = (uint16_t)vv[c];
            }
        }
        if (threadIdx.x == 0) again = 0;
        __syncthreads();
        if (pass == kRsPasses - 1 && !all) {
            for (int p = threadIdx.x; p < n; p += kRsThreads)
                if (rs_finish_run(kbuf, vbuf, n, p, (kRsPasses - kRsTopPassesSmall) * kRsBits)) again = 1;
            __syncthreads();
            if (again) {
                all = true;
                pass = -1;
            }
        }
#pragma unroll
        for (int c = 0; c < kRsItems; ++c) {
            const int p = wv * (64 * kRsItems) + c * 64 + lane;
            kk[c] = p < n ? kbuf[p] : 0ull;
            vv[c] = p < n ? vbuf[p] : 0u;
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < kRsItems; ++c) {
        const int p = wv * (64 * kRsItems) + c * 64 + lane;
        if (p >= n) continue;
        const float3v x = load3(src, vv[c]);
        const float wi = w[vv[c]];
        codes[p] = kk[c];
        perm[p] = vv[c];
        pts[p] = make_float4(x.x, x.y, x.z, wi);
        if (pdip) pdip[p] = point_dipole(load3(nrm, vv[c]), wi);
    }
}

// Scratch of the sort beside the second key and value buffers: the histograms and the chunks' totals.
static int rs_tiles(int64_t n) { return (int)((n + kRsTile - 1) / kRsTile); }
static int rs_per_chunk(int tiles) { return std::max(32, (tiles + kRsMaxChunks - 1) / kRsMaxChunks); }

// The codes in keys sorted in place by their digits from `first` on, with their values in vals
// (an even number of passes); fresh: their values are their indices 0 .. n - 1.
static hipError_t radix_sort_pairs(uint64_t* keys, uint32_t* vals, uint64_t* keys_tmp, uint32_t* vals_tmp, int64_t n,
                                   int first, bool fresh, uint32_t* hist, uint32_t* ctot, hipStream_t s)
{
    const int tiles = rs_tiles(n), per = rs_per_chunk(tiles), chunks = (tiles + per - 1) / per;
    const unsigned grid = (unsigned)((tiles + 7) / 8 * 8);
    for (int pass = 0; pass < kRsPasses - first; ++pass) {
        const int shift = (first + pass) * kRsBits;
        const bool even = pass % 2 == 0;
        const uint64_t* ks = even ? keys : keys_tmp;
        k_rs_hist<<<grid, kRsThreads, 0, s>>>(ks, n, shift, hist, tiles);
        k_rs_prefix<<<dim3(kRsBins / 256, (unsigned)chunks), 256, 0, s>>>(hist, tiles, per, ctot);
        k_rs_scatter<<<grid, kRsThreads, 0, s>>>(ks, fresh && pass == 0 ? nullptr : even ? vals : vals_tmp, n, shift, hist, tiles,
                                                 per, chunks, ctot, even ? keys_tmp : keys, even ? vals_tmp : vals);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// 4. Topology
// ---------------------------------------------------------------------------
// Level of the deepest node that holds both codes: their common leading digits
// (60 / bits for equal codes).  recip: ceil(2^16 / bits), by which the division
// of at most 60 is a product.
__device__ __forceinline__ int common_level(uint64_t a, uint64_t b, uint32_t recip)
{
    const uint64_t x = a ^ b;
    return (int)(((x == 0ull ? 60u : (uint32_t)__clzll((long long)x) - 4u) * recip) >> 16);
}

// Marks of point i: the nodes that start at it are those of levels s .. e, the
// internal ones those of levels s .. w (none when s > e).
//   w: a node that holds the leaf_size + 1 points from i on has more than
//      leaf_size points, so the nodes at i are internal down to the common
//      level of codes i and i + leaf_size (and above max_level);
//   s: one level below the deepest node that holds both i - 1 and i, if that
//      node is internal, that is if some leaf_size + 1 consecutive points
//      around i share its prefix.
constexpr int kTopoLevels = 22;    // levels of a tree: at most 60 / 3 + 1 = 21
constexpr int kTopoThreads = 256;
constexpr int kTopoChunks = 2;     // groups of 64 consecutive points per wavefront
constexpr int kTopoPoints = kTopoThreads * kTopoChunks;
struct Mark {
    int s, e, w;
};
__device__ __forceinline__ uint16_t pack_mark(Mark m) { return (uint16_t)(m.s | (m.e << 5) | ((m.w + 1) << 10)); }
__device__ __forceinline__ Mark unpack_mark(uint16_t v) { return {v & 31, (v >> 5) & 31, (int)(v >> 10) - 1}; }
constexpr uint16_t kNoNode = 31;   // s = 31, e = 0, w = -1

// adds to lane l the wavefront's nodes and internal nodes of level l
__device__ __forceinline__ void count_levels(Mark m, int lane, uint32_t& cn, uint32_t& ci)
{
    uint64_t todo = __ballot(m.s <= m.e);   // the points with nodes; each round takes the levels of the first one left
    for (uint32_t seen = 0u; todo != 0ull;) {
        const int p = (int)__builtin_ctzll(todo);
        const int s = __builtin_amdgcn_readlane(m.s, p), e = __builtin_amdgcn_readlane(m.e, p);
        for (uint32_t ls = ((2u << e) - (1u << s)) & ~seen; ls != 0u; ls &= ls - 1u) {
            const int l = (int)__builtin_ctz(ls);
            const uint64_t nm = __ballot(m.s <= l && l <= m.e), im = __ballot(m.s <= l && l <= m.w);
            if (lane == l) {
                cn += (uint32_t)__popcll(nm);
                ci += (uint32_t)__popcll(im);
            }
        }
        seen |= (2u << e) - (1u << s);
        // the points whose levels have all been seen
        todo &= __ballot((((2u << m.e) - (1u << m.s)) & ~seen) != 0u);
    }
}

// Marks of every point, and per block of kTopoPoints points the number of
// nodes (channel 2 l) and internal nodes (2 l + 1) of each level that start in
// it: counts[channel * gridDim.x + block].  One ballot per level and wavefront
// chunk, lane l keeping level l's counts.  Latency and vector issue bound it
// (2^22 points: 34 -> 27 us without a division by `bits` and with all of a
// point's windows read at once; blocks of 512 points, where 1,024 left a few
// thousand points to a handful of workgroups: 5,003 points 8.2 -> 4.9 us).
__global__ void __launch_bounds__(kTopoThreads) k_topo_mark(const uint64_t* __restrict__ codes, int64_t n,
                                                            uint32_t recip, int leaf, int max_level,
                                                            uint16_t* __restrict__ marks,
                                                            uint32_t* __restrict__ counts)
{
    __shared__ int8_t win[kTopoPoints + 64];   // w of the block's points and of the leaf_size points before them
    __shared__ uint32_t wc[kTopoThreads / 64][2][kTopoLevels];
    const int64_t base = (int64_t)blockIdx.x * kTopoPoints;
    for (int k = threadIdx.x; k < kTopoPoints + leaf; k += kTopoThreads) {
        const int64_t i = base - leaf + k;
        int w = -1;
        if (i >= 0 && i + leaf < n) w = min(common_level(codes[i], codes[i + leaf], recip), max_level - 1);
        win[k] = (int8_t)w;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t cn = 0u, ci = 0u;
    for (int c = 0; c < kTopoChunks; ++c) {
        const int k = (wv * kTopoChunks + c) * 64 + lane;   // the point's place in the block
        const int64_t i = base + k;
        Mark m{31, 0, -1};
        if (i < n) {
            m.w = win[k + leaf];
            const int up = i == 0 ? -1 : common_level(codes[i - 1], codes[i], recip);   // the parent's level
            int deepest = -1;   // of the windows from i - leaf to i - 1
#pragma unroll 8
            for (int t = 0; t < leaf; ++t) deepest = max(deepest, (int)win[k + t]);
            if (i == 0 || (up < max_level && deepest >= up)) {
                m.s = up + 1;
                m.e = max(m.s, m.w + 1);
            } else {
                m.w = -1;
            }
            marks[i] = pack_mark(m);
        }
        count_levels(m, lane, cn, ci);
    }
    if (lane < kTopoLevels) {
        wc[wv][0][lane] = cn;
        wc[wv][1][lane] = ci;
    }
    __syncthreads();
    if (threadIdx.x < 2 * (max_level + 1)) {
        uint32_t t = 0u;
        for (int v = 0; v < kTopoThreads / 64; ++v) t += wc[v][threadIdx.x & 1][threadIdx.x >> 1];
        counts[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// Exclusive scan of one channel's block counts per workgroup, in place; totals[channel] = its sum.
__global__ void __launch_bounds__(1024) k_topo_scan(uint32_t* __restrict__ counts, int nblocks,
                                                    uint32_t* __restrict__ totals)
{
    __shared__ uint32_t ws[16];
    uint32_t* __restrict__ c = counts + (int64_t)blockIdx.x * nblocks;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t carry = 0u;
    for (int b0 = 0; b0 < nblocks; b0 += 4096) {
        const int b = b0 + 4 * (int)threadIdx.x;
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = b + k < nblocks ? c[b + k] : 0u;
        const uint32_t sum = v[0] + v[1] + v[2] + v[3];
        const uint32_t incl = wave_inclusive_scan(sum, lane);
        if (lane == 63) ws[wv] = incl;
        __syncthreads();
        uint32_t run = carry + incl - sum;
        for (int k = 0; k < 16; ++k) {
            if (k < wv) run += ws[k];
            carry += ws[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (b + k < nblocks) c[b + k] = run;
            run += v[k];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// ---------------------------------------------------------------------------
// 5. Aggregates and packing
// ---------------------------------------------------------------------------
// Aggregates, in float64: from the points of a leaf, from the children's
// float64 aggregates for an internal node (mass, w-weighted centre of mass,
// summed w n, and the second moment about the centre of mass by the
// parallel-axis rule, a sum of non-negative terms).  The tree stores each as
// the float32 nearest to its float64 value: one rounding, so a one-point
// leaf's centre of mass is its point and its second moment exactly 0, as the
// definitions give.
struct BuildArrays {
    // nodes
    int32_t *nbegin, *ncount, *nlevel, *ndigit, *nparent, *nfirst, *nnchild, *npblk;
    float4 *nagg, *ndip;
    float* nspr;
    double4 *agg64, *dip64;
    double *spr64, *quad64;
    // child blocks, by internal node: its node id and its first child
    int32_t *inode, *bfirst;
    uint32_t* btopo;
    float4 *bagg, *bdip;
    float* bspr;
    int ts, d3, has_dip;
};

// stores node g's aggregates, float32 copies also in its slot of its parent's block (pblk, digit)
__device__ __forceinline__ void store_node(const BuildArrays& a, int32_t g, int32_t pblk, int32_t digit, uint32_t count,
                                           double m, double cx, double cy, double cz, double s2, double dx, double dy,
                                           double dz)
{
    const float4 ag = make_float4((float)cx, (float)cy, (float)cz, (float)m);
    const float4 di = make_float4((float)dx, (float)dy, (float)dz, 0.0f);
    a.agg64[g] = make_double4(cx, cy, cz, m);
    a.spr64[g] = s2;
    a.nagg[g] = ag;
    a.nspr[g] = (float)s2;
    a.ncount[g] = (int32_t)count;
    if (a.has_dip) {
        a.dip64[g] = make_double4(dx, dy, dz, 0.0);
        a.ndip[g] = di;
    }
    if (pblk < 0) return;   // the root
    const int64_t slot = (int64_t)pblk * a.d3 + digit;
    a.btopo[(int64_t)pblk * a.ts + digit] = count;
    a.bagg[slot] = ag;
    a.bspr[slot] = (float)s2;
    if (a.has_dip) a.bdip[slot] = di;
}

__device__ __forceinline__ void aggregate_leaf(const BuildArrays& a, int32_t g, int32_t pblk, int32_t digit, int32_t b,
                                               int32_t e, const float4* __restrict__ pts,
                                               const float4* __restrict__ pdip)
{
#pragma clang fp contract(off)
    double m = 0.0, sx = 0.0, sy = 0.0, sz = 0.0, dx = 0.0, dy = 0.0, dz = 0.0;
    float4 p[8];   // eight points' loads in flight together
    for (int32_t s = b; s < e; s += 8) {
        float4 q[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (s + t >= e) continue;
            p[t] = pts[s + t];
            if (pdip) q[t] = pdip[s + t];
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (s + t >= e) continue;
            const double w = p[t].w;
            m += w; sx += w * (double)p[t].x; sy += w * (double)p[t].y; sz += w * (double)p[t].z;
            if (pdip) { dx += q[t].x; dy += q[t].y; dz += q[t].z; }
        }
    }
    const double cx = sx / m, cy = sy / m, cz = sz / m;
    double s2 = 0.0;
    for (int32_t s = b; s < e; s += 8) {
        if (e - b > 8) {   // this group's again
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (s + t < e) p[t] = pts[s + t];
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (s + t >= e) continue;
            const double ex = (double)p[t].x - cx, ey = (double)p[t].y - cy, ez = (double)p[t].z - cz;
            s2 += (double)p[t].w * (ex * ex + ey * ey + ez * ez);
        }
    }
    s2 /= m;
    if (a.quad64) {
        // second-moment tensor about the centre of mass, Q = sum w (p - c)(p - c)^T
        double Q[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int32_t s = b; s < e; ++s) {
            const float4 p = pts[s];
            const double ww = p.w, ex = (double)p.x - cx, ey = (double)p.y - cy, ez = (double)p.z - cz;
            Q[0] += ww * ex * ex; Q[1] += ww * ey * ey; Q[2] += ww * ez * ez;
            Q[3] += ww * ex * ey; Q[4] += ww * ex * ez; Q[5] += ww * ey * ez;
        }
        for (int k = 0; k < 6; ++k) a.quad64[6 * (int64_t)g + k] = Q[k];
    }
    store_node(a, g, pblk, digit, (uint32_t)(e - b), m, cx, cy, cz, s2, dx, dy, dz);
}

// internal node of block k: its children are nodes bfirst[k] .. bfirst[k + 1] - 1 (the children of
// consecutive blocks follow one another through all levels).  Children are read eight at a time,
// all loads in flight together (an octree node's once for both sums).
__device__ __forceinline__ void aggregate_block(const BuildArrays& a, int32_t k, int32_t n_blocks, int32_t n_nodes)
{
#pragma clang fp contract(off)
    const int32_t g = a.inode[k], f = a.bfirst[k], e = k + 1 < n_blocks ? a.bfirst[k + 1] : n_nodes;
    const int32_t pblk = a.npblk[g], digit = a.ndigit[g];
    double m = 0.0, sx = 0.0, sy = 0.0, sz = 0.0, dx = 0.0, dy = 0.0, dz = 0.0;
    uint32_t count = 0u;
    double4 q[8];
    double sp[8];
    for (int32_t c = f; c < e; c += 8) {
        int32_t nc[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (c + t >= e) continue;
            q[t] = a.agg64[c + t];
            sp[t] = a.spr64[c + t];
            nc[t] = a.ncount[c + t];
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (c + t >= e) continue;
            m += q[t].w; sx += q[t].w * q[t].x; sy += q[t].w * q[t].y; sz += q[t].w * q[t].z;
            count += (uint32_t)nc[t];
        }
    }
    const double cx = sx / m, cy = sy / m, cz = sz / m;
    double s2 = 0.0;
    for (int32_t c = f; c < e; c += 8) {
        if (e - f > 8) {   // d = 4 and 8: this group's again
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                if (c + t >= e) continue;
                q[t] = a.agg64[c + t];
                sp[t] = a.spr64[c + t];
            }
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (c + t >= e) continue;
            const double ex = q[t].x - cx, ey = q[t].y - cy, ez = q[t].z - cz;
            s2 += q[t].w * (sp[t] + (ex * ex + ey * ey + ez * ez));
        }
    }
    s2 /= m;
    if (a.has_dip) {
        for (int32_t c = f; c < e; c += 4) {
            double4 d[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (c + t < e) d[t] = a.dip64[c + t];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (c + t < e) { dx += d[t].x; dy += d[t].y; dz += d[t].z; }
        }
    }
    if (a.quad64) {   // parallel-axis rule: Q = sum_c (Q_c + m_c (c_c - c)(c_c - c)^T)
        double Q[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int32_t c = f; c < e; ++c) {
            const double4 qq = a.agg64[c];
            const double* qc = a.quad64 + 6 * (int64_t)c;
            const double ex = qq.x - cx, ey = qq.y - cy, ez = qq.z - cz;
            Q[0] += qc[0] + qq.w * ex * ex; Q[1] += qc[1] + qq.w * ey * ey; Q[2] += qc[2] + qq.w * ez * ez;
            Q[3] += qc[3] + qq.w * ex * ey; Q[4] += qc[4] + qq.w * ex * ez; Q[5] += qc[5] + qq.w * ey * ez;
        }
        for (int t = 0; t < 6; ++t) a.quad64[6 * (int64_t)g + t] = Q[t];
    }
    a.nnchild[g] = e - f;
    store_node(a, g, pblk, digit, count, m, cx, cy, cz, s2, dx, dy, dz);
}

// the internal nodes of one level
__global__ void __launch_bounds__(256) k_aggregate(BuildArrays a, int32_t blk0, int32_t n, int32_t n_blocks,
                                                   int32_t n_nodes)
{
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) aggregate_block(a, blk0 + i, n_blocks, n_nodes);
}

struct TopoOff {
    int32_t node[kTopoLevels + 1];   // first node of each level
    int32_t blk[kTopoLevels + 1];    // first block of each level's internal nodes
};

// The internal nodes of levels top .. 0, which hold few nodes each, in one
// workgroup: a launch per level costs more than its work.
constexpr int kTopThreads = 512, kTopNodes = 1024;
__global__ void __launch_bounds__(kTopThreads) k_aggregate_top(BuildArrays a, TopoOff off, int top, int32_t n_blocks,
                                                             int32_t n_nodes)
{
    for (int l = top; l >= 0; --l) {
        for (int32_t k = off.blk[l] + (int32_t)threadIdx.x; k < off.blk[l + 1]; k += kTopThreads)
            aggregate_block(a, k, n_blocks, n_nodes);
        __threadfence_block();
        __syncthreads();
    }
}

// Every node, from the marks and the scanned counts: a point's nodes are
// numbered, level by level, by the nodes of that level that start before it
// (counts of the blocks before, of the block's wavefronts before, and a
// ballot).  The last node of level l - 1 to start at or before the point is
// its parent, and the first child of a node that starts at the point is its
// node of the next level.  A point with nodes has one leaf (its deepest node);
// the block collects its leaves in LDS and takes their aggregates with every
// lane busy.  Writes of about 180 bytes a node, in parts of lines over a dozen
// arrays, bound it (2^22 surface points: 0.30 GB in 160 us, 65 of them without
// the leaves; 180 with a bisection over all points for the block's last leaf;
// 5,003 points 18 -> 9.5 us).  Gathering the nodes in LDS so that every store is
// a full one (a quarter of the store instructions) gave 157.
__global__ void __launch_bounds__(kTopoThreads) k_topo_emit(const uint64_t* __restrict__ codes,
                                                            const uint16_t* __restrict__ marks, int64_t n,
                                                            const uint32_t* __restrict__ counts, TopoOff off,
                                                            int depth, int bits, BuildArrays a, const float4* __restrict__ pts,
                                                            const float4* __restrict__ pdip)
{
    __shared__ uint32_t wc[kTopoThreads / 64][2][kTopoLevels];
    __shared__ int4 leaves[kTopoPoints];   // {node, parent's block, digit, first point} of the block's leaves
    __shared__ int n_leaves[kTopoThreads / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * kTopoPoints;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint16_t mk[kTopoChunks];
    uint32_t cn = 0u, ci = 0u;   // lane l: level l's nodes and internal nodes before the wavefront's current chunk
    int nl = 0;                  // leaves of the wavefront: one for every point with a node
#pragma unroll
    for (int c = 0; c < kTopoChunks; ++c) {
        const int64_t i = base + (wv * kTopoChunks + c) * 64 + lane;
        mk[c] = i < n ? marks[i] : kNoNode;
        const Mark m = unpack_mark(mk[c]);
        count_levels(m, lane, cn, ci);
        nl += (int)__popcll(__ballot(m.s <= m.e));
    }
    if (lane < kTopoLevels) {
        wc[wv][0][lane] = cn;
        wc[wv][1][lane] = ci;
    }
    if (lane == 0) n_leaves[wv] = nl;
    __syncthreads();
    cn = ci = 0u;
    if (lane <= depth) {
        cn = counts[(int64_t)(2 * lane) * gridDim.x + blockIdx.x];
        ci = counts[(int64_t)(2 * lane + 1) * gridDim.x + blockIdx.x];
        for (int v = 0; v < wv; ++v) {
            cn += wc[v][0][lane];
            ci += wc[v][1][lane];
        }
    }
    int leaf0 = 0, all_leaves = 0;   // leaves of the wavefronts before, and of the block
    for (int v = 0; v < kTopoThreads / 64; ++v) {
        leaf0 += v < wv ? n_leaves[v] : 0;
        all_leaves += n_leaves[v];
    }
#pragma unroll
    for (int c = 0; c < kTopoChunks; ++c) {
        const int64_t i = base + (wv * kTopoChunks + c) * 64 + lane;
        const Mark m = unpack_mark(mk[c]);
        const uint64_t has = __ballot(m.s <= m.e);
        if (has == 0ull) continue;   // no node starts here
        const uint64_t code = i < n ? codes[i] : 0ull;
        int32_t id = -1, blk = -1;               // this point's node of the level before, its block
        int32_t before_n = 0, before_b = 0;      // nodes and blocks of the level before that start at or before it
        int4 lf = make_int4(-1, -1, 0, (int)i);
        for (int l = 0; l <= depth; ++l) {
            const bool node = m.s <= l && l <= m.e, inner = m.s <= l && l <= m.w;
            const uint64_t nm = __ballot(node), im = __ballot(inner);
            int32_t rn = (int32_t)__builtin_amdgcn_readlane((int)cn, l), ri = (int32_t)__builtin_amdgcn_readlane((int)ci, l);
            if (nm == 0ull) {   // (a node of this level starts wherever an internal one of the level before does)
                before_n = rn;
                before_b = ri;
                continue;
            }
            if (lane == l) {
                cn += (uint32_t)__popcll(nm);
                ci += (uint32_t)__popcll(im);
            }
            rn += (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(nm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)nm, 0u));
            ri += (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(im >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)im, 0u));
            if (blk >= 0) {   // the point's internal node of the level before: its children start here
                a.nfirst[id] = off.node[l] + rn;
                a.bfirst[blk] = off.node[l] + rn;
                a.inode[blk] = id;
                a.btopo[(int64_t)blk * a.ts + a.d3] = (uint32_t)(off.blk[l] + ri);
            }
            blk = -1;
            if (node) {
                id = off.node[l] + rn;
                const int32_t digit = l ? (int32_t)(code >> (60 - bits * l)) & (a.d3 - 1) : 0;
                const int32_t pblk = l ? off.blk[l - 1] + before_b - 1 : -1;
                a.nbegin[id] = (int32_t)i;
                a.nlevel[id] = l;
                a.ndigit[id] = digit;
                a.nparent[id] = l ? off.node[l - 1] + before_n - 1 : -1;
                a.npblk[id] = pblk;
                if (inner) {
                    blk = off.blk[l] + ri;
                } else {
                    a.nfirst[id] = -1;
                    a.nnchild[id] = 0;
                    lf = make_int4(id, pblk, digit, (int)i);
                }
            }
            before_n = rn + (node ? 1 : 0);
            before_b = ri + (inner ? 1 : 0);
        }
        if (lf.x >= 0)
            leaves[leaf0 + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u))] = lf;
        leaf0 += (int)__popcll(has);
    }
    __syncthreads();
    // the leaves' aggregates, a thread each: a leaf ends where the next point with a node starts
    for (int k = threadIdx.x; k < all_leaves; k += kTopoThreads) {
        const int4 lf = leaves[k];
        int64_t end;
        if (k + 1 < all_leaves) {
            end = leaves[k + 1].w;
        } else {   // the block's last leaf: the first point past its cell
            const Mark m = unpack_mark(marks[lf.w]);
            const int shift = 60 - bits * m.e;
            const uint64_t pre = codes[lf.w] >> shift;
            int64_t step = 1;   // most leaves end a few points on
            end = (int64_t)lf.w + 1;
            for (; end + step <= n && (codes[end + step - 1] >> shift) == pre; step <<= 1) end += step;
            int64_t hi = end + step - 1 < n ? end + step - 1 : n;
            while (end < hi) {
                const int64_t mid = end + ((hi - end) >> 1);
                if ((codes[mid] >> shift) == pre) end = mid + 1;
                else hi = mid;
            }
        }
        aggregate_leaf(a, lf.x, lf.y, lf.z, lf.w, (int32_t)end, pts, pdip);
    }
}

// binary16 value nearest to x (round to nearest even) as a double: the rounding
// is done on x itself (no float32 rounding first); |x| beyond binary16's range
// gives +-infinity, x below it the nearest subnormal.
__device__ __forceinline__ double f16_round_d(double x)
{
    if (!(x == x) || x == 0.0 || __builtin_isinf(x)) return x;
    int e;
    (void)frexp(x, &e);
    int ex = e - 1;
    if (ex < -14) ex = -14;
    const double quantum = ldexp(1.0, ex - 10);
    const double r = rint(x / quantum) * quantum;
    if (fabs(r) > 65504.0) return x > 0.0 ? __builtin_inf() : -__builtin_inf();
    return r;
}

__device__ __forceinline__ uint32_t f16_bits(double exact16)
{
    const _Float16 h = (_Float16)(float)exact16;   // exact: the value is a binary16 number
    return (uint32_t)__builtin_bit_cast(uint16_t, h);
}

// Compressed aggregates of one level's nodes (offset off, n of them; level
// >= 1), top-down: each node's binary16 offset from its decoded parent in
// units of its cell side sl, and its binary16 fraction of the decoded parent's
// mass, decoded again in float64 for its own children.  agg64 holds the exact
// aggregates (float64 sums, k_aggregate); qagg the decoded ones (com, mass).
__global__ void k_compress(int32_t off, int32_t n, double sl, const int32_t* __restrict__ nparent,
                           const int32_t* __restrict__ npblk, const int32_t* __restrict__ ndig,
                           const double4* __restrict__ agg64, double4* __restrict__ qagg, uint2* __restrict__ bq,
                           int d3)
{
#pragma clang fp contract(off)
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t g = off + i;
    const double4 a = agg64[g];
    const double4 pq = qagg[nparent[g]];
    const double ox = f16_round_d((a.x - pq.x) / sl);
    const double oy = f16_round_d((a.y - pq.y) / sl);
    const double oz = f16_round_d((a.z - pq.z) / sl);
    const double fm = f16_round_d(a.w / pq.w);
    qagg[g] = make_double4(pq.x + ox * sl, pq.y + oy * sl, pq.z + oz * sl, pq.w * fm);
    bq[(int64_t)npblk[g] * d3 + ndig[g]] = make_uint2(f16_bits(ox) | (f16_bits(oy) << 16), f16_bits(oz) | (f16_bits(fm) << 16));
}

// the root's decoded aggregate: its float32 centre of mass and mass
__global__ void k_compress_root(const double4* __restrict__ agg64, double4* __restrict__ qagg)
{
    const double4 a = agg64[0];
    qagg[0] = make_double4((double)(float)a.x, (double)(float)a.y, (double)(float)a.z, (double)(float)a.w);
}

// The children's second-moment tensors into their block slots, scaled for the
// second-order term (rounded once from float64).
__global__ void k_pack_quad(int32_t n_nodes, const int32_t* __restrict__ npblk, const int32_t* __restrict__ ndig,
                            const double* __restrict__ quad64, float4* __restrict__ bquad, int d3)
{
    const int32_t g = blockIdx.x * blockDim.x + threadIdx.x + 1;
    if (g >= n_nodes) return;
    const int64_t slot = (int64_t)npblk[g] * d3 + ndig[g];
    const double* Q = quad64 + 6 * (int64_t)g;
    bquad[2 * slot] = make_float4((float)(1.5 * Q[0]), (float)(1.5 * Q[1]), (float)(1.5 * Q[2]), (float)(3.0 * Q[3]));
    bquad[2 * slot + 1] = make_float4((float)(3.0 * Q[4]), (float)(3.0 * Q[5]), (float)(0.5 * (Q[0] + Q[1] + Q[2])), 0.0f);
}

// ---------------------------------------------------------------------------
// Host orchestration
// ---------------------------------------------------------------------------
namespace {

// The tree's own arrays are carved, at 256-B boundaries, out of three
// allocations (points, nodes, blocks) that the tree frees when it is released.
template <class T>
size_t carve_bytes(int64_t count)
{
    return ((size_t)count * sizeof(T) + 255) & ~(size_t)255;
}

struct Carver {
    char* p;
    template <class T> T* take(int64_t count)
    {
        T* r = (T*)p;
        p += carve_bytes<T>(count);
        return r;
    }
};

// Temporaries of one build: a bump allocator over a few large chunks.  A
// build takes some fifteen temporaries, some large and some of a few bytes.
// Chunks come from the library's allocator on the build's stream and go back to
// it, in stream order, when the build ends.
struct DevPool {
    static constexpr size_t kChunk = (size_t)64 << 20;
    Allocator mem;
    hipStream_t s;
    std::vector<std::pair<void*, size_t>> chunks;
    char* cur = nullptr;
    size_t left = 0;
    hipError_t err = hipSuccess;
    DevPool(const Allocator& a, hipStream_t st) : mem(a), s(st) {}
    template <class T>
    T* alloc(int64_t count)
    {
        if (err != hipSuccess) return nullptr;
        const size_t bytes = (((size_t)(count > 0 ? count : 1) * sizeof(T)) + 255) & ~(size_t)255;
        if (bytes > left) {
            void* p = nullptr;
            const size_t sz = bytes > kChunk ? bytes : kChunk;
            err = dev_alloc(mem, &p, sz, s);
            if (err != hipSuccess) return nullptr;
            chunks.push_back({p, sz});
            cur = (char*)p;
            left = sz;
        }
        T* r = (T*)cur;
        cur += bytes;
        left -= bytes;
        return r;
    }
    ~DevPool()
    {
        for (auto& c : chunks) dev_free(mem, c.first, c.second, s);
    }
};

// what the host reads once per build: the root cube with the validity flag (launch_bbox), and
// the nodes and internal nodes of every level
struct BuildInfo {
    float params[8];
    uint32_t totals[2 * kTopoLevels];
};

inline unsigned nblk(int64_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace

// Builds the tree into *t.  Returns SBH_OK or an error code with *msg set.
sbh_status build_tree_impl(const float* src, const float* w, const float* nrm, int64_t n, int d, int leaf_size,
                           int max_level, int compress, int quadrupole, hipStream_t s, sbh_tree_impl* t,
                           std::string* msg)
{
    DevPool tmp(t->mem, s);
    auto fail_hip = [&](hipError_t e, const char* where) {
        *msg = std::string(where) + ": " + hipGetErrorString(e);
        return e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation ? SBH_ENOMEM : SBH_EHIP;
    };
#define SBH_TRY(expr, where)                        \
    do {                                            \
        hipError_t e_ = (expr);                     \
        if (e_ != hipSuccess) return fail_hip(e_, where); \
    } while (0)
#define SBH_ALLOC_OK(where)                                    \
    do {                                                       \
        if (tmp.err != hipSuccess) return fail_hip(tmp.err, where); \
    } while (0)

    const int lg = d == 2 ? 1 : d == 4 ? 2 : 3;
    const int bits = 3 * lg;
    const int d3 = d * d * d;
    const int ts = topo_stride(d3);
    t->d = d; t->d3 = d3; t->bits = bits; t->leaf_size = leaf_size; t->max_level = max_level;
    t->n_points = n; t->has_normals = nrm != nullptr;

    // 1. root cube + validation
    const int nbb = (int)std::min<int64_t>(1024, (n + 2047) / 2048 > 0 ? (n + 2047) / 2048 : 1);
    BuildInfo* info = tmp.alloc<BuildInfo>(1);
    float* params = reinterpret_cast<float*>(info);   // its first member
    float* partial = tmp.alloc<float>((int64_t)nbb * 8);
    SBH_ALLOC_OK("allocating bbox buffers");
    SBH_TRY(launch_bbox(src, w, nrm, n, params, partial, nbb, s), "bbox kernel");
    // 2-3. codes, sort and the sorted points, in the tree's arrays
    t->slab_bytes[0] = carve_bytes<float4>(n) * (nrm ? 2 : 1) + carve_bytes<uint32_t>(n) + carve_bytes<uint64_t>(n);
    SBH_TRY(dev_alloc(t->mem, &t->slab[0], t->slab_bytes[0], s), "allocating points");
    {
        Carver c{(char*)t->slab[0]};
        t->pts = c.take<float4>(n);
        if (nrm) t->pdip = c.take<float4>(n);
        t->perm = c.take<uint32_t>(n);
        t->codes = c.take<uint64_t>(n);
    }
    const int64_t nblocks = (n + kTopoPoints - 1) / kTopoPoints;
    const int channels = 2 * (max_level + 1);
    uint16_t* marks = tmp.alloc<uint16_t>(n);
    uint32_t* counts = tmp.alloc<uint32_t>(nblocks * channels);
    SBH_ALLOC_OK("allocating topology buffers");
    BuildInfo h;
    // marks and counts of the sorted codes, then the sizes
    auto read_sizes = [&]() -> sbh_status {
        k_topo_mark<<<(unsigned)nblocks, kTopoThreads, 0, s>>>(t->codes, n, (65536u + bits - 1) / bits, leaf_size,
                                                               max_level, marks, counts);
        SBH_TRY(hipGetLastError(), "topology mark kernel");
        k_topo_scan<<<channels, 1024, 0, s>>>(counts, (int)nblocks, info->totals);
        SBH_TRY(hipGetLastError(), "topology scan kernel");
        SBH_TRY(hipMemcpyAsync(&h, info, sizeof(h), hipMemcpyDeviceToHost, s), "sizes copy");
        SBH_TRY(hipStreamSynchronize(s), "sizes sync");
        return SBH_OK;
    };
    if (n <= kRsTile) {
        k_sort_small<<<1, kRsThreads, 0, s>>>(src, w, nrm, (int)n, params, t->codes, t->perm, t->pts, t->pdip);
        SBH_TRY(hipGetLastError(), "sort kernel");
        if (const sbh_status st = read_sizes(); st != SBH_OK) return st;
    } else {
        const int64_t tiles = rs_tiles(n);
        uint64_t* keys2 = tmp.alloc<uint64_t>(n);
        uint32_t* vals2 = tmp.alloc<uint32_t>(n);
        float4* rec = tmp.alloc<float4>(nrm ? 2 * n : n);
        uint32_t* hist = tmp.alloc<uint32_t>(tiles * kRsBins);
        uint32_t* ctot = tmp.alloc<uint32_t>((int64_t)kRsMaxChunks * kRsBins);
        SBH_ALLOC_OK("allocating sort buffers");
        k_morton<<<nblk(n), 256, 0, s>>>(src, w, nrm, n, params, t->codes, rec);
        SBH_TRY(hipGetLastError(), "morton kernel");
        bool top = n <= kRsTopMax;   // the top bits first; the host learns with the sizes if that was not enough
        for (bool fresh = true;; fresh = top = false) {
            const int first = top ? kRsPasses - kRsTopPasses : 0;
            SBH_TRY(radix_sort_pairs(t->codes, t->perm, keys2, vals2, n, first, fresh, hist, ctot, s), "radix sort");
            if (top) {
                k_rs_finish<<<nblk(n), 256, 0, s>>>(t->codes, t->perm, n, first * kRsBits, params + 6);
                SBH_TRY(hipGetLastError(), "sort finish kernel");
            }
            k_gather_points<<<nblk(n), 256, 0, s>>>(rec, t->perm, n, t->pts, t->pdip);
            SBH_TRY(hipGetLastError(), "gather kernel");
            if (const sbh_status st = read_sizes(); st != SBH_OK) return st;
            if (!top || h.params[6] == 0.0f || h.params[5] != 0.0f) break;
        }
    }
    const uint64_t* codes = t->codes;

    // 4. topology
    if (h.params[5] != 0.0f) {
        *msg = "sbh_build: non-finite coordinate or normal, or weight not finite and > 0";
        return SBH_EINVAL;
    }
    t->lo[0] = h.params[0]; t->lo[1] = h.params[1]; t->lo[2] = h.params[2];
    t->side = h.params[3]; t->inv_side = h.params[4];
    for (int l = 0; l < kMaxLevels; ++l) t->diam[l] = (float)(std::sqrt(3.0) * (double)t->side / std::pow((double)d, l));
    TopoOff off{};
    int64_t n_nodes = 0, n_blocks = 0;
    int n_levels = 0;
    for (int l = 0; l <= max_level; ++l) {
        if (h.totals[2 * l] > 0) n_levels = l + 1;
        n_nodes += h.totals[2 * l];
        n_blocks += h.totals[2 * l + 1];
        if (n_nodes >= (int64_t)1 << 31) {
            *msg = "sbh_build: tree too large";
            return SBH_EINVAL;
        }
        off.node[l + 1] = (int32_t)n_nodes;
        off.blk[l + 1] = (int32_t)n_blocks;
    }
    t->n_nodes = n_nodes;
    t->n_blocks = n_blocks;
    t->depth = n_levels - 1;

    // node arrays
    t->slab_bytes[1] =
        carve_bytes<int32_t>(n_nodes) * 7 + carve_bytes<float4>(n_nodes) * (nrm ? 2 : 1) + carve_bytes<float>(n_nodes);
    SBH_TRY(dev_alloc(t->mem, &t->slab[1], t->slab_bytes[1], s), "allocating nodes");
    {
        Carver c{(char*)t->slab[1]};
        t->nbegin = c.take<int32_t>(n_nodes);
        t->ncount = c.take<int32_t>(n_nodes);
        t->nlevel = c.take<int32_t>(n_nodes);
        t->ndigit = c.take<int32_t>(n_nodes);
        t->nparent = c.take<int32_t>(n_nodes);
        t->nfirst = c.take<int32_t>(n_nodes);
        t->nnchild = c.take<int32_t>(n_nodes);
        t->nagg = c.take<float4>(n_nodes);
        if (nrm) t->ndip = c.take<float4>(n_nodes);
        t->nspr = c.take<float>(n_nodes);
    }
    // block arrays
    const int64_t nbk = n_blocks > 0 ? n_blocks : 1;
    {
        const size_t bytes = carve_bytes<uint32_t>(nbk * ts) + carve_bytes<float4>(nbk * d3) * (nrm ? 2 : 1) +
                             carve_bytes<float>(nbk * d3) + (compress ? carve_bytes<uint2>(nbk * d3) : 0) +
                             (quadrupole ? carve_bytes<float4>(2 * nbk * d3) : 0);
        t->slab_bytes[2] = bytes;
        SBH_TRY(dev_alloc(t->mem, &t->slab[2], bytes, s), "allocating blocks");
        SBH_TRY(hipMemsetAsync(t->slab[2], 0, bytes, s), "blocks clear");
        Carver c{(char*)t->slab[2]};
        t->btopo = c.take<uint32_t>(nbk * ts);
        t->bagg = c.take<float4>(nbk * d3);
        t->bspr = c.take<float>(nbk * d3);
        if (nrm) t->bdip = c.take<float4>(nbk * d3);
        if (compress) t->bq = c.take<uint2>(nbk * d3);
        if (quadrupole) t->bquad = c.take<float4>(2 * nbk * d3);
    }
    // nodes and leaves, then the internal nodes bottom-up, each also into its slot of its parent's block
    {
        int32_t* npblk = tmp.alloc<int32_t>(n_nodes);
        int32_t* inode = tmp.alloc<int32_t>(nbk);
        int32_t* bfirst = tmp.alloc<int32_t>(nbk);
        double4* agg64 = tmp.alloc<double4>(n_nodes);
        double4* dip64 = nrm ? tmp.alloc<double4>(n_nodes) : nullptr;
        double* spr64 = tmp.alloc<double>(n_nodes);
        double* quad64 = quadrupole ? tmp.alloc<double>(6 * n_nodes) : nullptr;
        SBH_ALLOC_OK("allocating float64 aggregates");
        const BuildArrays a{t->nbegin, t->ncount, t->nlevel, t->ndigit, t->nparent, t->nfirst, t->nnchild, npblk,
                            t->nagg,   t->ndip,   t->nspr,   agg64,     dip64,      spr64,     quad64,     inode,
                            bfirst,    t->btopo,  t->bagg,   t->bdip,   t->bspr,    ts,        d3,         nrm ? 1 : 0};
        k_topo_emit<<<(unsigned)nblocks, kTopoThreads, 0, s>>>(codes, marks, n, counts, off, t->depth, bits, a, t->pts,
                                                               t->pdip);
        SBH_TRY(hipGetLastError(), "topology kernel");
        int top = -1;   // levels 0 .. top hold at most kTopNodes internal nodes each
        while (top + 1 < n_levels - 1 && off.blk[top + 2] - off.blk[top + 1] <= kTopNodes) ++top;
        for (int l = n_levels - 2; l > top; --l) {
            const int32_t n_int = off.blk[l + 1] - off.blk[l];
            k_aggregate<<<nblk(n_int), 256, 0, s>>>(a, off.blk[l], n_int, (int32_t)n_blocks, (int32_t)n_nodes);
            SBH_TRY(hipGetLastError(), "aggregate kernel");
        }
        if (top >= 0) {
            k_aggregate_top<<<1, kTopThreads, 0, s>>>(a, off, top, (int32_t)n_blocks, (int32_t)n_nodes);
            SBH_TRY(hipGetLastError(), "aggregate kernel");
        }
        if (quadrupole && n_nodes > 1) {
            k_pack_quad<<<nblk(n_nodes - 1), 256, 0, s>>>((int32_t)n_nodes, npblk, t->ndigit, quad64, t->bquad, d3);
            SBH_TRY(hipGetLastError(), "quadrupole pack kernel");
        }
        if (compress && n_nodes > 1) {   // compressed aggregates, top-down from the root's
            double4* qagg = tmp.alloc<double4>(n_nodes);
            SBH_ALLOC_OK("allocating decoded aggregates");
            k_compress_root<<<1, 1, 0, s>>>(agg64, qagg);
            SBH_TRY(hipGetLastError(), "compress kernel");
            for (int l = 1; l < n_levels; ++l) {
                const double sl = (double)t->side / std::pow((double)d, (double)l);
                const int32_t cnt = off.node[l + 1] - off.node[l];
                k_compress<<<nblk(cnt), 256, 0, s>>>(off.node[l], cnt, sl, t->nparent, npblk, t->ndigit, agg64, qagg,
                                                     t->bq, d3);
                SBH_TRY(hipGetLastError(), "compress kernel");
            }
        }
    }
    SBH_TRY(hipStreamSynchronize(s), "build sync");
    return SBH_OK;
#undef SBH_TRY
#undef SBH_ALLOC_OK
}

}  // namespace sbh
