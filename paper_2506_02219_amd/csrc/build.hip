// Tree construction on the GPU (Section 3.1: an octree-like tree over the
// sources with per-node aggregate weight and centre of mass; the summed
// dipole w*n is added for the winding kernel).
//
// Pipeline, every step a kernel on the caller's stream:
//   1. root cube: per-axis min/max, side = largest extent, inv_side =
//      fl32(1/side) (correctly rounded), plus an input validity flag;
//   2. Morton code: cell_a = min(2^20-1, (u32) fl32(fl32(x_a - lo_a) *
//      inv_side) * 2^20), bits of x/y/z interleaved into 60 bits;
//   3. stable LSD radix sort of (code, index), 8-bit digits;
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
        const float x = src[3 * i], y = src[3 * i + 1], z = src[3 * i + 2];
        const float wi = w[i];
        bad |= !(__builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z));
        bad |= !(wi > 0.0f && __builtin_isfinite(wi));
        if (nrm) {
            const float a = nrm[3 * i], b = nrm[3 * i + 1], c = nrm[3 * i + 2];
            bad |= !(__builtin_isfinite(a) && __builtin_isfinite(b) && __builtin_isfinite(c));
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

// params: lo[3], side, inv_side, bad.  One workgroup: each thread folds a
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
}

hipError_t launch_bbox(const float* src, const float* w, const float* nrm, int64_t n, float* params_dev,
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

__global__ void k_morton(const float* __restrict__ src, int64_t n, const float* __restrict__ params,
                         uint64_t* __restrict__ keys, uint32_t* __restrict__ vals)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float inv = params[4];
    const uint32_t cx = quantize(src[3 * i], params[0], inv);
    const uint32_t cy = quantize(src[3 * i + 1], params[1], inv);
    const uint32_t cz = quantize(src[3 * i + 2], params[2], inv);
    keys[i] = spread_bits3(cx) | (spread_bits3(cy) << 1) | (spread_bits3(cz) << 2);
    vals[i] = (uint32_t)i;
}

hipError_t launch_morton(const float* src, int64_t n, const float* params_dev, uint64_t* keys, uint32_t* vals,
                         hipStream_t s)
{
    const int64_t nb = (n + 255) / 256;
    k_morton<<<(unsigned)nb, 256, 0, s>>>(src, n, params_dev, keys, vals);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Exclusive scan of uint32 (tile scan + recursive scan of tile sums)
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, int lane)
{
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_tile(const uint32_t* in, uint32_t* out, int64_t n,
                                                            uint32_t* __restrict__ tile_sums)
{
    __shared__ uint32_t tile[kScanTile];
    __shared__ uint32_t wsum[kScanThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t idx = base + k * kScanThreads + threadIdx.x;
        tile[k * kScanThreads + threadIdx.x] = idx < n ? in[idx] : 0u;
    }
    __syncthreads();
    uint32_t v[kScanItems], tsum = 0;
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = tile[threadIdx.x * kScanItems + k];
        tsum += v[k];
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t incl = wave_inclusive_scan(tsum, lane);
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    uint32_t woff = 0, total = 0;
    for (int k = 0; k < kScanThreads / 64; ++k) {
        if (k < wv) woff += wsum[k];
        total += wsum[k];
    }
    uint32_t run = woff + incl - tsum;
    for (int k = 0; k < kScanItems; ++k) {
        tile[threadIdx.x * kScanItems + k] = run;
        run += v[k];
    }
    __syncthreads();
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t idx = base + k * kScanThreads + threadIdx.x;
        if (idx < n) out[idx] = tile[k * kScanThreads + threadIdx.x];
    }
    if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

__global__ void k_scan_add(uint32_t* out, int64_t n, const uint32_t* __restrict__ offs)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx < n) out[idx] += offs[idx / kScanTile];
}

size_t scan_tmp_size(int64_t n)
{
    size_t total = 1;  // room for the final total
    while (n > 1) {
        const int64_t nb = (n + kScanTile - 1) / kScanTile;
        total += (size_t)nb + 64;
        n = nb;
    }
    return total + 64;
}

// out may alias in.  *total_dev receives the sum of all inputs.
hipError_t scan_exclusive_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total_dev, uint32_t* tmp,
                              hipStream_t s)
{
    if (n <= 0) return hipMemsetAsync(total_dev, 0, sizeof(uint32_t), s);
    const int64_t nb = (n + kScanTile - 1) / kScanTile;
    if (nb == 1) {
        k_scan_tile<<<1, kScanThreads, 0, s>>>(in, out, n, total_dev);
        return hipGetLastError();
    }
    uint32_t* sums = tmp;
    k_scan_tile<<<(unsigned)nb, kScanThreads, 0, s>>>(in, out, n, sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = scan_exclusive_u32(sums, sums, nb, total_dev, tmp + nb + 64, s);
    if (e != hipSuccess) return e;
    k_scan_add<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(out, n, sums);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 3. Stable LSD radix sort of (uint64 key, uint32 value), 8-bit digits.
// Each block owns a tile of 4096 keys; wave w of the block owns the w-th
// quarter and walks it in 16 chunks of 64 in order, so ranks computed as
// (digit offset of the tile) + (earlier waves) + (earlier chunks of this
// wave) + (earlier lanes of this chunk) preserve the input order of equal
// digits.
// ---------------------------------------------------------------------------
constexpr int kRsThreads = 256;
constexpr int kRsWaves = kRsThreads / 64;
constexpr int kRsChunks = 16;
constexpr int kRsTile = kRsThreads * kRsChunks;

__global__ void __launch_bounds__(kRsThreads) k_rs_hist(const uint64_t* __restrict__ keys, int64_t n, int shift,
                                                        uint32_t* __restrict__ hist, int nb)
{
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRsTile;
    for (int k = 0; k < kRsChunks; ++k) {
        const int64_t idx = base + k * kRsThreads + threadIdx.x;
        if (idx < n) atomicAdd(&h[(uint32_t)(keys[idx] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nb + blockIdx.x] = h[threadIdx.x];
}

__global__ void __launch_bounds__(kRsThreads) k_rs_scatter(const uint64_t* __restrict__ keys,
                                                           const uint32_t* __restrict__ vals, int64_t n, int shift,
                                                           const uint32_t* __restrict__ offs, int nb,
                                                           uint64_t* __restrict__ kout, uint32_t* __restrict__ vout)
{
    __shared__ uint32_t wcnt[kRsWaves][256];
    __shared__ uint32_t gbase[256];
    for (int w = 0; w < kRsWaves; ++w) wcnt[w][threadIdx.x] = 0;
    gbase[threadIdx.x] = offs[(int64_t)threadIdx.x * nb + blockIdx.x];
    __syncthreads();
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint64_t kk[kRsChunks];
    uint32_t vv[kRsChunks], rank[kRsChunks], dig[kRsChunks];
    const int64_t wbase = (int64_t)blockIdx.x * kRsTile + (int64_t)wv * (kRsChunks * 64);
    for (int c = 0; c < kRsChunks; ++c) {
        const int64_t idx = wbase + c * 64 + lane;
        const bool valid = idx < n;
        const uint64_t key = valid ? keys[idx] : 0ull;
        const uint32_t d = (uint32_t)(key >> shift) & 255u;
        uint64_t m = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint32_t below = __popcll(m & lt_mask);
        const uint32_t cnt = __popcll(m);
        const uint32_t base = wcnt[wv][d];
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) wcnt[wv][d] = base + cnt;
        __builtin_amdgcn_wave_barrier();
        kk[c] = key;
        vv[c] = valid ? vals[idx] : 0u;
        rank[c] = base + below;
        dig[c] = valid ? d : 256u;
    }
    __syncthreads();
    {
        uint32_t run = 0;
        for (int w = 0; w < kRsWaves; ++w) {
            const uint32_t t = wcnt[w][threadIdx.x];
            wcnt[w][threadIdx.x] = run;
            run += t;
        }
    }
    __syncthreads();
    for (int c = 0; c < kRsChunks; ++c) {
        if (dig[c] < 256u) {
            const uint32_t pos = gbase[dig[c]] + wcnt[wv][dig[c]] + rank[c];
            kout[pos] = kk[c];
            vout[pos] = vv[c];
        }
    }
}

size_t radix_sort_hist_size(int64_t n)
{
    const int64_t nb = (n + kRsTile - 1) / kRsTile;
    return (size_t)nb * 256;
}

hipError_t radix_sort_pairs(uint64_t* keys, uint32_t* vals, uint64_t* keys_tmp, uint32_t* vals_tmp, int64_t n,
                            int begin_bit, int end_bit, uint32_t* hist, uint32_t* scan_tmp, hipStream_t s)
{
    const int nb = (int)((n + kRsTile - 1) / kRsTile);
    uint64_t *ks = keys, *kd = keys_tmp;
    uint32_t *vs = vals, *vd = vals_tmp;
    int passes = 0;
    for (int shift = begin_bit; shift < end_bit; shift += 8, ++passes) {
        k_rs_hist<<<nb, kRsThreads, 0, s>>>(ks, n, shift, hist, nb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = scan_exclusive_u32(hist, hist, (int64_t)nb * 256, scan_tmp, scan_tmp + 1, s);
        if (e != hipSuccess) return e;
        k_rs_scatter<<<nb, kRsThreads, 0, s>>>(ks, vs, n, shift, hist, nb, kd, vd);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        uint64_t* tk = ks; ks = kd; kd = tk;
        uint32_t* tv = vs; vs = vd; vd = tv;
    }
    if (passes & 1) {
        hipError_t e = hipMemcpyAsync(keys, ks, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
        e = hipMemcpyAsync(vals, vs, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// 4. Levels
// ---------------------------------------------------------------------------
struct float3v {
    float x, y, z;
};

__global__ void k_gather_points(const float* __restrict__ src, const float* __restrict__ w,
                                const float* __restrict__ nrm, const uint32_t* __restrict__ perm, int64_t n,
                                float4* __restrict__ pts, float4* __restrict__ pdip)
{
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    const uint32_t i = perm[s];
    const float wi = w[i];
    // a point's three floats in one 12-byte load: the reads are random, so each
    // separate load would be another cache-line request
    float3v x;
    __builtin_memcpy(&x, src + 3 * (int64_t)i, sizeof(x));
    pts[s] = make_float4(x.x, x.y, x.z, wi);
    if (pdip) {
        float3v m;
        __builtin_memcpy(&m, nrm + 3 * (int64_t)i, sizeof(m));
        pdip[s] = make_float4(wi * m.x, wi * m.y, wi * m.z, 0.0f);
    }
}

// Level of the deepest node that holds both codes: their common leading digits
// (60 / bits for equal codes).
__device__ __forceinline__ int common_level(uint64_t a, uint64_t b, int bits)
{
    const uint64_t x = a ^ b;
    return x == 0ull ? 60 / bits : (__clzll((long long)x) - 4) / bits;
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
constexpr int kTopoChunks = 4;     // groups of 64 consecutive points per wavefront
constexpr int kTopoPoints = kTopoThreads * kTopoChunks;
struct Mark {
    int s, e, w;
};
__device__ __forceinline__ uint16_t pack_mark(Mark m) { return (uint16_t)(m.s | (m.e << 5) | ((m.w + 1) << 10)); }
__device__ __forceinline__ Mark unpack_mark(uint16_t v) { return {v & 31, (v >> 5) & 31, (int)(v >> 10) - 1}; }
constexpr uint16_t kNoNode = 31;   // s = 31, e = 0, w = -1

// Marks of every point, and per block of kTopoPoints points the number of
// nodes (channel 2 l) and internal nodes (2 l + 1) of each level that start in
// it: counts[channel * gridDim.x + block].  One ballot per level and wavefront
// chunk, lane l keeping level l's counts.
__global__ void __launch_bounds__(kTopoThreads) k_topo_mark(const uint64_t* __restrict__ codes, int64_t n, int bits,
                                                            int leaf, int max_level, uint16_t* __restrict__ marks,
                                                            uint32_t* __restrict__ counts)
{
    __shared__ int8_t win[kTopoPoints + 64];   // w of the block's points and of the leaf_size points before them
    __shared__ uint32_t wc[kTopoThreads / 64][2][kTopoLevels];
    const int64_t base = (int64_t)blockIdx.x * kTopoPoints;
    for (int k = threadIdx.x; k < kTopoPoints + leaf; k += kTopoThreads) {
        const int64_t i = base - leaf + k;
        int w = -1;
        if (i >= 0 && i + leaf < n) w = min(common_level(codes[i], codes[i + leaf], bits), max_level - 1);
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
            const int up = i == 0 ? -1 : common_level(codes[i - 1], codes[i], bits);   // the parent's level
            bool starts = i == 0;
            if (i > 0 && up < max_level)
                for (int t = 0; t < leaf && !starts; ++t) starts = win[k + t] >= up;   // windows from i - leaf to i - 1
            if (starts) {
                m.s = up + 1;
                m.e = max(m.s, m.w + 1);
            } else {
                m.w = -1;
            }
            marks[i] = pack_mark(m);
        }
        for (int l = 0; l <= max_level; ++l) {
            const uint64_t nm = __ballot(m.s <= l && l <= m.e), im = __ballot(m.s <= l && l <= m.w);
            if (lane == l) {
                cn += (uint32_t)__popcll(nm);
                ci += (uint32_t)__popcll(im);
            }
        }
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
    for (int32_t s = b; s < e; ++s) {
        const float4 p = pts[s];
        const double w = p.w;
        m += w; sx += w * (double)p.x; sy += w * (double)p.y; sz += w * (double)p.z;
        if (pdip) { const float4 q = pdip[s]; dx += q.x; dy += q.y; dz += q.z; }
    }
    const double cx = sx / m, cy = sy / m, cz = sz / m;
    double s2 = 0.0;
    for (int32_t s = b; s < e; ++s) {
        const float4 p = pts[s];
        const double ex = (double)p.x - cx, ey = (double)p.y - cy, ez = (double)p.z - cz;
        s2 += (double)p.w * (ex * ex + ey * ey + ez * ez);
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
// consecutive blocks follow one another through all levels)
__device__ __forceinline__ void aggregate_block(const BuildArrays& a, int32_t k, int32_t n_blocks, int32_t n_nodes)
{
#pragma clang fp contract(off)
    const int32_t g = a.inode[k], f = a.bfirst[k], e = k + 1 < n_blocks ? a.bfirst[k + 1] : n_nodes;
    double m = 0.0, sx = 0.0, sy = 0.0, sz = 0.0, dx = 0.0, dy = 0.0, dz = 0.0;
    uint32_t count = 0u;
    for (int32_t c = f; c < e; ++c) {
        const double4 q = a.agg64[c];
        m += q.w; sx += q.w * q.x; sy += q.w * q.y; sz += q.w * q.z;
        count += (uint32_t)a.ncount[c];
        if (a.has_dip) { const double4 d = a.dip64[c]; dx += d.x; dy += d.y; dz += d.z; }
    }
    const double cx = sx / m, cy = sy / m, cz = sz / m;
    double s2 = 0.0;
    for (int32_t c = f; c < e; ++c) {
        const double4 q = a.agg64[c];
        const double ex = q.x - cx, ey = q.y - cy, ez = q.z - cz;
        s2 += q.w * (a.spr64[c] + (ex * ex + ey * ey + ez * ez));
    }
    s2 /= m;
    if (a.quad64) {   // parallel-axis rule: Q = sum_c (Q_c + m_c (c_c - c)(c_c - c)^T)
        double Q[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int32_t c = f; c < e; ++c) {
            const double4 q = a.agg64[c];
            const double* qc = a.quad64 + 6 * (int64_t)c;
            const double ex = q.x - cx, ey = q.y - cy, ez = q.z - cz;
            Q[0] += qc[0] + q.w * ex * ex; Q[1] += qc[1] + q.w * ey * ey; Q[2] += qc[2] + q.w * ez * ez;
            Q[3] += qc[3] + q.w * ex * ey; Q[4] += qc[4] + q.w * ex * ez; Q[5] += qc[5] + q.w * ey * ez;
        }
        for (int t = 0; t < 6; ++t) a.quad64[6 * (int64_t)g + t] = Q[t];
    }
    a.nnchild[g] = e - f;
    store_node(a, g, a.npblk[g], a.ndigit[g], count, m, cx, cy, cz, s2, dx, dy, dz);
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
constexpr int kTopNodes = 1024;
__global__ void __launch_bounds__(kTopNodes) k_aggregate_top(BuildArrays a, TopoOff off, int top, int32_t n_blocks,
                                                             int32_t n_nodes)
{
    for (int l = top; l >= 0; --l) {
        const int32_t k = off.blk[l] + (int32_t)threadIdx.x;
        if (k < off.blk[l + 1]) aggregate_block(a, k, n_blocks, n_nodes);
        __threadfence_block();
        __syncthreads();
    }
}

// Every node, from the marks and the scanned counts: a point's nodes are
// numbered, level by level, by the nodes of that level that start before it
// (counts of the blocks before, of the block's wavefronts before, and a
// ballot).  The last node of level l - 1 to start at or before the point is
// its parent, and the first child of a node that starts at the point is its
// node of the next level.  A point has at most one leaf (its deepest node),
// whose aggregates follow once the levels are done.
__global__ void __launch_bounds__(kTopoThreads) k_topo_emit(const uint64_t* __restrict__ codes,
                                                            const uint16_t* __restrict__ marks, int64_t n,
                                                            const uint32_t* __restrict__ counts, TopoOff off,
                                                            int depth, int bits, int leaf, int max_level,
                                                            BuildArrays a, const float4* __restrict__ pts,
                                                            const float4* __restrict__ pdip)
{
    __shared__ uint32_t wc[kTopoThreads / 64][2][kTopoLevels];
    const int64_t base = (int64_t)blockIdx.x * kTopoPoints;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint16_t mk[kTopoChunks];
    uint32_t cn = 0u, ci = 0u;   // lane l: level l's nodes and internal nodes before the wavefront's current chunk
#pragma unroll
    for (int c = 0; c < kTopoChunks; ++c) {
        const int64_t i = base + (wv * kTopoChunks + c) * 64 + lane;
        mk[c] = i < n ? marks[i] : kNoNode;
        const Mark m = unpack_mark(mk[c]);
        for (int l = 0; l <= depth; ++l) {
            const uint64_t nm = __ballot(m.s <= l && l <= m.e), im = __ballot(m.s <= l && l <= m.w);
            if (lane == l) {
                cn += (uint32_t)__popcll(nm);
                ci += (uint32_t)__popcll(im);
            }
        }
    }
    if (lane < kTopoLevels) {
        wc[wv][0][lane] = cn;
        wc[wv][1][lane] = ci;
    }
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
#pragma unroll
    for (int c = 0; c < kTopoChunks; ++c) {
        const int64_t i = base + (wv * kTopoChunks + c) * 64 + lane;
        const Mark m = unpack_mark(mk[c]);
        if (__ballot(m.s <= m.e) == 0ull) continue;   // no node starts here
        const uint64_t code = i < n ? codes[i] : 0ull;
        int32_t id = -1, blk = -1;               // this point's node of the level before, its block
        int32_t before_n = 0, before_b = 0;      // nodes and blocks of the level before that start at or before it
        int32_t leaf_id = -1, leaf_pblk = -1, leaf_digit = 0;
        for (int l = 0; l <= depth; ++l) {
            const bool node = m.s <= l && l <= m.e, inner = m.s <= l && l <= m.w;
            const uint64_t nm = __ballot(node), im = __ballot(inner);
            const int32_t rn = (int32_t)__builtin_amdgcn_readlane((int)cn, l) +
                               (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(nm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)nm, 0u));
            const int32_t ri = (int32_t)__builtin_amdgcn_readlane((int)ci, l) +
                               (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(im >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)im, 0u));
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
                    leaf_id = id;
                    leaf_pblk = pblk;
                    leaf_digit = digit;
                }
            }
            before_n = rn + (node ? 1 : 0);
            before_b = ri + (inner ? 1 : 0);
            if (lane == l) {
                cn += (uint32_t)__popcll(nm);
                ci += (uint32_t)__popcll(im);
            }
        }
        if (leaf_id >= 0) {
            // its end: within leaf_size points, except at the deepest level
            const int shift = 60 - bits * m.e;
            const uint64_t pre = code >> shift;
            int64_t end = i + 1;
            while (end < n && end <= i + leaf && (codes[end] >> shift) == pre) ++end;
            if (end == i + leaf + 1 && end < n && (codes[end] >> shift) == pre) {   // the first code past the prefix
                int64_t hi = n;
                while (end < hi) {
                    const int64_t mid = end + ((hi - end) >> 1);
                    if ((codes[mid] >> shift) == pre) end = mid + 1;
                    else hi = mid;
                }
            }
            aggregate_leaf(a, leaf_id, leaf_pblk, leaf_digit, (int32_t)i, (int32_t)end, pts, pdip);
        }
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
// build takes some two hundred temporaries, and one allocation each cost
// several times the build's kernels.  Chunks come from the library's
// allocator on the build's stream and go back to it, in stream order, when
// the build ends.
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
    // 2-3. codes and sort
    uint64_t* keys = tmp.alloc<uint64_t>(n);
    uint32_t* vals = tmp.alloc<uint32_t>(n);
    uint64_t* keys2 = tmp.alloc<uint64_t>(n);
    uint32_t* vals2 = tmp.alloc<uint32_t>(n);
    uint32_t* hist = tmp.alloc<uint32_t>((int64_t)radix_sort_hist_size(n));
    uint32_t* stmp = tmp.alloc<uint32_t>((int64_t)scan_tmp_size((int64_t)radix_sort_hist_size(n)) + 8);
    const int64_t nblocks = (n + kTopoPoints - 1) / kTopoPoints;
    const int channels = 2 * (max_level + 1);
    uint16_t* marks = tmp.alloc<uint16_t>(n);
    uint32_t* counts = tmp.alloc<uint32_t>(nblocks * channels);
    SBH_ALLOC_OK("allocating sort buffers");
    SBH_TRY(launch_morton(src, n, params, keys, vals, s), "morton kernel");
    SBH_TRY(radix_sort_pairs(keys, vals, keys2, vals2, n, 0, 64, hist, stmp, s), "radix sort");

    // sorted points (owned by the tree)
    t->slab_bytes[0] = carve_bytes<float4>(n) * (nrm ? 2 : 1) + carve_bytes<uint32_t>(n) + carve_bytes<uint64_t>(n);
    SBH_TRY(dev_alloc(t->mem, &t->slab[0], t->slab_bytes[0], s), "allocating points");
    {
        Carver c{(char*)t->slab[0]};
        t->pts = c.take<float4>(n);
        if (nrm) t->pdip = c.take<float4>(n);
        t->perm = c.take<uint32_t>(n);
        t->codes = c.take<uint64_t>(n);
    }
    k_gather_points<<<nblk(n), 256, 0, s>>>(src, w, nrm, vals, n, t->pts, t->pdip);
    SBH_TRY(hipGetLastError(), "gather kernel");
    SBH_TRY(hipMemcpyAsync(t->perm, vals, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s), "perm copy");
    SBH_TRY(hipMemcpyAsync(t->codes, keys, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s), "codes copy");
    const uint64_t* codes = t->codes;

    // 4. topology: the marks and counts, then the sizes
    k_topo_mark<<<(unsigned)nblocks, kTopoThreads, 0, s>>>(codes, n, bits, leaf_size, max_level, marks, counts);
    SBH_TRY(hipGetLastError(), "topology mark kernel");
    k_topo_scan<<<channels, 1024, 0, s>>>(counts, (int)nblocks, info->totals);
    SBH_TRY(hipGetLastError(), "topology scan kernel");
    BuildInfo h;
    SBH_TRY(hipMemcpyAsync(&h, info, sizeof(h), hipMemcpyDeviceToHost, s), "sizes copy");
    SBH_TRY(hipStreamSynchronize(s), "sizes sync");
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
        k_topo_emit<<<(unsigned)nblocks, kTopoThreads, 0, s>>>(codes, marks, n, counts, off, t->depth, bits, leaf_size,
                                                               max_level, a, t->pts, t->pdip);
        SBH_TRY(hipGetLastError(), "topology kernel");
        int top = -1;   // levels 0 .. top hold at most kTopNodes internal nodes each
        while (top + 1 < n_levels - 1 && off.blk[top + 2] - off.blk[top + 1] <= kTopNodes) ++top;
        for (int l = n_levels - 2; l > top; --l) {
            const int32_t n_int = off.blk[l + 1] - off.blk[l];
            k_aggregate<<<nblk(n_int), 256, 0, s>>>(a, off.blk[l], n_int, (int32_t)n_blocks, (int32_t)n_nodes);
            SBH_TRY(hipGetLastError(), "aggregate kernel");
        }
        if (top >= 0) {
            k_aggregate_top<<<1, kTopNodes, 0, s>>>(a, off, top, (int32_t)n_blocks, (int32_t)n_nodes);
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
