// Exact evaluation of Eq. (1), F(q_j) = sum_i m_i f(p_i, q_j).  The float64
// variant computes every term and the sum in double and provides the
// reference values; the float32 variant is the GPU brute-force comparator.
//
// A workgroup of 16 wavefronts owns 64 U queries (U per lane), and every
// wavefront sums its own share of the sources for all of them: tiles of 64
// consecutive sources, tile t to wavefront t mod 16, staged in the
// wavefront's own part of LDS and read back as broadcast loads, so that the
// main loop has no workgroup barrier.  The sixteen partial sums are added in
// wavefront order at the end.  The shares do not depend on U or on the
// launch, and neither does the result.
//
// The arithmetic bounds it (vector issue).  Splitting the sources inside the
// workgroup is what fills the chip for the query counts of an error
// measurement: 16,384 queries against 2^20 sources are 256 workgroups of 16
// wavefronts, where one query per lane and all sources per lane (the former
// kernel) gave 64 workgroups of four.  U is the largest of 4, 2, 1 that still
// leaves a workgroup for each of the 256 compute units: more queries per lane
// mean fewer LDS reads per term (the smooth distance stops at 2: its groups of
// sources fill the registers, 27.6 against 26.8 ms in float64 for 2^14 sources
// x 10^6 queries with 4).  Measured, one query per lane and a correctly rounded
// square root and division before -> now, 2^18 sources x 2^14 queries: float64
// potential 27.5 -> 2.2 ms, winding 42.7 -> 3.7, smooth distance 47.5 -> 6.9;
// float32 23.8 -> 1.04, 42.7 -> 1.86, 42.7 -> 4.2.  2^20 x 2^14, float64
// potential: 110.8 -> 9.0 ms, 1.9e12 terms/s, about 20 issue slots a term
// against the 3.9e13 lane operations a second of the chip.
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>
#include <type_traits>

#include "sbh_internal.hpp"

namespace sbh {

constexpr int kBruteWaves = 16;
constexpr int kBruteThreads = 64 * kBruteWaves;
constexpr int kBruteCUs = 256;   // compute units of an MI355X
constexpr int kSmGroup = 4;      // sources of the smooth distance taken together

template <typename R>
struct alignas(16) Vec4 {
    R x, y, z, w;
};

template <bool Z>
__device__ __forceinline__ double rsqrt_r(double x) { return rsqrt64<Z>(x); }
template <bool Z>
__device__ __forceinline__ float rsqrt_r(float x) { return __builtin_amdgcn_rsqf(x); }

__device__ __forceinline__ float fma_r(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_r(double a, double b, double c) { return fma(a, b, c); }

// one wavefront's LDS stores become visible to its own loads (and the other way round)
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ bool infinitely_far(float x, float y, float z)
{
    return (__builtin_isinf(x) || __builtin_isinf(y) || __builtin_isinf(z)) &&
           !(__builtin_isnan(x) || __builtin_isnan(y) || __builtin_isnan(z));
}

// Z: the potential's eps is 0 or infinite, so that the squares under the root
// reach 0 (a source at the query gives an infinite term) or infinity.
// The smooth-distance sum is kept relative to the nearest source seen so far
// (s = sum w exp(-alpha (r - rmin))), so that it neither underflows nor
// overflows; the result is rmin - log(s) / alpha.  Sources are taken kSmGroup
// at a time (one test for a nearer source each); rmin starts at the smallest
// distance of the wavefront's first tile, so that the rescaling of s at a
// nearer source is seldom reached.
template <int K, typename R, int U, bool Z>
__global__ void __launch_bounds__(kBruteThreads) k_brute(const float* __restrict__ src, const float* __restrict__ w,
                                                         const float* __restrict__ nrm, int64_t n,
                                                         const float* __restrict__ queries, int64_t nq, R eps2,
                                                         R alpha, R* __restrict__ out)
{
    constexpr bool WN = K == SBH_WINDING, SM = K == SBH_SMOOTHDIST;
    // (an infinite sharpness gives the distance to the nearest source, which infinity times 0 would lose)
    const R sharp = alpha < R(FLT_MAX) ? alpha : R(FLT_MAX);
    // (finite, so that a source at infinity weighs 0 beside it and a NaN stays one)
    constexpr R kFar = std::is_same_v<R, double> ? R(DBL_MAX) : R(FLT_MAX);
    // Sources a loop iteration.  The float32 winding number issues faster one by one (5.5 against 6.7 ms
    // for 2^14 sources x 10^6 queries): unrolled, the compiler sends every term's comparison through
    // the one vcc register.
    constexpr int kUnroll = WN && std::is_same_v<R, float> ? 1 : 4;
    // rsqrt64<false> takes no infinity: a source there adds its weight times 0 at a finite place instead
    constexpr bool kNoInf = K == SBH_POTENTIAL && std::is_same_v<R, double> && !Z;
    __shared__ Vec4<R> tile[kBruteWaves][64];
    __shared__ Vec4<R> tdip[WN ? kBruteWaves : 1][WN ? 64 : 1];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t j0 = (int64_t)blockIdx.x * (64 * U) + lane;
    R qx[U], qy[U], qz[U], total[U], rmin[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t j = j0 + 64 * u;
        const bool valid = j < nq;
        qx[u] = valid ? (R)queries[3 * j] : R(0);
        qy[u] = valid ? (R)queries[3 * j + 1] : R(0);
        qz[u] = valid ? (R)queries[3 * j + 2] : R(0);
        total[u] = R(0);
        rmin[u] = kFar;
    }
    // the wavefront's next tile travels in registers while the current one is summed
    float gx = 0.f, gy = 0.f, gz = 0.f, gw = 0.f, hx = 0.f, hy = 0.f, hz = 0.f;
    auto load = [&](int64_t t0) {
        const int64_t i = t0 + lane;
        if (i >= n) return;
        gx = src[3 * i];
        gy = src[3 * i + 1];
        gz = src[3 * i + 2];
        gw = w[i];
        if constexpr (WN) {
            hx = nrm[3 * i];
            hy = nrm[3 * i + 1];
            hz = nrm[3 * i + 2];
        }
    };
    constexpr int64_t kStride = 64 * kBruteWaves;
    int64_t t0 = (int64_t)wv * 64;
    load(t0);
    for (; t0 < n; t0 += kStride) {
        // (the smooth distance takes whole groups of sources: lanes past the end hold one infinitely far away)
        if (SM && t0 + lane >= n) tile[wv][lane] = {R(INFINITY), R(0), R(0), R(0)};
        else if (kNoInf && infinitely_far(gx, gy, gz)) tile[wv][lane] = {R(0), R(0), R(0), R(0) * (R)gw};
        else tile[wv][lane] = {(R)gx, (R)gy, (R)gz, (R)gw};
        if constexpr (WN) tdip[wv][lane] = {(R)gw * (R)hx, (R)gw * (R)hy, (R)gw * (R)hz, R(0)};
        load(t0 + kStride);
        wave_lds_fence();
        const int cnt = (int)((n - t0) < 64 ? (n - t0) : 64);
        if (SM && t0 == (int64_t)wv * 64) {   // the first tile's smallest distance
            for (int k = 0; k < cnt; ++k) {
                const Vec4<R> p = tile[wv][k];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const R dx = p.x - qx[u], dy = p.y - qy[u], dz = p.z - qz[u];
                    const R r2 = fma_r(dz, dz, fma_r(dy, dy, dx * dx));
                    rmin[u] = r2 < rmin[u] ? r2 : rmin[u];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) rmin[u] = sqrt(rmin[u]);
        }
        R acc[U];   // the tile's partial sums, added to the totals after the tile
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = R(0);
        if constexpr (SM) {
            for (int k = 0; k < cnt; k += kSmGroup) {
                R r[kSmGroup][U], pw[kSmGroup];
#pragma unroll
                for (int i = 0; i < kSmGroup; ++i) {
                    const Vec4<R> p = tile[wv][k + i];
                    pw[i] = p.w;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const R dx = p.x - qx[u], dy = p.y - qy[u], dz = p.z - qz[u];
                        r[i][u] = sqrt(fma_r(dz, dz, fma_r(dy, dy, dx * dx)));
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    R m = r[0][u];
#pragma unroll
                    for (int i = 1; i < kSmGroup; ++i) m = fmin(m, r[i][u]);
                    if (m < rmin[u]) {   // a nearer source: the sums so far move to its distance
                        const R f = exp(-sharp * (rmin[u] - m));
                        total[u] *= f;
                        acc[u] *= f;
                        rmin[u] = m;
                    }
#pragma unroll
                    for (int i = 0; i < kSmGroup; ++i) acc[u] = fma_r(pw[i], exp(-sharp * (r[i][u] - rmin[u])), acc[u]);
                }
            }
        } else
#pragma unroll kUnroll
        for (int k = 0; k < cnt; ++k) {
            const Vec4<R> p = tile[wv][k];
            Vec4<R> m{};
            if constexpr (WN) m = tdip[wv][k];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const R dx = p.x - qx[u], dy = p.y - qy[u], dz = p.z - qz[u];
                if constexpr (K == SBH_POTENTIAL) {
                    const R r2 = fma_r(dz, dz, fma_r(dy, dy, fma_r(dx, dx, eps2)));
                    acc[u] = fma_r(p.w, rsqrt_r<Z>(r2), acc[u]);
                } else {
                    // (n . d) / (4 pi |d|^3), the constant at the end; a source at the query itself adds nothing
                    const R r2 = fma_r(dz, dz, fma_r(dy, dy, dx * dx));
                    const R ir = rsqrt_r<false>(r2);
                    const R v = fma_r(m.z, dz, fma_r(m.y, dy, m.x * dx)) * (ir * ir * ir);
                    acc[u] += r2 > R(0) ? v : R(0);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) total[u] += acc[u];
        wave_lds_fence();   // the tile is overwritten next
    }
    // the wavefronts' partial sums in wavefront order (each wavefront's tile holds its U x 64 values)
    static_assert(U <= 4, "a wavefront's tile must hold its partial sums");
    R* part = reinterpret_cast<R*>(&tile[wv][0]);
#pragma unroll
    for (int u = 0; u < U; ++u) part[64 * u + lane] = total[u];
    __shared__ R pmin[SM ? kBruteWaves : 1][SM ? 64 * U : 1];
    if constexpr (SM) {
#pragma unroll
        for (int u = 0; u < U; ++u) pmin[wv][64 * u + lane] = rmin[u];
    }
    __syncthreads();
    if (threadIdx.x >= 64 * U) return;
    const int s = threadIdx.x;   // this thread's query of the workgroup
    const int64_t j = (int64_t)blockIdx.x * (64 * U) + s;
    if (j >= nq) return;
    R sum = R(0), m = kFar;
    if constexpr (SM) {
        for (int v = 0; v < kBruteWaves; ++v) m = pmin[v][s] < m ? pmin[v][s] : m;
    }
    for (int v = 0; v < kBruteWaves; ++v) {
        const R x = reinterpret_cast<const R*>(&tile[v][0])[s];
        if constexpr (SM) sum += x * exp(-sharp * (pmin[v][s] - m));
        else sum += x;
    }
    if constexpr (WN) sum *= R(1.0 / (4.0 * M_PI));
    if constexpr (SM) sum = m - log(sum) / alpha;
    // a query with a non-finite coordinate has no defined value
    const float x = queries[3 * j], y = queries[3 * j + 1], z = queries[3 * j + 2];
    const bool fin = __builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z);
    out[j] = fin ? sum : R(NAN);
}

template <int K, typename R, bool Z>
static void launch_brute_u(const float* src, const float* w, const float* nrm, int64_t n, const float* q, int64_t nq,
                           R eps2, R alpha, void* out, hipStream_t s)
{
    const auto blocks = [&](int u) { return (unsigned)((nq + 64 * u - 1) / (64 * u)); };
    if constexpr (K != SBH_SMOOTHDIST) {
        if (nq >= (int64_t)64 * 4 * kBruteCUs) {
            k_brute<K, R, 4, Z><<<blocks(4), kBruteThreads, 0, s>>>(src, w, nrm, n, q, nq, eps2, alpha, (R*)out);
            return;
        }
    }
    if (nq >= (int64_t)64 * 2 * kBruteCUs)
        k_brute<K, R, 2, Z><<<blocks(2), kBruteThreads, 0, s>>>(src, w, nrm, n, q, nq, eps2, alpha, (R*)out);
    else
        k_brute<K, R, 1, Z><<<blocks(1), kBruteThreads, 0, s>>>(src, w, nrm, n, q, nq, eps2, alpha, (R*)out);
}

template <int K, typename R>
static hipError_t launch_brute_k(const float* src, const float* w, const float* nrm, int64_t n, const float* q,
                                 int64_t nq, R eps2, R alpha, void* out, hipStream_t s)
{
    if constexpr (K == SBH_POTENTIAL && std::is_same_v<R, double>) {
        if (eps2 == R(0) || eps2 == R(INFINITY)) {
            launch_brute_u<K, R, true>(src, w, nrm, n, q, nq, eps2, alpha, out, s);
            return hipGetLastError();
        }
    }
    launch_brute_u<K, R, false>(src, w, nrm, n, q, nq, eps2, alpha, out, s);
    return hipGetLastError();
}

hipError_t launch_brute(const float* src, const float* w, const float* nrm, int64_t n, const float* queries,
                        int64_t nq, int kernel, float eps, float alpha, int fp64, void* out, hipStream_t s)
{
#define SBH_BRUTE(KK)                                                                                             \
    (fp64 ? launch_brute_k<KK, double>(src, w, nrm, n, queries, nq, (double)eps * (double)eps, (double)alpha, out, \
                                       s)                                                                         \
          : launch_brute_k<KK, float>(src, w, nrm, n, queries, nq, eps * eps, alpha, out, s))
    if (kernel == SBH_POTENTIAL) return SBH_BRUTE(SBH_POTENTIAL);
    if (kernel == SBH_WINDING) return SBH_BRUTE(SBH_WINDING);
    return SBH_BRUTE(SBH_SMOOTHDIST);
#undef SBH_BRUTE
}

}  // namespace sbh
