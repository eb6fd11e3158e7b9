// Exact evaluation of Eq. (1), F(q_j) = sum_i m_i f(p_i, q_j).  The float64
// variant computes every term and the sum in double and provides the
// reference values; the float32 variant is the GPU brute-force comparator.
//
// A workgroup owns 64 U queries (U per lane) and sums sixteen shares of the
// sources for all of them: tiles of 64 consecutive sources, tile t to share t
// mod 16.  Its 16, 4 or 1 wavefronts take the shares, staging tiles in their own
// part of LDS and reading them back as broadcast loads, so that the main loop
// has no workgroup barrier.  The partial sums are added four consecutive shares
// at a time and then four by four, in order, whoever holds them: the result
// does not depend on U, on the number of wavefronts or on the launch.
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

constexpr int kBruteShares = 16;   // the sources' shares, summed apart
constexpr int kBruteCUs = 256;   // compute units of an MI355X
constexpr int kFewSources = 512;   // (brute_waves)
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

__device__ __forceinline__ float exp_r(float x) { return expf(x); }
__device__ __forceinline__ double exp_r(double x) { return exp(x); }
__device__ __forceinline__ float sqrt_r(float x) { return sqrtf(x); }
__device__ __forceinline__ double sqrt_r(double x) { return sqrt(x); }
__device__ __forceinline__ float abs_r(float x) { return fabsf(x); }
__device__ __forceinline__ double abs_r(double x) { return fabs(x); }
__device__ __forceinline__ float fmin_r(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ double fmin_r(double a, double b) { return fmin(a, b); }

// one wavefront's LDS stores become visible to its own loads (and the other way round)
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Adds the sum s1, relative to the distance m1 (s1 = sum w exp(-alpha (r - m1))), to the sum s relative to m.
template <typename R>
__device__ __forceinline__ void merge_smooth(R& m, R& s, R m1, R s1, R alpha)
{
    const R mm = m1 < m ? m1 : m;
    s = fma_r(s, exp_r(-alpha * (m - mm)), s1 * exp_r(-alpha * (m1 - mm)));
    m = mm;
}

// an infinite coordinate and no NaN (one comparison for the others, which are every source in earnest)
__device__ __forceinline__ bool infinitely_far(float x, float y, float z)
{
    if (__builtin_expect(fmaxf(fmaxf(fabsf(x), fabsf(y)), fabsf(z)) < INFINITY, true)) return false;
    return !(__builtin_isnan(x) || __builtin_isnan(y) || __builtin_isnan(z));
}

// Z: the potential's eps is 0 or infinite, so that the squares under the root
// reach 0 (a source at the query gives an infinite term) or infinity.
// The smooth-distance sum is kept relative to the nearest source seen so far
// (s = sum w exp(-alpha (r - rmin))), so that it neither underflows nor
// overflows; the result is rmin - log(s) / alpha.  Sources are taken kSmGroup
// at a time, one test for a nearer source each.  In the share's first tile a
// nearer source is met too often for a branch: in float64, and with few sources,
// each of its terms scales the sum so far or itself instead; in float32 with
// more sources rmin starts at the tile's smallest distance (10^6 queries on 1,000
// sources 850 us, 990 the other way; on 256 in float64 451, 477 this way).
template <int K, typename R, int U, bool Z, int NW>
__global__ void __launch_bounds__(64 * NW) k_brute(const float* __restrict__ src, const float* __restrict__ w,
                                                   const float* __restrict__ nrm, int64_t n,
                                                   const float* __restrict__ queries, int64_t nq, R eps2, R alpha,
                                                   R* __restrict__ out)
{
#pragma clang fp contract(off)
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
    __shared__ Vec4<R> tile[NW][64];
    __shared__ Vec4<R> tdip[WN ? NW : 1][WN ? 64 : 1];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t j0 = (int64_t)blockIdx.x * (64 * U) + lane;
    R qx[U], qy[U], qz[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t j = j0 + 64 * u;
        const bool valid = j < nq;
        qx[u] = valid ? (R)queries[3 * j] : R(0);
        qy[u] = valid ? (R)queries[3 * j + 1] : R(0);
        qz[u] = valid ? (R)queries[3 * j + 2] : R(0);
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
    constexpr int64_t kStride = 64 * kBruteShares;
    const bool online = SM && (std::is_same_v<R, double> || n <= kFewSources);
    constexpr int kOwn = kBruteShares / NW;   // shares of this wavefront
    R grp[U], gmin[U], all[U], amin[U];   // sums of the current four shares, and of the fours before
#pragma unroll
    for (int u = 0; u < U; ++u) {
        grp[u] = all[u] = R(0);
        gmin[u] = amin[u] = kFar;
    }
    int sh = wv * kOwn;
    load((int64_t)sh * 64);
    for (; sh < wv * kOwn + kOwn; ++sh) {
        if ((int64_t)sh * 64 >= n) break;   // this share is empty, and so are the next ones
        R total[U], rmin[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            total[u] = R(0);
            rmin[u] = kFar;
        }
        for (int64_t t0 = (int64_t)sh * 64; t0 < n; t0 += kStride) {
            if (kNoInf && infinitely_far(gx, gy, gz)) tile[wv][lane] = {R(0), R(0), R(0), R(0) * (R)gw};
            else tile[wv][lane] = {(R)gx, (R)gy, (R)gz, (R)gw};
            if constexpr (WN) tdip[wv][lane] = {(R)gw * (R)hx, (R)gw * (R)hy, (R)gw * (R)hz, R(0)};
            load(kOwn == 1 || t0 + kStride < n ? t0 + kStride : (int64_t)(sh + 1) * 64);
            wave_lds_fence();
            const int cnt = (int)((n - t0) < 64 ? (n - t0) : 64);
            if (SM && !online && t0 == (int64_t)sh * 64) {   // the first tile's smallest distance
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
                for (int u = 0; u < U; ++u) rmin[u] = sqrt_r(rmin[u]);
            }
            R acc[U];   // the tile's partial sums, added to the totals after the tile
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = R(0);
            if constexpr (SM) {
                auto take = [&](int k, auto group) {
                    constexpr int G = decltype(group)::value;
                    R r[G][U], pw[G];
#pragma unroll
                    for (int i = 0; i < G; ++i) {
                        const Vec4<R> p = tile[wv][k + i];
                        pw[i] = p.w;
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const R dx = p.x - qx[u], dy = p.y - qy[u], dz = p.z - qz[u];
                            r[i][u] = sqrt_r(fma_r(dz, dz, fma_r(dy, dy, dx * dx)));
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        R m = r[0][u];
#pragma unroll
                        for (int i = 1; i < G; ++i) m = fmin_r(m, r[i][u]);
                        if (m < rmin[u]) {   // a nearer source: the sums so far move to its distance
                            const R f = exp_r(-sharp * (rmin[u] - m));
                            total[u] *= f;
                            acc[u] *= f;
                            rmin[u] = m;
                        }
#pragma unroll
                        for (int i = 0; i < G; ++i) acc[u] = fma_r(pw[i], exp_r(-sharp * (r[i][u] - rmin[u])), acc[u]);
                    }
                };
                int k = 0;
                if (online && t0 == (int64_t)sh * 64) {
                    // (total is still 0)
#pragma unroll 4
                    for (; k < cnt; ++k) {
                        const Vec4<R> p = tile[wv][k];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const R dx = p.x - qx[u], dy = p.y - qy[u], dz = p.z - qz[u];
                            const R r = sqrt_r(fma_r(dz, dz, fma_r(dy, dy, dx * dx)));
                            const bool nearer = r < rmin[u];
                            const R e = exp_r(-sharp * abs_r(r - rmin[u]));
                            acc[u] = fma_r(nearer ? acc[u] : p.w, e, nearer ? p.w : acc[u]);
                            rmin[u] = fmin_r(rmin[u], r);
                        }
                    }
                }
                for (; k + kSmGroup <= cnt; k += kSmGroup) take(k, std::integral_constant<int, kSmGroup>{});
                for (; k < cnt; ++k) take(k, std::integral_constant<int, 1>{});
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
#pragma unroll
        for (int u = 0; u < U; ++u) {   // shares by fours, then the fours, each in order
            if (kOwn > 4 && sh % 4 == 0) {
                if constexpr (SM) merge_smooth(amin[u], all[u], gmin[u], grp[u], sharp);
                else all[u] += grp[u];
                grp[u] = R(0);
                gmin[u] = kFar;
            }
            if constexpr (SM) merge_smooth(gmin[u], grp[u], rmin[u], total[u], sharp);
            else grp[u] += total[u];
        }
    }
    auto finish = [&](int64_t j, R sum, R m) {
        if constexpr (WN) sum *= R(1.0 / (4.0 * M_PI));
        if constexpr (SM) sum = m - log(sum) / alpha;
        // a query with a non-finite coordinate has no defined value
        const float x = queries[3 * j], y = queries[3 * j + 1], z = queries[3 * j + 2];
        const bool fin = __builtin_isfinite(x) && __builtin_isfinite(y) && __builtin_isfinite(z);
        out[j] = fin ? sum : R(NAN);
    };
    if constexpr (NW == 1) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (SM) merge_smooth(amin[u], all[u], gmin[u], grp[u], sharp);
            else all[u] += grp[u];
            if (j0 + 64 * u < nq) finish(j0 + 64 * u, all[u], amin[u]);
        }
    } else {
        // each wavefront's tile holds its U x 64 sums
        static_assert(U <= 4, "a wavefront's tile must hold its partial sums");
        R* part = reinterpret_cast<R*>(&tile[wv][0]);
        __shared__ R pmin[SM ? NW : 1][SM ? 64 * U : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            part[64 * u + lane] = grp[u];
            if constexpr (SM) pmin[wv][64 * u + lane] = gmin[u];
        }
        __syncthreads();
        for (int s = threadIdx.x; s < 64 * U; s += 64 * NW) {   // a query of the workgroup
            const int64_t j = (int64_t)blockIdx.x * (64 * U) + s;
            if (j >= nq) break;
            R sum = R(0), m = kFar;
            for (int v = 0; v < NW; v += NW / 4) {
                R g = R(0), gm = kFar;
                for (int i = v; i < v + NW / 4; ++i) {
                    const R x = reinterpret_cast<const R*>(&tile[i][0])[s];
                    if constexpr (SM) merge_smooth(gm, g, pmin[i][s], x, sharp);
                    else g += x;
                }
                if constexpr (SM) merge_smooth(m, sum, gm, g, sharp);
                else sum += g;
            }
            finish(j, sum, m);
        }
    }
}

template <int K, typename R, bool Z, int NW>
static void launch_brute_nw(const float* src, const float* w, const float* nrm, int64_t n, const float* q, int64_t nq,
                            R eps2, R alpha, void* out, int u, hipStream_t s)
{
    const unsigned blocks = (unsigned)((nq + 64 * u - 1) / (64 * u));
    if constexpr (K != SBH_SMOOTHDIST) {
        if (u == 4) {
            k_brute<K, R, 4, Z, NW><<<blocks, 64 * NW, 0, s>>>(src, w, nrm, n, q, nq, eps2, alpha, (R*)out);
            return;
        }
    }
    if (u >= 2) k_brute<K, R, 2, Z, NW><<<blocks, 64 * NW, 0, s>>>(src, w, nrm, n, q, nq, eps2, alpha, (R*)out);
    else k_brute<K, R, 1, Z, NW><<<blocks, 64 * NW, 0, s>>>(src, w, nrm, n, q, nq, eps2, alpha, (R*)out);
}

// Wavefronts of a workgroup, which share the sixteen shares of the sources.  Sixteen where queries are few
// (16,384 on 1,000 sources, float64 potential: 12 us, 46 with one).  With few sources there is nothing to
// share, and where queries fill the chip sixteen cost more than they save: 10^6 queries in us, one wavefront
// / sixteen: 64 sources, potential 17 / 54 in float32, 34 / 167 in float64, winding number 27 / 100, 51 / 238,
// smooth distance 63 / 224, 121 / 623; 256 sources 58 / 68, 125 / 174, 95 / 103, 192 / 245, 236 / 289,
// 451 / 633; but 1,000 sources 217 / 214 and 1,046 / 851 (float32 potential and smooth distance), and
// 65,536 queries on 256 sources 45 / 26 (float32 smooth distance).  Four where the registers of the longer
// float64 terms leave a CU one workgroup of sixteen: 10^6 queries on 1,000 sources, winding number 688 /
// 769, smooth distance 1,670 / 1,867.
template <int K, typename R>
static int brute_waves(int64_t n, int64_t nq)
{
    if (n <= 64 || (n <= kFewSources && nq >= 1000 * n)) return 1;
    if (std::is_same_v<R, double> && K != SBH_POTENTIAL && nq >= ((int64_t)1 << 18)) return 4;
    return 16;
}

template <int K, typename R, bool Z>
static void launch_brute_u(const float* src, const float* w, const float* nrm, int64_t n, const float* q, int64_t nq,
                           R eps2, R alpha, void* out, hipStream_t s)
{
    const int nw = brute_waves<K, R>(n, nq);
    if (nw == 1) {
        launch_brute_nw<K, R, Z, 1>(src, w, nrm, n, q, nq, eps2, alpha, out, nq >= ((int64_t)1 << 19) ? 2 : 1, s);
    } else if (nw == 4) {
        if constexpr (std::is_same_v<R, double> && K != SBH_POTENTIAL)
            launch_brute_nw<K, R, Z, 4>(src, w, nrm, n, q, nq, eps2, alpha, out, 2, s);
    } else {
        const int u = K != SBH_SMOOTHDIST && nq >= (int64_t)64 * 4 * kBruteCUs ? 4 : nq >= (int64_t)64 * 2 * kBruteCUs ? 2 : 1;
        launch_brute_nw<K, R, Z, 16>(src, w, nrm, n, q, nq, eps2, alpha, out, u, s);
    }
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

// (a launch holds at most 2^32 - 1 work-items along a dimension, and a query takes up to eight from 2^15 on)
constexpr int64_t kBruteQueries = (int64_t)1 << 28;

hipError_t launch_brute(const float* src, const float* w, const float* nrm, int64_t n, const float* queries,
                        int64_t nq, int kernel, float eps, float alpha, int fp64, void* out, hipStream_t s)
{
    hipError_t e = hipSuccess;
    for (int64_t j0 = 0; j0 < nq && e == hipSuccess; j0 += kBruteQueries) {
        const float* q = queries + 3 * j0;
        const int64_t m = nq - j0 < kBruteQueries ? nq - j0 : kBruteQueries;
        void* o = (char*)out + j0 * (fp64 ? sizeof(double) : sizeof(float));
#define SBH_BRUTE(KK)                                                                                     \
    (fp64 ? launch_brute_k<KK, double>(src, w, nrm, n, q, m, (double)eps * (double)eps, (double)alpha, o, s) \
          : launch_brute_k<KK, float>(src, w, nrm, n, q, m, eps * eps, alpha, o, s))
        if (kernel == SBH_POTENTIAL) e = SBH_BRUTE(SBH_POTENTIAL);
        else if (kernel == SBH_WINDING) e = SBH_BRUTE(SBH_WINDING);
        else e = SBH_BRUTE(SBH_SMOOTHDIST);
#undef SBH_BRUTE
    }
    return e;
}

}  // namespace sbh
