// Learned child proposal: an 8 -> 32 -> 32 -> 8 ReLU network on MFMA
// (v_mfma_f32_16x16x16f16: binary16 operands, float32 accumulation).
//
// The paper draws the path index uniformly and leaves importance sampling
// open (Section 3.3); Theorem 1 holds for any child distribution with
// q_c > 0.  At an internal node the network sees one feature per child slot,
// the log of the child's quadrupole score relative to its siblings,
//   score_c = m_c s_c^2 / (|p_c - q|^2 + s_c^2)^(3/2),  f_c = max(-1, ln(score_c / max score) / 16)
// (m_c weight, p_c centre of mass, s_c^2 second moment; f = -1 for an empty
// slot), and returns logits z = W3 h2 + b3 + 16 f.  The proposal is
//   pi_c = exp(z_c) / sum_c' exp(z_c')   over non-empty slots,
//   q_c  = (1 - 1/8) pi_c + (1/8) n_c / n_T,
// so an all-zero network samples in proportion to the scores (the "score"
// proposal, which also runs without the network) and every non-empty child
// keeps q_c >= n_c / (8 n_T).
//
// Parameters: float32 [1608] = W1[32][8] b1[32] W2[32][32] b2[32] W3[8][32]
// b3[8]; the kernels round the weight matrices to binary16 (nearest even).
//
// MFMA fragment layout (16x16x16, wave64): lane l holds A[l%16][4(l/16)+j],
// B[4(l/16)+j][l%16] (j = 0..3) and D[4(l/16)+i][l%16] (i = 0..3).  The
// network is evaluated transposed (weights as A, activations as B), so a
// layer's D fragment, after bias and ReLU, is already the next layer's B
// fragment: inference needs no LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "sbh_internal.hpp"

namespace sbh {

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kOffW1 = 0, kOffB1 = 256, kOffW2 = 288, kOffB2 = 1312, kOffW3 = 1344, kOffB3 = 1600;
constexpr float kLambda = 0.125f;

__device__ __forceinline__ f4 mfma(h4 a, h4 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0); }

// A-operand fragments of the three weight matrices and this lane's biases
struct MlpRegs {
    h4 w1[2];       // [t]: W1[16t + l%16][4(l/16) + j] (inputs >= 8 are 0)
    h4 w2[2][2];    // [t][kc]: W2[16t + l%16][16kc + 4(l/16) + j]
    h4 w3[2];       // [kc]: W3[l%16][16kc + 4(l/16) + j] (outputs >= 8 are 0)
    float b1[2][4], b2[2][4], b3[4];
};

// ---------------------------------------------------------------------------
// Per-lane weight fragments for inference
// ---------------------------------------------------------------------------
__device__ __forceinline__ void mlp_load_regs(MlpRegs& R, const float* __restrict__ prm, int lane)
{
    const int r = lane & 15, q = (lane >> 4) * 4;
    for (int t = 0; t < 2; ++t) {
        h4 w;
        for (int j = 0; j < 4; ++j) w[j] = (q + j < 8) ? (_Float16)prm[kOffW1 + (16 * t + r) * 8 + q + j] : (_Float16)0.0f;
        R.w1[t] = w;
        for (int kc = 0; kc < 2; ++kc) {
            h4 v;
            for (int j = 0; j < 4; ++j) v[j] = (_Float16)prm[kOffW2 + (16 * t + r) * 32 + 16 * kc + q + j];
            R.w2[t][kc] = v;
        }
        h4 u;
        for (int j = 0; j < 4; ++j) u[j] = (r < 8) ? (_Float16)prm[kOffW3 + r * 32 + 16 * t + q + j] : (_Float16)0.0f;
        R.w3[t] = u;
        for (int i = 0; i < 4; ++i) {
            R.b1[t][i] = prm[kOffB1 + 16 * t + q + i];
            R.b2[t][i] = prm[kOffB2 + 16 * t + q + i];
        }
    }
    for (int i = 0; i < 4; ++i) R.b3[i] = (q + i < 8) ? prm[kOffB3 + q + i] : 0.0f;
}

__device__ __forceinline__ h4 bias_relu_h(f4 d, const float* b)
{
    h4 h;
    for (int i = 0; i < 4; ++i) {
        const float v = d[i] + b[i];
        h[i] = v > 0.0f ? (_Float16)v : (_Float16)0.0f;
    }
    return h;
}

// Logits z = W3 h2 + b3 + 16 f of every lane's own sample (features f[8]) for
// the whole wavefront: four groups of 16 samples, eight MFMAs each.  All 64
// lanes must be active.
__device__ __forceinline__ void mlp_forward_wave(const MlpRegs& R, const float f[8], float z[8], int lane)
{
    const int r = lane & 15, hi = lane >> 4;
    for (int g = 0; g < 4; ++g) {
        const int src = 16 * g + r;
        float v[8];
        for (int k = 0; k < 8; ++k) v[k] = __shfl(f[k], src, 64);
        h4 xb;
        for (int j = 0; j < 4; ++j) xb[j] = hi == 0 ? (_Float16)v[j] : hi == 1 ? (_Float16)v[4 + j] : (_Float16)0.0f;
        const f4 zero = {0.f, 0.f, 0.f, 0.f};
        const h4 h1a = bias_relu_h(mfma(R.w1[0], xb, zero), R.b1[0]);
        const h4 h1b = bias_relu_h(mfma(R.w1[1], xb, zero), R.b1[1]);
        const h4 h2a = bias_relu_h(mfma(R.w2[0][1], h1b, mfma(R.w2[0][0], h1a, zero)), R.b2[0]);
        const h4 h2b = bias_relu_h(mfma(R.w2[1][1], h1b, mfma(R.w2[1][0], h1a, zero)), R.b2[1]);
        f4 o = mfma(R.w3[1], h2b, mfma(R.w3[0], h2a, zero));
        for (int i = 0; i < 4; ++i) o[i] += R.b3[i];
        // lane r holds logits 0..3 and lane 16 + r logits 4..7 of sample 16 g + r
        float zl[4], zh[4];
        for (int i = 0; i < 4; ++i) {
            zl[i] = __shfl(o[i], r, 64);
            zh[i] = __shfl(o[i], 16 + r, 64);
        }
        if (hi == g) {
            for (int i = 0; i < 4; ++i) {
                z[i] = zl[i];
                z[4 + i] = zh[i];
            }
        }
    }
    for (int k = 0; k < 8; ++k) z[k] += 16.0f * f[k];   // the features pass straight to the logits
}

// Features of (internal node, query q) from the node's child block: the
// relative log quadrupole score of each slot, -1 for empty slots (and for
// every slot when all scores are 0).
__device__ __forceinline__ void score_features(const float4* __restrict__ ba, const float* __restrict__ bs,
                                               const uint32_t cnt[8], float qx, float qy, float qz, float f[8])
{
#pragma clang fp contract(off)
    float sc[8];
    float smax = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float4 a = ba[c];
        const float s2 = bs[c];
        const float dx = a.x - qx, dy = a.y - qy, dz = a.z - qz;
        const float x = norm2(dx, dy, dz) + s2;
        const float r = x > 0.0f ? __frsqrt_rn(x) : 0.0f;
        const float v = cnt[c] ? a.w * s2 * (r * r * r) : 0.0f;
        sc[c] = v;
        smax = fmaxf(smax, v);
    }
    const float inv = smax > 0.0f ? 1.0f / smax : 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c)
        f[c] = sc[c] >= smax && smax > 0.0f ? 0.0f
             : sc[c] > 0.0f                 ? fmaxf(-1.0f, __logf(sc[c] * inv) * 0.0625f)
                                            : -1.0f;
}

// Proposal without the network (z = 16 f): softmax(16 f)_c is
// max(score_c / max score, e^-16) normalised over the non-empty slots, so no
// logarithm or exponential is needed.
__device__ __forceinline__ void score_probs(const float4* __restrict__ ba, const float* __restrict__ bs,
                                            const uint32_t cnt[8], uint32_t nT, float qx, float qy, float qz,
                                            float qv[8])
{
#pragma clang fp contract(off)
    float sc[8];
    float smax = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float4 a = ba[c];
        const float s2 = bs[c];
        const float dx = a.x - qx, dy = a.y - qy, dz = a.z - qz;
        const float x = norm2(dx, dy, dz) + s2;
        const float r = x > 0.0f ? __frsqrt_rn(x) : 0.0f;
        const float v = cnt[c] ? a.w * s2 * (r * r * r) : 0.0f;
        sc[c] = v;
        smax = fmaxf(smax, v);
    }
    const float inv = smax > 0.0f ? frcp(smax) : 0.0f;
    float tot = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        // a slot whose score is 0 has feature -1, i.e. the floor e^-16 (all slots when every score is 0)
        sc[c] = cnt[c] ? (smax > 0.0f ? fmaxf(sc[c] * inv, 1.12535175e-7f) : 1.0f) : 0.0f;
        tot += sc[c];
    }
    const float w = (1.0f - kLambda) * frcp(tot), fn = kLambda * frcp((float)nT);
#pragma unroll
    for (int c = 0; c < 8; ++c) qv[c] = cnt[c] ? sc[c] * w + (float)cnt[c] * fn : 0.0f;
}

// q_c for the eight slots from the logits and the slot counts; empty slots 0.
__device__ __forceinline__ void learned_probs(const float z[8], const uint32_t cnt[8], uint32_t nT, float qv[8])
{
    float zmax = -INFINITY;
    for (int c = 0; c < 8; ++c)
        if (cnt[c]) zmax = fmaxf(zmax, z[c]);
    float e[8], s = 0.0f;
    for (int c = 0; c < 8; ++c) {
        e[c] = cnt[c] ? __expf(z[c] - zmax) : 0.0f;
        s += e[c];
    }
    const float inv = 1.0f / s, fn = 1.0f / (float)nT;
    for (int c = 0; c < 8; ++c) qv[c] = cnt[c] ? (1.0f - kLambda) * e[c] * inv + kLambda * (float)cnt[c] * fn : 0.0f;
}

// ---------------------------------------------------------------------------
// Forward over rows of features (verification entry point)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_mlp_forward(const float* __restrict__ prm, const float* __restrict__ x,
                                                     int64_t n, float* __restrict__ z)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t w0 = i - lane;
    if (w0 >= n) return;   // whole wavefront past the end
    MlpRegs R;
    mlp_load_regs(R, prm, lane);
    float f[8], o[8];
    for (int k = 0; k < 8; ++k) f[k] = i < n ? x[8 * i + k] : 0.0f;
    mlp_forward_wave(R, f, o, lane);
    if (i < n)
        for (int k = 0; k < 8; ++k) z[8 * i + k] = o[k];
}

// ---------------------------------------------------------------------------
// Training: forward + backward for 64 rows per workgroup, operand fragments
// staged through LDS.  The workgroups' partial gradients are summed in a fixed
// order by reduced_entry (deterministic).
// ---------------------------------------------------------------------------
// A fragment of a 16 x 16 operand, four consecutive k a lane: stored with k along the rows (one
// 8-byte read), or down the columns.
__device__ __forceinline__ h4 frag_row(const _Float16* p, int stride)
{
    const int l = threadIdx.x & 63, r = l & 15, q = (l >> 4) * 4;
    return *reinterpret_cast<const h4*>(p + r * stride + q);
}
__device__ __forceinline__ h4 frag_col(const _Float16* p, int stride)
{
    const int l = threadIdx.x & 63, r = l & 15, q = (l >> 4) * 4;
    h4 v;
    for (int j = 0; j < 4; ++j) v[j] = p[(q + j) * stride + r];
    return v;
}

// Row strides: whole 8-byte (16 for float32) units whose 16 rows start in different banks.
constexpr int kN16 = 16 + 4, kN32 = 32 + 4, kN8 = 8 + 4;
struct TrainLds {
    alignas(16) _Float16 w1[32 * kN16];   // W1 padded to 16 inputs
    alignas(16) _Float16 w2[32 * kN32];
    alignas(16) _Float16 w3[16 * kN32];   // W3 padded to 16 outputs
    alignas(16) _Float16 x[64 * kN16], dz[64 * kN16];
    alignas(16) _Float16 h1[64 * kN32], h2[64 * kN32], dh2[64 * kN32], dh1[64 * kN32];
    alignas(16) float zf[64 * kN8], dh2f[64 * kN32], dh1f[64 * kN32];
    alignas(16) float xf[64 * kN8];   // float32 features (skip term)
    alignas(16) float tg[64 * kN8], cn[64 * kN8];
    alignas(16) float b1[32], b2[32], b3[16];
    float loss[64];
    int valid[64];
};

constexpr int kGradStride = 1608 + 8;   // partial-gradient row: 1608 parameters, then the loss

// one wavefront's LDS stores become visible to its own loads
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a hidden layer's activations max(d + b, 0), four consecutive units of a row
__device__ __forceinline__ void store_relu(_Float16* h, const float* b, f4 d)
{
    const f4 bv = *reinterpret_cast<const f4*>(b);
    h4 v;
    for (int i = 0; i < 4; ++i) {
        const float x = d[i] + bv[i];
        v[i] = x > 0.0f ? (_Float16)x : (_Float16)0.0f;
    }
    *reinterpret_cast<h4*>(h) = v;
}

// a hidden layer's deltas, d where the unit was active, in float32 and binary16
__device__ __forceinline__ void store_delta(float* df, _Float16* dh, const _Float16* h, f4 d)
{
    const h4 a = *reinterpret_cast<const h4*>(h);
    f4 v;
    h4 w;
    for (int i = 0; i < 4; ++i) {
        v[i] = (float)a[i] > 0.0f ? d[i] : 0.0f;
        w[i] = (_Float16)v[i];
    }
    *reinterpret_cast<f4*>(df) = v;
    *reinterpret_cast<h4*>(dh) = w;
}

// Rows [row_begin + 64 b, row_begin + 64 b + 64) for block b; rows >= n or
// with all counts 0 contribute nothing.  Sums (not means) over the rows:
// the deltas stay O(1) in binary16; k_mlp_reduce divides by the row count.
// The chain of dependent layers bounds it, not the matrix units: wavefront g
// takes the 16 rows of group g through both directions on its own, and then a
// quarter of the weight gradients' tiles over all 64 rows (one wavefront for
// all groups in turn took 21.5 us for 8192 rows, four 12.5).  Every global load
// is issued before the first is waited for, the loss is taken from the output
// tile's registers by two lanes a row, four slots each, and rows of LDS start in
// different banks: 6.0.
__global__ void __launch_bounds__(256) k_mlp_grad(const float* __restrict__ prm, const float* __restrict__ X,
                                                  const float* __restrict__ Tg, const float* __restrict__ Cn, int64_t n,
                                                  int64_t row_begin, int64_t rows, float* __restrict__ partial)
{
    __shared__ TrainLds S;
    const int tid = threadIdx.x, l = tid & 63, r = l & 15, q = (l >> 4) * 4;
    const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
    {   // thread t: two columns of row t / 4, and its share of the parameters
        const int row = tid >> 2, k = (tid & 3) * 2;
        const int64_t rel = (int64_t)blockIdx.x * 64 + row, at = 8 * (row_begin + rel) + k;
        const bool in = rel < rows && row_begin + rel < n;
        float2 x = make_float2(0.f, 0.f), t = x, c = x;
        if (in) {
            x = make_float2(X[at], X[at + 1]);
            t = make_float2(Tg[at], Tg[at + 1]);
            c = make_float2(Cn[at], Cn[at + 1]);
        }
        const float w1 = prm[kOffW1 + tid], w3 = prm[kOffW3 + tid];
        float w2[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) w2[i] = prm[kOffW2 + i * 256 + tid];
        const int bi = tid < 32 ? kOffB1 + tid : tid < 64 ? kOffB2 + tid - 32 : kOffB3 + (tid & 7);
        const float b = prm[bi];
        *reinterpret_cast<float2*>(S.xf + row * kN8 + k) = x;
        *reinterpret_cast<float2*>(S.tg + row * kN8 + k) = t;
        *reinterpret_cast<float2*>(S.cn + row * kN8 + k) = c;
        S.x[row * kN16 + k] = (_Float16)x.x;
        S.x[row * kN16 + k + 1] = (_Float16)x.y;
        S.x[row * kN16 + 8 + k] = (_Float16)0.0f;
        S.x[row * kN16 + 9 + k] = (_Float16)0.0f;
        S.w1[(tid >> 3) * kN16 + (tid & 7)] = (_Float16)w1;
        S.w1[(tid >> 3) * kN16 + 8 + (tid & 7)] = (_Float16)0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) S.w2[(8 * i + (tid >> 5)) * kN32 + (tid & 31)] = (_Float16)w2[i];
        S.w3[(tid >> 5) * kN32 + (tid & 31)] = (_Float16)w3;
        S.w3[(8 + (tid >> 5)) * kN32 + (tid & 31)] = (_Float16)0.0f;
        if (tid < 32) S.b1[tid] = b;
        else if (tid < 64) S.b2[tid - 32] = b;
        else if (tid < 72) S.b3[tid - 64] = b;
    }
    __syncthreads();
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    const int s0 = 16 * g;
    const int hr = (s0 + r) * kN32 + q;   // the lane's row and units in the arrays of a hidden layer
    // forward (same operands and accumulation order as inference)
    {
        const h4 x = frag_row(S.x + s0 * kN16, kN16);
        for (int t = 0; t < 2; ++t)
            store_relu(S.h1 + hr + 16 * t, S.b1 + 16 * t + q, mfma(frag_row(S.w1 + 16 * t * kN16, kN16), x, zero));
    }
    wave_lds_sync();
    {
        const h4 ha = frag_row(S.h1 + s0 * kN32, kN32), hb = frag_row(S.h1 + s0 * kN32 + 16, kN32);
        for (int t = 0; t < 2; ++t) {
            f4 d = mfma(frag_row(S.w2 + 16 * t * kN32, kN32), ha, zero);
            d = mfma(frag_row(S.w2 + 16 * t * kN32 + 16, kN32), hb, d);
            store_relu(S.h2 + hr + 16 * t, S.b2 + 16 * t + q, d);
        }
    }
    wave_lds_sync();
    // the outputs of row r, slots q .. q + 3 (none from q = 8 on); loss and dL/dz: soft cross-entropy against the
    // softmax over non-empty slots
    {
        f4 o = mfma(frag_row(S.w3, kN32), frag_row(S.h2 + s0 * kN32, kN32), zero);
        o = mfma(frag_row(S.w3 + 16, kN32), frag_row(S.h2 + s0 * kN32 + 16, kN32), o);
        const int row = s0 + r, at = row * kN8 + (q & 4);
        const f4 x = *reinterpret_cast<const f4*>(S.xf + at);
        const f4 b3 = *reinterpret_cast<const f4*>(S.b3 + (q & 4));
        f4 tg = *reinterpret_cast<const f4*>(S.tg + at), cn = *reinterpret_cast<const f4*>(S.cn + at);
        if (q >= 8) tg = cn = zero;
        float z[4], csum = 0.0f, zmax = -INFINITY;
        for (int i = 0; i < 4; ++i) {
            z[i] = o[i] + b3[i];
            z[i] = z[i] + 16.0f * x[i];
            csum += cn[i];
            if (cn[i] > 0.0f) zmax = fmaxf(zmax, z[i]);
        }
        csum += __shfl_xor(csum, 16, 64);
        zmax = fmaxf(zmax, __shfl_xor(zmax, 16, 64));
        const bool valid = csum > 0.0f;
        // (sums run over the slots in order: the row's second lane carries on from its first)
        float e[4], s = 0.0f, loss = 0.0f;
        for (int i = 0; i < 4; ++i) {
            e[i] = cn[i] > 0.0f ? expf(z[i] - zmax) : 0.0f;
            s += e[i];
        }
        s = __shfl(s, r, 64);
        if (q == 4)
            for (int i = 0; i < 4; ++i) s += e[i];
        s = __shfl(s, r + 16, 64);
        f4 dz;
        h4 dh;
        float lp[4];
        for (int i = 0; i < 4; ++i) {
            const float pi = e[i] / s;
            const bool on = valid && cn[i] > 0.0f;
            const bool counts = on && tg[i] > 0.0f;
            lp[i] = counts ? logf(pi) : 0.0f;
            dz[i] = on ? pi - tg[i] : 0.0f;
            dh[i] = (_Float16)dz[i];
            if (!counts) tg[i] = 0.0f;   // (a target without a count may hold anything)
            loss -= tg[i] * lp[i];
        }
        loss = __shfl(loss, r, 64);
        if (q == 4)
            for (int i = 0; i < 4; ++i) loss -= tg[i] * lp[i];
        *reinterpret_cast<h4*>(S.dz + row * kN16 + q) = dh;
        if (q < 8) *reinterpret_cast<f4*>(S.zf + at) = dz;
        if (q == 4) {
            S.loss[row] = loss;
            S.valid[row] = valid ? 1 : 0;
        }
    }
    wave_lds_sync();
    // back-propagate deltas
    {   // dH2^T = W3^T dZ^T, masked by H2 > 0
        const h4 dz = frag_row(S.dz + s0 * kN16, kN16);
        for (int kt = 0; kt < 2; ++kt) {
            const int at = hr + 16 * kt;
            store_delta(S.dh2f + at, S.dh2 + at, S.h2 + at, mfma(frag_col(S.w3 + 16 * kt, kN32), dz, zero));
        }
    }
    wave_lds_sync();
    {   // dH1^T = W2^T dH2^T, masked by H1 > 0
        const h4 da = frag_row(S.dh2 + s0 * kN32, kN32), db = frag_row(S.dh2 + s0 * kN32 + 16, kN32);
        for (int kt = 0; kt < 2; ++kt) {
            const int at = hr + 16 * kt;
            f4 d = mfma(frag_col(S.w2 + 16 * kt, kN32), da, zero);
            d = mfma(frag_col(S.w2 + 16 * kN32 + 16 * kt, kN32), db, d);
            store_delta(S.dh1f + at, S.dh1 + at, S.h1 + at, d);
        }
    }
    __syncthreads();
    // weight gradients: sums over the 64 rows (K = rows, 16 at a time), two tiles per wavefront
    float* out = partial + (int64_t)blockIdx.x * kGradStride;
    for (int kt = 0; kt < 2; ++kt) {
        f4 d = zero;
        if (g == 0) {          // dW3[c][k] = sum_s dz[s][c] h2[s][k]
            for (int s = 0; s < 4; ++s)
                d = mfma(frag_col(S.dz + 16 * s * kN16, kN16), frag_col(S.h2 + 16 * s * kN32 + 16 * kt, kN32), d);
            for (int i = 0; i < 4; ++i)
                if (q + i < 8) out[kOffW3 + (q + i) * 32 + 16 * kt + r] = d[i];
        } else if (g < 3) {    // dW2[n][k] = sum_s dh2[s][n] h1[s][k]
            const int nt = g - 1;
            for (int s = 0; s < 4; ++s)
                d = mfma(frag_col(S.dh2 + 16 * s * kN32 + 16 * nt, kN32), frag_col(S.h1 + 16 * s * kN32 + 16 * kt, kN32), d);
            for (int i = 0; i < 4; ++i) out[kOffW2 + (16 * nt + q + i) * 32 + 16 * kt + r] = d[i];
        } else {               // dW1[n][k] = sum_s dh1[s][n] x[s][k]
            for (int s = 0; s < 4; ++s)
                d = mfma(frag_col(S.dh1 + 16 * s * kN32 + 16 * kt, kN32), frag_col(S.x + 16 * s * kN16, kN16), d);
            for (int i = 0; i < 4; ++i)
                if (r < 8) out[kOffW1 + (16 * kt + q + i) * 8 + r] = d[i];
        }
    }
    // bias gradients from the float32 deltas, in row order, and the block's loss (fixed-order wave reduction)
    if (g == 0) {
        if (l < 8) {
            float a = 0.0f;
#pragma unroll
            for (int s = 0; s < 64; ++s) a += S.zf[s * kN8 + l];
            out[kOffB3 + l] = a;
        }
        float loss = S.loss[l];
        for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
        const float nvalid = (float)__popcll(__ballot(S.valid[l] != 0));
        if (l == 0) {
            out[1608] = loss;
            out[1609] = nvalid;
        }
    } else if (l < 32 && g < 3) {
        const float* d = g == 1 ? S.dh2f : S.dh1f;
        float a = 0.0f;
#pragma unroll
        for (int s = 0; s < 64; ++s) a += d[s * kN32 + l];
        out[(g == 1 ? kOffB2 : kOffB1) + l] = a;
    }
}

// Means over the rows that count, sums over blocks in a fixed order: entry p
// of the gradient (p <= 1607), the loss (1608), the number of rows (1609).  A
// workgroup takes 64 consecutive entries; its kReduceParts wavefronts each sum
// one run of consecutive blocks in block order, sixteen loads in flight, and the
// runs' sums are added in run order.  Valid in the first wavefront's lanes.
constexpr int kReduceParts = 8;
struct ReduceLds {
    float ps[kReduceParts][64];
    float pc[kReduceParts];
};
__device__ __forceinline__ float reduced_entry(ReduceLds& S, const float* __restrict__ partial, int nblocks)
{
    const int l = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + l, at = p <= 1609 ? p : 1609;
    const int per = (nblocks + kReduceParts - 1) / kReduceParts;
    const int b0 = g * per, b1 = min(nblocks, b0 + per);
    float s = 0.0f, cnt = 0.0f;
    for (int b = b0; b < b1; b += 16) {
        float v[16], c[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int64_t row = (int64_t)min(b + k, b1 - 1) * kGradStride;
            v[k] = partial[row + at];
            c[k] = partial[row + 1609];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (b + k < b1) {
                s += v[k];
                cnt += c[k];
            }
    }
    S.ps[g][l] = s;
    if (l == 0) S.pc[g] = cnt;
    __syncthreads();
    float t = S.ps[0][l], c = S.pc[0];
    for (int k = 1; k < kReduceParts; ++k) {
        t += S.ps[k][l];
        c += S.pc[k];
    }
    return p == 1609 ? c : t / fmaxf(c, 1.0f);
}

__global__ void __launch_bounds__(64 * kReduceParts) k_mlp_reduce(const float* __restrict__ partial, int nblocks,
                                                                  float* __restrict__ grad)
{
    __shared__ ReduceLds S;
    const float v = reduced_entry(S, partial, nblocks);
    const int p = blockIdx.x * 64 + threadIdx.x;
    if (threadIdx.x < 64 && p <= 1609) grad[p] = v;
}

// A training step's second half: the reduction and Adam (Kingma and Ba; state
// m[1608], v[1608]) on the parameters whose gradients the workgroup holds
// (10.2 us with one load in flight per wavefront and 4.4 for Adam's own launch,
// now 3.8 together, sixteen loads in flight).
__global__ void __launch_bounds__(64 * kReduceParts) k_mlp_step(const float* __restrict__ partial, int nblocks,
                                                                float* __restrict__ prm, float* __restrict__ state,
                                                                float lr, float bc1, float bc2,
                                                                float* __restrict__ loss_out)
{
    __shared__ ReduceLds S;
    const int p = blockIdx.x * 64 + threadIdx.x;
    float m0 = 0.0f, v0 = 0.0f, x0 = 0.0f;   // loaded along with the partials
    if (threadIdx.x < 64 && p < 1608) {
        m0 = state[p];
        v0 = state[1608 + p];
        x0 = prm[p];
    }
    const float g = reduced_entry(S, partial, nblocks);
    if (threadIdx.x >= 64) return;
    if (p == 1608 && loss_out) *loss_out = g;
    if (p >= 1608) return;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float m = b1 * m0 + (1.0f - b1) * g;
    const float v = b2 * v0 + (1.0f - b2) * g * g;
    state[p] = m;
    state[1608 + p] = v;
    prm[p] = x0 - lr * (m / bc1) / (sqrtf(v / bc2) + eps);
}

// ---------------------------------------------------------------------------
// Training pairs: uniform paths from every subdomain on the Philox stream
// (query, slot, step/2, 0xFFFFFFFF); each internal node on a path is a row
// [query][slot][depth] with its features, child counts and the location of
// its children block for the target kernel.
// ---------------------------------------------------------------------------
__global__ void k_mlp_pairs(TreeView tv, const float* __restrict__ queries, int64_t nq, int lmax, uint32_t key0,
                            uint32_t key1, float* __restrict__ X, float* __restrict__ Cn, int4* __restrict__ loc)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nq * 8) return;
    const int64_t j = t / 8;
    const int slot = (int)(t % 8);
    const float qx = queries[3 * j], qy = queries[3 * j + 1], qz = queries[3 * j + 2];
    const uint32_t* rt = tv.btopo;
    const uint32_t n_a = tv.root_internal ? rt[slot] : 0u;
    uint32_t beginT = 0u;
    int32_t nint = 0;
    for (int c = 0; c < slot; ++c) {
        beginT += rt[c];
        nint += ((int)rt[c] > tv.leaf_size && 1 < tv.max_level) ? 1 : 0;
    }
    int32_t blk = (int32_t)rt[8] + nint;
    uint32_t nT = n_a;
    int level = 1;
    u32x4 rnd = {0u, 0u, 0u, 0u};
    for (int k = 0; k < lmax; ++k) {
        const int64_t row = (j * 8 + slot) * lmax + k;
        const bool internal = n_a > 0u && (int)nT > tv.leaf_size && level < tv.max_level;
        if (!internal) {
            for (int c = 0; c < 8; ++c) {
                X[8 * row + c] = 0.0f;
                Cn[8 * row + c] = 0.0f;
            }
            loc[row] = make_int4(-1, 0, 0, 0);
            nT = 0u;
            continue;
        }
        const uint32_t* bt = tv.btopo + (int64_t)blk * topo_stride(8);
        uint32_t cnt[8];
        for (int c = 0; c < 8; ++c) cnt[c] = bt[c];
        float f[8];
        score_features(tv.bagg + (int64_t)blk * 8, tv.bspr + (int64_t)blk * 8, cnt, qx, qy, qz, f);
        for (int c = 0; c < 8; ++c) {
            X[8 * row + c] = f[c];
            Cn[8 * row + c] = (float)cnt[c];
        }
        loc[row] = make_int4(blk, (int32_t)beginT, (int32_t)nT, level);
        if ((k & 1) == 0) rnd = philox4x32_10((uint32_t)j, (uint32_t)slot, (uint32_t)(k >> 1), 0xFFFFFFFFu, key0, key1);
        const uint32_t r = __umulhi((k & 1) ? rnd.z : rnd.x, nT);
        uint32_t pre = 0u, preC = 0u, nC = 0u;
        int32_t ni = 0, niC = 0;
        for (int c = 0; c < 8; ++c) {
            const bool hit = (r - pre) < cnt[c];
            preC = hit ? pre : preC;
            niC = hit ? ni : niC;
            nC = hit ? cnt[c] : nC;
            ni += ((int)cnt[c] > tv.leaf_size && level + 1 < tv.max_level) ? 1 : 0;
            pre += cnt[c];
        }
        beginT += preC;
        nT = nC;
        blk = (int32_t)bt[8] + niC;
        ++level;
    }
}

// acc plus the float64 term of one source for the targets (no smooth-distance shift, nor the winding
// number's constant, of which ratios of residuals are free).  SOFT: potential with eps > 0.
template <int K, bool SOFT>
__device__ __forceinline__ double add_term64(double acc, float4 p, float4 dp, double qx, double qy, double qz,
                                             double eps2, double alpha)
{
#pragma clang fp contract(off)   // the same value for points and aggregates: a one-point child's residual is exactly 0
    const double dx = (double)p.x - qx, dy = (double)p.y - qy, dz = (double)p.z - qz;
    if constexpr (K == SBH_POTENTIAL) {
        return fma((double)p.w, rsqrt64<!SOFT>(fma(dz, dz, fma(dy, dy, fma(dx, dx, eps2)))), acc);
    } else if constexpr (K == SBH_WINDING) {
        const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
        const double u = rsqrt64<true>(r2);
        const double v = fma((double)dp.z, dz, fma((double)dp.y, dy, (double)dp.x * dx)) * (u * u * u);
        return acc + (r2 > 0.0 ? v : 0.0);
    } else {
        return fma((double)p.w, exp(-alpha * sqrt(fma(dz, dz, fma(dy, dy, dx * dx)))), acc);
    }
}

// Targets of one path (query, subdomain) per workgroup: for every node T on it
// the float64 sum of each child's points, the residual against the child's
// aggregate term, normalised.  The nodes of a path are nested, so only the
// children that the path does not enter are summed over their points (every
// point of the subdomain once); the sum of an entered child is that of its own
// children.  A large child is shared by the workgroup's wavefronts in eight
// parts, a small one (most of them) is one wavefront's, and the partial sums are
// added in the parts' order, whoever took them.  Path p = 8 j + slot is workgroup p,
// which the round-robin dispatch gives to die p mod 8: each die's L2 keeps one
// subdomain's points for every query (2^20 points: 2 MB of 4).  Float64
// arithmetic and those reads bound it; a workgroup per row, summing every row
// anew with a square root, a division and eight range tests a point, left most
// of the chip to a few rows near the root: 6.5 ms for 512 queries on 2^20
// points, now 0.5 ms (17 float64 instructions a point, 76% of the issue slots).
constexpr int kTgParts = 8;             // parts of a shared child
constexpr int kTgMaxRows = 20;          // internal nodes on a path: at most the tree's levels
constexpr uint32_t kTgShared = 2048;    // points from which a child is shared by the wavefronts

template <int K, bool SOFT, int NW>
__global__ void __launch_bounds__(64 * NW) k_mlp_targets(TreeView tv, const float* __restrict__ queries, int lmax,
                                                         const int4* __restrict__ loc, double eps2, double alpha,
                                                         float* __restrict__ Tg)
{
#pragma clang fp contract(off)
    __shared__ int4 node[kTgMaxRows];                        // {children block, first point, points, level}
    __shared__ uint32_t first[kTgMaxRows][9];                // first point of each child, then the end
    __shared__ double part[kTgMaxRows * 8][kTgParts];
    __shared__ double sums[kTgMaxRows][8], resid[kTgMaxRows][8];
    const int64_t path = blockIdx.x;
    const int64_t row0 = path * lmax, j = path / 8;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double qx = queries[3 * j], qy = queries[3 * j + 1], qz = queries[3 * j + 2];
    if ((int)threadIdx.x < lmax) node[threadIdx.x] = loc[row0 + threadIdx.x];
    __syncthreads();
    int rows = 0;   // the path's nodes are its first rows
    while (rows < lmax && node[rows].x >= 0) ++rows;
    if ((int)threadIdx.x < rows) {
        const int4 L = node[threadIdx.x];
        const uint32_t* bt = tv.btopo + (int64_t)L.x * topo_stride(8);
        uint32_t b = (uint32_t)L.y;
        for (int c = 0; c < 8; ++c) {
            first[threadIdx.x][c] = b;
            b += bt[c];
        }
        first[threadIdx.x][8] = b;
    }
    for (int i = threadIdx.x; i < rows * 8 * kTgParts; i += 64 * NW) (&part[0][0])[i] = 0.0;
    __syncthreads();
    // the child of row k that row k + 1 subdivides
    auto entered = [&](int k, int c) {
        return k + 1 < rows && first[k][c] == (uint32_t)node[k + 1].y && first[k][c + 1] - first[k][c] == (uint32_t)node[k + 1].z;
    };
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < rows * 8; ++s) {
        const int k = s >> 3, c = s & 7;
        const uint32_t b = __builtin_amdgcn_readfirstlane(first[k][c]), e = __builtin_amdgcn_readfirstlane(first[k][c + 1]);
        const bool shared = e - b >= kTgShared;
        if (b == e || (!shared && s % NW != wv) || entered(k, c)) continue;
        const uint32_t step = shared ? 64 * kTgParts : 64;
        for (int v = shared ? wv : 0; v < (shared ? kTgParts : 1); v += NW) {
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            uint32_t u = b + 64u * v;   // the part's next 64 points
            float4 p[4], m[4];          // four loads in flight
            for (; u + 3 * step + 64 <= e; u += 4 * step) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    p[t] = (tv.pts + (u + t * step))[lane];
                    m[t] = K == SBH_WINDING ? (tv.pdip + (u + t * step))[lane] : zero4;
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) a[t] = add_term64<K, SOFT>(a[t], p[t], m[t], qx, qy, qz, eps2, alpha);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (u + t * step + lane >= e) continue;
                p[t] = (tv.pts + (u + t * step))[lane];
                m[t] = K == SBH_WINDING ? (tv.pdip + (u + t * step))[lane] : zero4;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (u + t * step + lane < e) a[t] = add_term64<K, SOFT>(a[t], p[t], m[t], qx, qy, qz, eps2, alpha);
            double acc = (a[0] + a[1]) + (a[2] + a[3]);
            for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
            if (lane == 0) part[s][v] = acc;
        }
    }
    __syncthreads();
    for (int s = threadIdx.x; s < rows * 8; s += 64 * NW) {
        double t = part[s][0];
        for (int v = 1; v < kTgParts; ++v) t += part[s][v];
        sums[s >> 3][s & 7] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0)   // an entered child: the sum of its own children
        for (int k = rows - 2; k >= 0; --k)
            for (int c = 0; c < 8; ++c)
                if (entered(k, c)) {
                    double t = 0.0;
                    for (int d = 0; d < 8; ++d) t += sums[k + 1][d];
                    sums[k][c] = t;
                }
    __syncthreads();
    for (int s = threadIdx.x; s < rows * 8; s += 64 * NW) {
        const int k = s >> 3, c = s & 7;
        double r = 0.0;
        if (first[k][c + 1] != first[k][c]) {
            const int64_t slot = (int64_t)node[k].x * 8 + c;
            r = fabs(sums[k][c] - add_term64<K, SOFT>(0.0, tv.bagg[slot], (K == SBH_WINDING) ? tv.bdip[slot] : zero4, qx, qy, qz, eps2, alpha));
        }
        resid[k][c] = r;
    }
    __syncthreads();
    for (int s = threadIdx.x; s < lmax * 8; s += 64 * NW) {
        const int k = s >> 3, c = s & 7;
        float t = 0.0f;   // rows past the end of the path
        if (k < rows) {
            double rs = 0.0;
            for (int d = 0; d < 8; ++d) rs += resid[k][d];
            t = rs > 0.0 ? (float)(resid[k][c] / rs) : (float)(first[k][c + 1] - first[k][c]) / (float)node[k].z;
        }
        Tg[8 * row0 + s] = t;
    }
}

// ---------------------------------------------------------------------------
// Estimator with the learned (NET) or score proposal (d = 2).  Lanes as in
// the per-query kernel (8 queries x 8 subdomain slots per wavefront, every
// lane its own path); the walk is a wavefront-uniform loop so that the
// network runs on MFMA for all 64 lanes at once, every step at which some
// lane stands on an internal node.  At an internal node the child block is
// scanned first (its terms give the swap, its aggregates the features), then
// a slot is drawn by inverse CDF from q_c with a 24-bit uniform, then the
// roulette of Eq. (5); at a leaf a point is drawn uniformly.  The swap of a
// step is weighted by 1 / (prod q * prod p) (Eq. (7) with p(I in T) the
// product of the selection probabilities).
// ---------------------------------------------------------------------------
struct LearnArgs {
    int32_t samples;
    int32_t group;
    int32_t rr_mode;
    uint32_t batch;
    uint32_t key0, key1;
    float eps2, alpha;
    int32_t* paths;
    const float* prm;
};

template <int K, bool TRACE, bool NET>
__global__ void __launch_bounds__(256) k_sbh_learned(TreeView tv, const float* __restrict__ queries, int64_t nq,
                                                     LearnArgs a, float* __restrict__ out)
{
#pragma clang fp contract(off)
    constexpr int D3 = 8;
    constexpr int TS = topo_stride(D3);
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    const int lane = threadIdx.x & 63;
    const int slot = lane & 7;
    const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t j = wave * 8 + (lane >> 3);
    if (wave * 8 >= nq) return;   // whole wavefront past the end
    const bool valid = j < nq;
    float qx = 0.f, qy = 0.f, qz = 0.f;
    if (valid) {
        qx = queries[3 * j];
        qy = queries[3 * j + 1];
        qz = queries[3 * j + 2];
    }
    MlpRegs R;
    bool net = NET;
    if constexpr (NET) {
        // parameters that are not all finite are ignored (the zero network: the score proposal)
        bool bad = false;
        for (int i = lane; i < kMlpParams; i += 64) bad |= !__builtin_isfinite(a.prm[i]);
        net = __ballot(bad) == 0ull;
        mlp_load_regs(R, a.prm, lane);
    }
    KParams kp{a.eps2, a.alpha, 1.0f};
    float logwbar = 0.f, r0 = 0.f;
    if constexpr (K == SBH_SMOOTHDIST) {
        const float wbar = tv.nagg[0].w / (float)tv.n_points;
        kp.wscale = 1.0f / wbar;
        logwbar = logf(wbar);
        r0 = smooth_shift<2>(tv, qx, qy, qz, a.alpha);
    }
    const uint32_t* __restrict__ rt = tv.btopo;
    const uint32_t n_a = valid ? rt[slot] : 0u;
    uint32_t begin_a = 0u;
    int32_t nint_a = 0;
    for (int c = 0; c < slot; ++c) {
        begin_a += rt[c];
        nint_a += ((int)rt[c] > tv.leaf_size && 1 < tv.max_level) ? 1 : 0;
    }
    const int32_t blk_a = (int32_t)rt[D3] + nint_a;
    const float4 agg_a = tv.bagg[slot];
    float4 dip_a = zero4;
    if (tv.bdip) dip_a = tv.bdip[slot];
    const float cv = n_a ? term<K>(agg_a, (K == SBH_WINDING) ? dip_a : zero4, qx, qy, qz, kp, r0) : 0.0f;
    const uint32_t stream = (uint32_t)(a.group == 1 ? j : j / a.group);
    float fa = 0.0f;
    u32x4 rnd = {0u, 0u, 0u, 0u};
    for (int s = 0; s < a.samples; ++s) {
        bool act = n_a > 0u;
        uint32_t nT = n_a, beginT = begin_a;
        int32_t blk = blk_a;
        int level = 1;
        float diamT = tv.diam0 * 0.5f;
        float4 aggT = agg_a;
        float dT = fsqrt(norm2(agg_a.x - qx, agg_a.y - qy, agg_a.z - qz));   // |com_T - q|, carried step to step
        float tT = cv, prr = 1.0f, psel = 1.0f, acc = 0.0f;
        int steps = 0, flag = 0;
        int32_t end_b = (int32_t)beginT, end_l = level;
        const uint32_t ctr1 = (uint32_t)(slot * a.samples + s);
        for (int k = 0;; ++k) {
            if (act && nT == 1u) {
                flag = 1;
                end_b = (int32_t)beginT;
                end_l = level;
                act = false;
            }
            if (__ballot(act) == 0ull) break;
            if (act && (k & 1) == 0) rnd = philox4x32_10(stream, ctr1, (uint32_t)(k >> 1), a.batch, a.key0, a.key1);
            const uint32_t xsel = (k & 1) ? rnd.z : rnd.x;
            const uint32_t xrr = (k & 1) ? rnd.w : rnd.y;
            const bool internal = act && (int)nT > tv.leaf_size && level < tv.max_level;
            const float4* __restrict__ ba = tv.bagg + (int64_t)blk * D3;
            const uint32_t* __restrict__ bt = tv.btopo + (int64_t)blk * TS;
            uint32_t cnt[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
            float tv8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            float sumc = 0.0f;
            if (internal) {
                // the child block: terms for the swap, scores for the proposal
                const float4* __restrict__ bd = tv.bdip + (int64_t)blk * D3;
#pragma unroll
                for (int c = 0; c < D3; ++c) {
                    cnt[c] = bt[c];
                    const float4 gd = (K == SBH_WINDING) ? bd[c] : zero4;
                    const float v = term<K>(ba[c], gd, qx, qy, qz, kp, r0);
                    tv8[c] = cnt[c] ? v : 0.0f;
                    sumc += tv8[c];
                }
                if constexpr (NET) score_features(ba, tv.bspr + (int64_t)blk * D3, cnt, qx, qy, qz, f);
            }
            float z[8];
            if constexpr (NET) {
                if (net) {
                    if (__ballot(internal) != 0ull) mlp_forward_wave(R, f, z, lane);
                } else {
#pragma unroll
                    for (int c = 0; c < 8; ++c) z[c] = 16.0f * f[c];
                }
            }
            if (!act) continue;
            float4 aggC;
            uint32_t nC = 1u, beginC;
            int32_t blkC = 0;
            int csel = 0;
            float qsel, tC = 0.0f;
            if (internal) {
                float qv[8];
                if constexpr (NET) learned_probs(z, cnt, nT, qv);
                else score_probs(ba, tv.bspr + (int64_t)blk * D3, cnt, nT, qx, qy, qz, qv);
                const float u_sel = (float)(xsel >> 8) * 5.9604644775390625e-8f;
                // first slot whose running sum exceeds u; rounding can leave the
                // total just below u, then the last non-empty slot is taken
                float cum = 0.0f;
                uint32_t pre = 0u, preC = 0u, preL = 0u, nL = 0u;
                int32_t ni = 0, niC = 0, niL = 0;
                int last = 0;
                float qL = 0.0f, tL = 0.0f;
                bool found = false;
                nC = 0u;
                qsel = 0.0f;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const bool ne = cnt[c] != 0u;
                    last = ne ? c : last;
                    preL = ne ? pre : preL;
                    niL = ne ? ni : niL;
                    nL = ne ? cnt[c] : nL;
                    qL = ne ? qv[c] : qL;
                    tL = ne ? tv8[c] : tL;
                    cum += qv[c];
                    const bool hit = !found && ne && u_sel < cum;
                    csel = hit ? c : csel;
                    preC = hit ? pre : preC;
                    niC = hit ? ni : niC;
                    nC = hit ? cnt[c] : nC;
                    qsel = hit ? qv[c] : qsel;
                    tC = hit ? tv8[c] : tC;
                    found = found || hit;
                    ni += ((int)cnt[c] > tv.leaf_size && level + 1 < tv.max_level) ? 1 : 0;
                    pre += cnt[c];
                }
                if (!found) {
                    csel = last;
                    preC = preL;
                    niC = niL;
                    nC = nL;
                    qsel = qL;
                    tC = tL;
                }
                aggC = ba[csel];
                beginC = beginT + preC;
                blkC = (int32_t)bt[D3] + niC;
            } else {
                const uint32_t r = __umulhi(xsel, nT);
                aggC = tv.pts[beginT + r];
                beginC = beginT + r;
                csel = (int)r;
                qsel = 1.0f / (float)nT;
            }
            float p, dC = 0.0f;
            if (a.rr_mode == 0) {
                const float cx = aggC.x - qx, cy = aggC.y - qy, cz = aggC.z - qz;
                dC = fsqrt(norm2(cx, cy, cz));
                p = fminf(1.0f, fmaxf(diamT, dT) * frcp(2.0f * dC));
            } else {
                p = a.rr_mode == 1 ? 1.0f : 0.5f;
            }
            const float u = (float)(xrr >> 8) * 5.9604644775390625e-8f;
            if (u >= p) {
                flag = 0;
                end_b = (int32_t)beginT;
                end_l = level;
                act = false;
                continue;
            }
            if (!internal) {   // leaf: its points are the virtual children
                for (uint32_t i = 0; i < nT; ++i) {
                    const float4 g = tv.pts[beginT + i];
                    const float4 gd = (K == SBH_WINDING) ? tv.pdip[beginT + i] : zero4;
                    sumc = term_acc<K>(g, gd, qx, qy, qz, kp, r0, sumc);
                }
            }
            prr *= p;
            acc += (sumc - tT) * frcp(psel * prr);
            psel *= qsel;
            ++steps;
            if (!internal) {
                flag = 2;
                end_b = (int32_t)beginC;
                end_l = level + 1;
                act = false;
                continue;
            }
            aggT = aggC;
            dT = dC;
            tT = tC;
            nT = nC;
            beginT = beginC;
            blk = blkC;
            ++level;
            diamT *= 0.5f;
        }
        if constexpr (TRACE) {
            if (valid)
                reinterpret_cast<int4*>(a.paths)[(j * D3 + slot) * (int64_t)a.samples + s] =
                    n_a ? make_int4(end_b, end_l, steps, flag) : make_int4(-1, 0, 0, 0);
        }
        fa += acc;
    }
    float val = n_a ? cv + fa / (float)a.samples : 0.0f;
#pragma unroll
    for (int o = 1; o < D3; o <<= 1) val += __shfl_xor(val, o);
    if (valid && slot == 0) out[j] = query_value<K>(val, r0, logwbar, a.alpha, qx, qy, qz);
}

// The same estimator with lane refill: a wavefront owns a pool of kLearnPool
// paths (Q queries x 8 subdomains x S samples); a lane whose path has ended
// takes the next one, handed out in lane order, so lanes do not idle while
// the wavefront's longest path finishes.  The network still runs once per
// step for all 64 lanes.  Every path's sum is stored at its own place in LDS,
// and each query adds CV_a + F_a / S over its subdomains in slot order at the
// end.  The step is the one above, operation for operation.
constexpr int kLearnPool = 256;

template <int K, bool TRACE, bool NET>
__global__ void __launch_bounds__(256) k_sbh_learned_pool(TreeView tv, const float* __restrict__ queries, int64_t nq,
                                                          LearnArgs a, float* __restrict__ out)
{
#pragma clang fp contract(off)
    constexpr int D3 = 8;
    constexpr int TS = topo_stride(D3);
    __shared__ float res[4][kLearnPool];
    __shared__ float cvs[4][kLearnPool];
    __shared__ uint32_t tab[4][D3][3];
    __shared__ float4 root_agg[D3];
    __shared__ float4 root_dip[K == SBH_WINDING ? D3 : 1];
    __shared__ float qpos[4][kLearnPool / D3 * 3];
    __shared__ float qr0[K == SBH_SMOOTHDIST ? 4 : 1][kLearnPool / D3];   // the queries' smooth-distance shifts
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    const int lane = threadIdx.x & 63;
    const int wv = threadIdx.x >> 6;
    const int S = a.samples;
    const int Q = kLearnPool / (D3 * S);   // the launcher keeps 8 S <= kLearnPool
    const int NP = Q * D3 * S;
    const int64_t q0 = ((int64_t)blockIdx.x * 4 + wv) * Q;
    for (int c = threadIdx.x; c < D3; c += 256) {   // before the block's waves part: all reach the barrier
        root_agg[c] = tv.bagg[c];
        if constexpr (K == SBH_WINDING) root_dip[c] = tv.bdip[c];
    }
    __syncthreads();
    if (q0 >= nq) return;
    MlpRegs R;
    bool net = NET;
    if constexpr (NET) {
        // parameters that are not all finite are ignored (the zero network: the score proposal)
        bool bad = false;
        for (int i = lane; i < kMlpParams; i += 64) bad |= !__builtin_isfinite(a.prm[i]);
        net = __ballot(bad) == 0ull;
        mlp_load_regs(R, a.prm, lane);
    }
    KParams kp{a.eps2, a.alpha, 1.0f};
    float logwbar = 0.f;
    if constexpr (K == SBH_SMOOTHDIST) {
        const float wbar = tv.nagg[0].w / (float)tv.n_points;
        kp.wscale = 1.0f / wbar;
        logwbar = logf(wbar);
    }
    {   // the root block's subdomains and the wavefront's queries, once per wavefront
        const uint32_t* __restrict__ rt = tv.btopo;
        const int32_t base = (int32_t)rt[D3];
        uint32_t begin = 0u;
        int32_t nint = 0;
        for (int c = 0; c < D3; ++c) {
            const uint32_t n = rt[c];
            if (lane == 0) {
                tab[wv][c][0] = n;
                tab[wv][c][1] = begin;
                tab[wv][c][2] = (uint32_t)(base + nint);
            }
            begin += n;
            nint += ((int)n > tv.leaf_size && 1 < tv.max_level) ? 1 : 0;
        }
        for (int i = lane; i < 3 * Q; i += 64) qpos[wv][i] = q0 * 3 + i < 3 * nq ? queries[3 * q0 + i] : 0.0f;
        if constexpr (K == SBH_SMOOTHDIST) {
            if (lane < Q) {
                const int64_t jq = q0 + lane;
                qr0[wv][lane] = jq < nq ? smooth_shift<2>(tv, queries[3 * jq], queries[3 * jq + 1], queries[3 * jq + 2],
                                                          a.alpha)
                                        : 0.0f;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    int p = lane, slot = 0, smp = 0, k = 0, level = 1, steps = 0, flag = 0;
    int64_t j = 0;
    float qx = 0.f, qy = 0.f, qz = 0.f, r0 = 0.f;
    uint32_t nT = 0u, beginT = 0u, stream = 0u, ctr1 = 0u;
    int32_t blk = 0, end_b = 0, end_l = 1;
    float diamT = 0.f, dT = 0.f, tT = 0.f, prr = 1.f, psel = 1.f, acc = 0.f;
    u32x4 rnd = {0u, 0u, 0u, 0u};
    bool open = false;   // a path with points is being walked
    auto start = [&](int np) {
        p = np;
        open = false;
        if (p >= NP) {
            p = -1;
            return;
        }
        const int qi = p / (D3 * S), rem = p % (D3 * S);
        slot = rem / S;
        smp = rem % S;
        j = q0 + qi;
        acc = 0.0f;
        if (j >= nq) return;   // past the end of the query set: an empty path
        qx = qpos[wv][3 * qi];
        qy = qpos[wv][3 * qi + 1];
        qz = qpos[wv][3 * qi + 2];
        if constexpr (K == SBH_SMOOTHDIST) r0 = qr0[wv][qi];
        const uint32_t n_a = tab[wv][slot][0];
        if (n_a == 0u) {   // empty subdomain
            if constexpr (TRACE) reinterpret_cast<int4*>(a.paths)[(j * D3 + slot) * (int64_t)S + smp] = make_int4(-1, 0, 0, 0);
            return;
        }
        const float4 agg_a = root_agg[slot];
        const float cv = term<K>(agg_a, (K == SBH_WINDING) ? root_dip[slot] : zero4, qx, qy, qz, kp, r0);
        if (smp == 0) cvs[wv][p / S] = cv;
        nT = n_a;
        beginT = tab[wv][slot][1];
        blk = (int32_t)tab[wv][slot][2];
        level = 1;
        diamT = tv.diam0 * 0.5f;
        dT = fsqrt(norm2(agg_a.x - qx, agg_a.y - qy, agg_a.z - qz));
        tT = cv;
        prr = 1.0f;
        psel = 1.0f;
        steps = 0;
        flag = 0;
        k = 0;
        stream = (uint32_t)(a.group == 1 ? j : j / a.group);
        ctr1 = (uint32_t)(slot * S + smp);
        end_b = (int32_t)beginT;
        end_l = level;
        open = true;
    };
    start(lane);
    int next = 64;   // the next path of the pool to hand out
    while (__ballot(p >= 0) != 0ull) {
        bool done = p >= 0 && !open;   // an empty path ends at once
        bool internal = false;
        uint32_t xsel = 0u, xrr = 0u;
        const float4* __restrict__ ba = tv.bagg + (int64_t)blk * D3;
        const uint32_t* __restrict__ bt = tv.btopo + (int64_t)blk * TS;
        uint32_t cnt[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        float tv8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float f[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float sumc = 0.0f;
        if (open) {
            if (nT == 1u) {
                flag = 1;
                end_b = (int32_t)beginT;
                end_l = level;
                done = true;
            } else {
                if ((k & 1) == 0) rnd = philox4x32_10(stream, ctr1, (uint32_t)(k >> 1), a.batch, a.key0, a.key1);
                xsel = (k & 1) ? rnd.z : rnd.x;
                xrr = (k & 1) ? rnd.w : rnd.y;
                internal = (int)nT > tv.leaf_size && level < tv.max_level;
                if (internal) {
                    // the child block: terms for the swap, scores for the proposal
                    const float4* __restrict__ bd = tv.bdip + (int64_t)blk * D3;
#pragma unroll
                    for (int c = 0; c < D3; ++c) {
                        cnt[c] = bt[c];
                        const float4 gd = (K == SBH_WINDING) ? bd[c] : zero4;
                        const float v = term<K>(ba[c], gd, qx, qy, qz, kp, r0);
                        tv8[c] = cnt[c] ? v : 0.0f;
                        sumc += tv8[c];
                    }
                    if constexpr (NET) score_features(ba, tv.bspr + (int64_t)blk * D3, cnt, qx, qy, qz, f);
                }
            }
        }
        float z[8];
        if constexpr (NET) {
            if (net) {
                if (__ballot(internal) != 0ull) mlp_forward_wave(R, f, z, lane);
            } else {
#pragma unroll
                for (int c = 0; c < 8; ++c) z[c] = 16.0f * f[c];
            }
        }
        if (open && !done) {
            float4 aggC;
            uint32_t nC = 1u, beginC;
            int32_t blkC = 0;
            int csel = 0;
            float qsel, tC = 0.0f;
            if (internal) {
                float qv[8];
                if constexpr (NET) learned_probs(z, cnt, nT, qv);
                else score_probs(ba, tv.bspr + (int64_t)blk * D3, cnt, nT, qx, qy, qz, qv);
                const float u_sel = (float)(xsel >> 8) * 5.9604644775390625e-8f;
                // first slot whose running sum exceeds u; rounding can leave the
                // total just below u, then the last non-empty slot is taken
                float cum = 0.0f;
                uint32_t pre = 0u, preC = 0u, preL = 0u, nL = 0u;
                int32_t ni = 0, niC = 0, niL = 0;
                int last = 0;
                float qL = 0.0f, tL = 0.0f;
                bool found = false;
                nC = 0u;
                qsel = 0.0f;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const bool ne = cnt[c] != 0u;
                    last = ne ? c : last;
                    preL = ne ? pre : preL;
                    niL = ne ? ni : niL;
                    nL = ne ? cnt[c] : nL;
                    qL = ne ? qv[c] : qL;
                    tL = ne ? tv8[c] : tL;
                    cum += qv[c];
                    const bool hit = !found && ne && u_sel < cum;
                    csel = hit ? c : csel;
                    preC = hit ? pre : preC;
                    niC = hit ? ni : niC;
                    nC = hit ? cnt[c] : nC;
                    qsel = hit ? qv[c] : qsel;
                    tC = hit ? tv8[c] : tC;
                    found = found || hit;
                    ni += ((int)cnt[c] > tv.leaf_size && level + 1 < tv.max_level) ? 1 : 0;
                    pre += cnt[c];
                }
                if (!found) {
                    csel = last;
                    preC = preL;
                    niC = niL;
                    nC = nL;
                    qsel = qL;
                    tC = tL;
                }
                aggC = ba[csel];
                beginC = beginT + preC;
                blkC = (int32_t)bt[D3] + niC;
            } else {
                const uint32_t r = __umulhi(xsel, nT);
                aggC = tv.pts[beginT + r];
                beginC = beginT + r;
                qsel = 1.0f / (float)nT;
            }
            float pr, dC = 0.0f;
            if (a.rr_mode == 0) {
                const float cx = aggC.x - qx, cy = aggC.y - qy, cz = aggC.z - qz;
                dC = fsqrt(norm2(cx, cy, cz));
                pr = fminf(1.0f, fmaxf(diamT, dT) * frcp(2.0f * dC));
            } else {
                pr = a.rr_mode == 1 ? 1.0f : 0.5f;
            }
            const float u = (float)(xrr >> 8) * 5.9604644775390625e-8f;
            if (u >= pr) {
                flag = 0;
                end_b = (int32_t)beginT;
                end_l = level;
                done = true;
            } else {
                if (!internal) {   // leaf: its points are the virtual children
                    for (uint32_t i = 0; i < nT; ++i) {
                        const float4 g = tv.pts[beginT + i];
                        const float4 gd = (K == SBH_WINDING) ? tv.pdip[beginT + i] : zero4;
                        sumc = term_acc<K>(g, gd, qx, qy, qz, kp, r0, sumc);
                    }
                }
                prr *= pr;
                acc += (sumc - tT) * frcp(psel * prr);
                psel *= qsel;
                ++steps;
                if (!internal) {
                    flag = 2;
                    end_b = (int32_t)beginC;
                    end_l = level + 1;
                    done = true;
                } else {
                    dT = dC;
                    tT = tC;
                    nT = nC;
                    beginT = beginC;
                    blk = blkC;
                    ++level;
                    diamT *= 0.5f;
                    ++k;
                }
            }
        }
        if (done && open) {
            if constexpr (TRACE) reinterpret_cast<int4*>(a.paths)[(j * D3 + slot) * (int64_t)S + smp] = make_int4(end_b, end_l, steps, flag);
        }
        if (done) res[wv][p] = acc;
        // hand the next paths of the pool to the lanes that finished, in lane order
        const uint64_t fin = __ballot(done);
        if (fin != 0ull) {
            if (done) start(next + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(fin >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)fin, 0u)));
            next += __popcll(fin);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // per query: the subdomain totals CV_a + F_a / S in slot order
    const int64_t jq = q0 + lane;
    if (lane < Q && jq < nq) {
        float val = 0.0f;
        for (int c = 0; c < D3; ++c) {
            if (tab[wv][c][0] == 0u) continue;
            float fa = 0.0f;
            for (int t = 0; t < S; ++t) fa += res[wv][(lane * D3 + c) * S + t];
            val += cvs[wv][lane * D3 + c] + fa / (float)S;
        }
        const float rq = (K == SBH_SMOOTHDIST) ? qr0[wv][lane] : 0.0f;
        out[jq] = query_value<K>(val, rq, logwbar, a.alpha, queries[3 * jq], queries[3 * jq + 1], queries[3 * jq + 2]);
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_mlp_forward(const float* prm, const float* x, int64_t n, float* z, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_mlp_forward<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(prm, x, n, z);
    return hipGetLastError();
}

size_t mlp_partial_floats(int64_t rows) { return (size_t)((rows + 63) / 64) * kGradStride; }

// the partial gradients of the rows' groups of 64; returns their number
static int launch_mlp_partial(const float* prm, const float* X, const float* Tg, const float* Cn, int64_t n,
                              int64_t row_begin, int64_t rows, float* partial, hipStream_t s)
{
    constexpr int64_t kRows = (int64_t)1 << 28;   // (four work-items a row, of 2^32 - 1 that a launch holds)
    for (int64_t r0 = 0; r0 < rows; r0 += kRows) {
        const int64_t m = std::min(rows - r0, kRows);
        k_mlp_grad<<<(unsigned)((m + 63) / 64), 256, 0, s>>>(prm, X, Tg, Cn, n, row_begin + r0, m,
                                                             partial + r0 / 64 * kGradStride);
    }
    return (int)((rows + 63) / 64);
}

hipError_t launch_mlp_grad(const float* prm, const float* X, const float* Tg, const float* Cn, int64_t n,
                           int64_t row_begin, int64_t rows, float* partial, float* grad, hipStream_t s)
{
    const int nb = launch_mlp_partial(prm, X, Tg, Cn, n, row_begin, rows, partial, s);
    k_mlp_reduce<<<(1610 + 63) / 64, 64 * kReduceParts, 0, s>>>(partial, nb, grad);
    return hipGetLastError();
}

hipError_t launch_mlp_step(float* prm, float* state, const float* X, const float* Tg, const float* Cn, int64_t n,
                           int64_t row_begin, int64_t rows, float* partial, float lr, int step, float* loss_out,
                           hipStream_t s)
{
    const int nb = launch_mlp_partial(prm, X, Tg, Cn, n, row_begin, rows, partial, s);
    const float bc1 = 1.0f - powf(0.9f, (float)(step + 1));
    const float bc2 = 1.0f - powf(0.999f, (float)(step + 1));
    k_mlp_step<<<(1610 + 63) / 64, 64 * kReduceParts, 0, s>>>(partial, nb, prm, state, lr, bc1, bc2, loss_out);
    return hipGetLastError();
}

// Wavefronts of a path's workgroup: eight where paths are few and their children large, fewer where a path has
// little to share and its workgroup's barriers are what it waits for. us with eight / four / two, winding: 16
// queries on 2^20 sources, all levels 87 / 109 / 175; 512 on 2^20 711 / 692 / 747, on 200,000 239 / 200 / 198, on
// 20,000 116 / 84 / 70; 2,000 on 300, the first level 108 / 72 / 53 (a workgroup of four per row before: 52); 100 on
// 20,000 45 / 38 / 41, on 2^20 207 / 206 / 228.
template <int K, bool SOFT>
static void launch_mlp_targets(const TreeView& tv, unsigned paths, const float* q, int lmax, const int4* l, double eps2,
                               double alpha, float* t, hipStream_t s)
{
    const bool small = tv.n_points < (1 << 17);
    if (paths >= 4096 && small) k_mlp_targets<K, SOFT, 2><<<paths, 64 * 2, 0, s>>>(tv, q, lmax, l, eps2, alpha, t);
    else if (paths >= 4096 || (paths >= 512 && small)) k_mlp_targets<K, SOFT, 4><<<paths, 64 * 4, 0, s>>>(tv, q, lmax, l, eps2, alpha, t);
    else k_mlp_targets<K, SOFT, 8><<<paths, 64 * 8, 0, s>>>(tv, q, lmax, l, eps2, alpha, t);
}

hipError_t launch_mlp_pairs(const sbh_tree_impl* t, const float* queries, int64_t nq, int lmax, uint64_t seed,
                            int kernel, float eps, float alpha, float* X, float* Tg, float* Cn, int4* loc,
                            hipStream_t s)
{
    const TreeView tv = make_view(t);
    k_mlp_pairs<<<(unsigned)((nq * 8 + 127) / 128), 128, 0, s>>>(tv, queries, nq, lmax, (uint32_t)seed,
                                                                   (uint32_t)(seed >> 32), X, Cn, loc);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // (lmax <= the tree's max_level <= kTgMaxRows; a launch holds at most 2^32 - 1 work-items along a dimension)
    const double eps2 = (double)eps * (double)eps;
    constexpr int64_t kPaths = (int64_t)1 << 22;
    for (int64_t p0 = 0; p0 < nq * 8; p0 += kPaths) {
        const unsigned paths = (unsigned)std::min<int64_t>(nq * 8 - p0, kPaths);
        const float* q = queries + 3 * (p0 / 8);
        const int4* l = loc + p0 * lmax;
        float* t = Tg + 8 * p0 * lmax;
        if (kernel == SBH_POTENTIAL && eps2 > 0.0) launch_mlp_targets<SBH_POTENTIAL, true>(tv, paths, q, lmax, l, eps2, alpha, t, s);
        else if (kernel == SBH_POTENTIAL) launch_mlp_targets<SBH_POTENTIAL, false>(tv, paths, q, lmax, l, eps2, alpha, t, s);
        else if (kernel == SBH_WINDING) launch_mlp_targets<SBH_WINDING, false>(tv, paths, q, lmax, l, eps2, alpha, t, s);
        else launch_mlp_targets<SBH_SMOOTHDIST, false>(tv, paths, q, lmax, l, eps2, alpha, t, s);
    }
    return hipGetLastError();
}

}  // namespace sbh

namespace sbh {
hipError_t launch_sbh_learned(const sbh_tree_impl* t, const float* queries, int64_t nq, const EvalLaunch& e,
                              const float* prm, float* out, hipStream_t s)
{
    const TreeView tv = make_view(t);
    LearnArgs a{e.samples, e.group, e.rr_mode, e.batch, (uint32_t)e.seed, (uint32_t)(e.seed >> 32),
                e.eps * e.eps, e.alpha, e.paths, prm};
    // lane refill from a pool of paths per wavefront while 8 S <= kLearnPool (one path per lane beyond)
    const bool pool = 8 * (int64_t)e.samples <= kLearnPool;
    const int64_t qpw = pool ? kLearnPool / (8 * e.samples) : 8;
    const int64_t waves = (nq + qpw - 1) / qpw;
    const unsigned blocks = (unsigned)((waves + 3) / 4);
#define SBH_LAUNCH_L(KK, NN)                                                                               \
    do {                                                                                                   \
        if (pool) {                                                                                        \
            if (e.paths) k_sbh_learned_pool<KK, true, NN><<<blocks, 256, 0, s>>>(tv, queries, nq, a, out);   \
            else k_sbh_learned_pool<KK, false, NN><<<blocks, 256, 0, s>>>(tv, queries, nq, a, out);          \
        } else {                                                                                           \
            if (e.paths) k_sbh_learned<KK, true, NN><<<blocks, 256, 0, s>>>(tv, queries, nq, a, out);        \
            else k_sbh_learned<KK, false, NN><<<blocks, 256, 0, s>>>(tv, queries, nq, a, out);               \
        }                                                                                                  \
    } while (0)
#define SBH_LAUNCH_K(NN)                                        \
    do {                                                        \
        if (e.kernel == SBH_POTENTIAL) SBH_LAUNCH_L(SBH_POTENTIAL, NN);    \
        else if (e.kernel == SBH_WINDING) SBH_LAUNCH_L(SBH_WINDING, NN);   \
        else SBH_LAUNCH_L(SBH_SMOOTHDIST, NN);                  \
    } while (0)
    if (prm) SBH_LAUNCH_K(true);
    else SBH_LAUNCH_K(false);
#undef SBH_LAUNCH_K
#undef SBH_LAUNCH_L
    return hipGetLastError();
}
}  // namespace sbh
