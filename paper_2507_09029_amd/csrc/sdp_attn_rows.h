// Causal attention one row at a time, by one wave, in fp32 arithmetic on fp32 or bf16 tensors: the rows of an attention core's
// result in which a matrix tile has left something that is not finite.
//
// A tile multiplies masked pairs (key after query) by a probability of zero, and 0 x NaN or 0 x Inf is NaN: one bad token
// reaches up to a tile of rows that do not depend on it.  A product with an infinite operand split into two bf16 terms is NaN
// as well.  Both show as a result that is not finite, so the cores look at their results and compute such rows again here, where
// only the pairs with key <= query are ever read.  Results that are finite cost the check alone.
//
// The 64 lanes take 64 keys (or queries) for the dot products and then, key by key, the columns lane and lane + 64 of the sum.
#pragma once
#include "sdp_internal.h"
#include "sdp_swiglu.h"

namespace sdp {

// one (sequence, head): pointers at its first row and column, row strides in elements
template <typename T>
struct AttnRows {
    const T *Q, *K, *V;
    int64_t ldq;
    const T* dO; // backward
    int64_t ldo;
    int S, hd;
    float scale, scale2; // 1 / sqrt(head width), and that times log2(e)
};

__device__ inline float row_value(const float* p) { return *p; }
__device__ inline float row_value(const uint16_t* p) { return bf16_to_f32(*p); }
__device__ inline void set_row_value(float* p, float v) { *p = v; }
__device__ inline void set_row_value(uint16_t* p, float v) { *p = f32_to_bf16(v); }

template <typename T>
__device__ inline float row_dot(const T* a, const T* b, int hd) {
    float z = 0.f;
    for (int h = 0; h < hd; ++h) z = __builtin_fmaf(row_value(a + h), row_value(b + h), z);
    return z;
}
__device__ inline float row_wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// acc[c] += sum over j < n of (lane j's f) x[j ld + lane + 64 c]
template <typename T>
__device__ inline void row_accumulate(float f, const T* x, int64_t ld, int n, int hd, int lane, float (&acc)[2]) {
    for (int j = 0; j < n; ++j) {
        const float fj = __shfl(f, j, 64);
#pragma unroll
        for (int c = 0; c < 2; ++c)
            if (lane + 64 * c < hd) acc[c] = __builtin_fmaf(fj, row_value(x + j * ld + lane + 64 * c), acc[c]);
    }
}
template <typename T>
__device__ inline void row_store(T* out, const float (&acc)[2], int hd, int lane) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
        if (lane + 64 * c < hd) set_row_value(out + lane + 64 * c, acc[c]);
}

// O[q] = sum_{k <= q} softmax(z[q][.])[k] V[k], and the base-2 log-sum-exp of the scaled logits
template <typename T>
__device__ __forceinline__ void attn_row_fwd(const AttnRows<T>& a, int q, int lane, T* out, float* lse) {
    const T* Q = a.Q + q * a.ldq;
    float mx = -INFINITY;
    for (int k = lane; k <= q; k += 64) mx = fmaxf(mx, row_dot(Q, a.K + k * a.ldq, a.hd) * a.scale2);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    float acc[2] = {0.f, 0.f}, den = 0.f;
    for (int k0 = 0; k0 <= q; k0 += 64) {
        const int k = k0 + lane;
        const float p = k <= q ? exp2f(row_dot(Q, a.K + k * a.ldq, a.hd) * a.scale2 - mx) : 0.f;
        den += p;
        row_accumulate(p, a.V + k0 * a.ldq, a.ldq, q - k0 < 63 ? q - k0 + 1 : 64, a.hd, lane, acc);
    }
    den = row_wave_sum(den);
    acc[0] /= den, acc[1] /= den;
    row_store(out, acc, a.hd, lane);
    if (lane == 0) *lse = mx + log2f(den);
}

// dQ[q] = scale sum_{k <= q} dZ[q][k] K[k], dZ = P (dP - delta), dP[q][k] = dO[q] . V[k]
template <typename T>
__device__ __forceinline__ void attn_row_dq(const AttnRows<T>& a, int q, int lane, float lse, float delta, T* out) {
    const T *Q = a.Q + q * a.ldq, *dO = a.dO + q * a.ldo;
    float acc[2] = {0.f, 0.f};
    for (int k0 = 0; k0 <= q; k0 += 64) {
        const int k = k0 + lane;
        float dz = 0.f;
        if (k <= q) {
            const float p = exp2f(row_dot(Q, a.K + k * a.ldq, a.hd) * a.scale2 - lse);
            dz = p * (row_dot(dO, a.V + k * a.ldq, a.hd) - delta);
        }
        row_accumulate(dz, a.K + k0 * a.ldq, a.ldq, q - k0 < 63 ? q - k0 + 1 : 64, a.hd, lane, acc);
    }
    acc[0] *= a.scale, acc[1] *= a.scale;
    row_store(out, acc, a.hd, lane);
}

// dV[k] = sum_{q >= k} P[q][k] dO[q], dK[k] = scale sum_{q >= k} dZ[q][k] Q[q]; lse of the sequence's rows; delta of
// these or, OWN_DELTA, O's rows (strides of dO) to compute it from
template <bool OWN_DELTA, typename T>
__device__ __forceinline__ void attn_row_dkv(const AttnRows<T>& a, int k, int lane, const float* lse, const float* delta, T* dK, T* dV, const T* O) {
    const T *K = a.K + k * a.ldq, *V = a.V + k * a.ldq;
    float ak[2] = {0.f, 0.f}, av[2] = {0.f, 0.f};
    for (int q0 = k; q0 < a.S; q0 += 64) {
        const int q = q0 + lane, n = a.S - q0 < 64 ? a.S - q0 : 64;
        float p = 0.f, dz = 0.f;
        if (q < a.S) {
            p = exp2f(row_dot(a.Q + q * a.ldq, K, a.hd) * a.scale2 - lse[q]);
            dz = p * (row_dot(a.dO + q * a.ldo, V, a.hd) - (OWN_DELTA ? row_dot(a.dO + q * a.ldo, O + q * a.ldo, a.hd) : delta[q]));
        }
        row_accumulate(p, a.dO + q0 * a.ldo, a.ldo, n, a.hd, lane, av);
        row_accumulate(dz, a.Q + q0 * a.ldq, a.ldq, n, a.hd, lane, ak);
    }
    ak[0] *= a.scale, ak[1] *= a.scale;
    row_store(dK, ak, a.hd, lane);
    row_store(dV, av, a.hd, lane);
}

} // namespace sdp
