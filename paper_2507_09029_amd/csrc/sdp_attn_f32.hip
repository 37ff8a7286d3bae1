// fp32 causal attention core (forward, dQ, dK/dV) for the head-masked attention block: fp32 storage, fp32 matrix
// instructions (v_mfma_f32_16x16x4_f32) and fp32 softmax arithmetic, any head width up to 128 (parity to 1e-5).  Same
// interface and the same saved statistics as the bf16 core: base-2 log-sum-exp of the scaled logits,
// delta = sum_h dO[t][h] O[t][h].  Nothing of size S x S is stored.
//
// A workgroup takes 16 rows (queries, or keys in the dK/dV kernel) of one (sequence, head); its 4 waves share out the
// other axis in tiles of 16 and their partial results meet in LDS, in wave order.  fp32 sequences are short (tests and
// reference runs), so the chain of tiles per wave and the number of workgroups decide, not the traffic: 16 rows and a
// fourfold split keep both small.
//
// Registers only.  The MFMA computes D[m][n] += sum_k A[m][k] B[k][n]: lane L supplies A[L % 16][k] and B[k][L % 16] of
// depth slot k = L / 16 and holds D[4 (L / 16) + r][L % 16].  A depth slot may stand for any index as long as A and B
// agree, which gives every operand of the core from plain global loads and every second product's B operand (P, dZ) from
// the accumulators of the first:
//   rows along the depth (logits, dP): slot j of a 16-deep group = columns 4 (L / 16) + j: one 16-byte load per group
//   rows as the depth (O, dQ, dK, dV): slot j = row 4 (L / 16) + j, the lane's own accumulator element j; the other
//   operand's 16-column fragment i takes column NF (L % 16) + i (NF = width / 16), so a lane loads NF consecutive
//   columns of a row and later stores NF consecutive ones
// One wave per (row, head) with scalar dot products, as this core was first written, took 555 / 563 / 590 us (forward,
// dQ, dK/dV) for 2 x 256 tokens and 8 heads of 64.  Rows whose result is not finite are still computed that way (sdp_attn_rows.h).
#include "sdp_attn_rows.h"

#include <cmath>

namespace sdp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

struct Args {
    const float* qkv; // [T][ldq]: Q | K | V, head i at columns i * hd of each part
    int64_t ldq;
    const float* o;   // [T][ldo]
    float* o_out;
    const float* dO;
    int64_t ldo;
    float* lse;   // [Bt][n][S]
    float* delta; // [Bt][n][S]
    float* dqkv;
    int S, n, hd;
    float scale2; // log2(e) / sqrt(hd)
    float scale;  // 1 / sqrt(hd)
};

constexpr int NW = 4; // waves per workgroup

// One head's width as the kernels see it: HW columns, of which hd exist (the rest read as zero and are not stored).
// VEC: hd and the row strides are multiples of 4 and the bases 16-byte aligned.
template <int HW, bool VEC>
struct Head {
    static constexpr int NF = HW / 16;
    static constexpr int PIECE = NF % 4 == 0 ? 4 : 2; // floats per load of a row's NF columns

    // depth along the row: element j of x[t] = column 16 t + 4 g + j
    static __device__ void row(const float* p, int hd, int g, f32x4 (&x)[NF]) {
#pragma unroll
        for (int t = 0; t < NF; ++t) {
            const int c = 16 * t + 4 * g;
            if (VEC) {
                const f32x4 v = *(const f32x4*)(p + (c < hd ? c : 0));
                x[t] = c < hd ? v : f32x4{0.f, 0.f, 0.f, 0.f};
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = p[c + j < hd ? c + j : 0];
                    x[t][j] = c + j < hd ? v : 0.f;
                }
            }
        }
    }
    // NF consecutive columns of a row: x[i] = column NF l + i
    static __device__ void cols(const float* p, int hd, int l, float (&x)[NF]) {
        if (VEC) {
#pragma unroll
            for (int i = 0; i < NF; i += PIECE) {
                const int c = NF * l + i;
                if (PIECE == 4) {
                    const f32x4 v = *(const f32x4*)(p + (c < hd ? c : 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[i + e] = c < hd ? v[e] : 0.f;
                } else {
                    const f32x2 v = *(const f32x2*)(p + (c < hd ? c : 0));
                    x[i] = c < hd ? v[0] : 0.f;
                    x[i + 1] = c < hd ? v[1] : 0.f;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const int c = NF * l + i;
                const float v = p[c < hd ? c : 0];
                x[i] = c < hd ? v : 0.f;
            }
        }
    }
};

__device__ inline f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// D[row of a][row of b] = sum over the columns of a b
template <int NF>
__device__ inline f32x4 dot_tile(const f32x4 (&a)[NF], const f32x4 (&b)[NF]) {
    f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NF; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) d = mfma(a[t][j], b[t][j], d);
    return d;
}

// sum / maximum over the four lanes L % 16 = const (the four depth slots)
__device__ inline float sum_slots(float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}
__device__ inline float max_slots(float v) {
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}

// The waves' accumulators acc[i][r] = X[column NF (4 g + r) + i][row l] -> LDS [wave][row][HW + 4], then for every row
// (tid / 16) the thread's NF columns NF (tid % 16) .. summed in wave order with weights w[wave]
template <int HW>
struct Merge {
    static constexpr int NF = HW / 16, RS = HW + 4;
    static __device__ void put(float* lds, const f32x4 (&acc)[NF], int wave, int l, int g) {
        float* p = lds + (wave * 16 + l) * RS;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < NF; ++i) p[NF * (4 * g + r) + i] = acc[i][r];
    }
    static __device__ void get(const float* lds, int row, int piece, const float (&w)[NW], float (&x)[NF]) {
#pragma unroll
        for (int i = 0; i < NF; ++i) x[i] = 0.f;
#pragma unroll
        for (int k = 0; k < NW; ++k)
#pragma unroll
            for (int i = 0; i < NF; ++i) x[i] += w[k] * lds[(k * 16 + row) * RS + NF * piece + i];
    }
};

template <int NF>
__device__ inline void store_cols(float* p, int hd, int piece, const float (&x)[NF]) {
#pragma unroll
    for (int i = 0; i < NF; ++i)
        if (NF * piece + i < hd) p[NF * piece + i] = x[i];
}

// 0 when every x is finite, else NaN
template <int N>
__device__ inline float finite_check(const float (&x)[N]) {
    float c = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) c += x[i] * 0.f;
    return c;
}
// Of the four result rows a wave holds (16 lanes each): bit 16 r set when row r has to be computed again.  bad: this lane holds
// a value that is not finite, of a row that exists.
__device__ inline uint64_t rows_again(bool bad) {
    uint64_t m = __builtin_amdgcn_ballot_w64(bad);
    m |= m >> 8, m |= m >> 4, m |= m >> 2, m |= m >> 1;
    return m & 0x0001000100010001ull;
}

// Long items first: blocks of rows along the grid's slowest axis (heads, sequences, blocks), so that no axis is a product of
// sizes.  A grid has 65535 on its slower axes: with more blocks than that (16 rows each) they take the first one instead.
constexpr int kSlowAxis = 65535;
struct Item {
    int row0, head, b;
};
__device__ inline Item item_of(int nblocks, bool first_is_long) {
    const bool slow = nblocks <= kSlowAxis;
    const int blk = slow ? blockIdx.z : blockIdx.x;
    return {16 * (first_is_long ? blk : nblocks - 1 - blk), (int)(slow ? blockIdx.x : blockIdx.y), (int)(slow ? blockIdx.y : blockIdx.z)};
}
inline dim3 item_grid(int nblocks, int n, int Bt) { return nblocks <= kSlowAxis ? dim3(n, Bt, nblocks) : dim3(nblocks, n, Bt); }

template <int HW>
constexpr int merge_floats() { return NW * 16 * (HW + 4); }

// forward: O[q] = sum_{k <= q} softmax(z[q][.])[k] V[k]
template <int HW, bool VEC>
__global__ __launch_bounds__(64 * NW) void attn_f32_fwd_kernel(Args a, int nblocks) {
    typedef Head<HW, VEC> H;
    constexpr int NF = H::NF;
    __shared__ __attribute__((aligned(16))) float sO[NW * 16 * (HW + 4)];
    __shared__ float sM[NW][16], sL[NW][16];
    const int tid = threadIdx.x, lane = tid & 63, l = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Item it = item_of(nblocks, false);
    const int hd = a.hd, last = a.S - 1;
    const float* Q0 = a.qkv + (int64_t)it.b * a.S * a.ldq + it.head * hd;
    const float* K0 = Q0 + a.n * hd;
    const float* V0 = K0 + a.n * hd;
    const int q = it.row0 + l;
    f32x4 qf[NF];
    H::row(Q0 + (int64_t)(q < last ? q : last) * a.ldq, hd, g, qf);

    f32x4 acc[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, den = 0.f;
    const int ntiles = it.row0 / 16 + 1; // key tiles up to the diagonal
    f32x4 kf[NF];
    auto fetch_k = [&](int t) {
        const int k = 16 * t + l;
        H::row(K0 + (int64_t)(k < last ? k : last) * a.ldq, hd, g, kf);
    };
    if (wave < ntiles) fetch_k(wave);
    for (int t = wave; t < ntiles; t += NW) {
        float v[4][NF];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 16 * t + 4 * g + j;
            H::cols(V0 + (int64_t)(k < last ? k : last) * a.ldq, hd, l, v[j]);
        }
        f32x4 s = dot_tile<NF>(kf, qf); // s[r]: key 16 t + 4 g + r, query l
        if (t + NW < ntiles) fetch_k(t + NW);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = 16 * t + 4 * g + r;
            s[r] = k <= q && k <= last ? s[r] * a.scale2 : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        const float m_new = fmaxf(m, max_slots(mx));
        const float base = m_new == -INFINITY ? 0.f : m_new; // no key of the tile counts for this query yet
        const float alpha = exp2f(m - base);
        m = m_new;
        float p[4], ps = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = exp2f(s[r] - base), ps += p[r];
        den = den * alpha + ps;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            acc[i] *= alpha;
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i] = mfma(v[j][i], p[j], acc[i]);
        }
    }
    den = sum_slots(den);
    Merge<HW>::put(sO, acc, wave, l, g);
    if (g == 0) sM[wave][l] = m, sL[wave][l] = den;
    __syncthreads();
    const int row = tid >> 4, piece = tid & 15;
    float w[NW], top = -INFINITY, total = 0.f;
#pragma unroll
    for (int k = 0; k < NW; ++k) top = fmaxf(top, sM[k][row]); // finite: wave 0 holds key 0 of every query
#pragma unroll
    for (int k = 0; k < NW; ++k) w[k] = exp2f(sM[k][row] - top), total += w[k] * sL[k][row];
    float x[NF];
    Merge<HW>::get(sO, row, piece, w, x);
    const int qr = it.row0 + row;
#pragma unroll
    for (int i = 0; i < NF; ++i) x[i] /= total;
    float* const out = a.o_out + (int64_t)it.b * a.S * a.ldo + it.head * hd;
    float* const lse = a.lse + ((int64_t)it.b * a.n + it.head) * a.S;
    const uint64_t again = rows_again(qr <= last && finite_check(x) != 0.f);
    if (qr <= last && !(again >> (lane & 48) & 1)) {
        store_cols<NF>(out + qr * a.ldo, hd, piece, x);
        if (piece == 0) lse[qr] = top + log2f(total);
    }
    if (again == 0) return;
    const AttnRows<float> ar{Q0, K0, V0, a.ldq, nullptr, 0, a.S, hd, a.scale, a.scale2};
    for (int r = 0; r < 4; ++r) {
        const int qa = it.row0 + 4 * wave + r;
        if (again >> (16 * r) & 1) attn_row_fwd(ar, qa, lane, out + qa * a.ldo, lse + qa);
    }
}

// backward, dQ and delta: dQ[q] = scale sum_{k <= q} dZ[q][k] K[k], dZ = P (dP - delta), dP[q][k] = dO[q] . V[k]
template <int HW, bool VEC, bool STORE_DELTA>
__device__ inline void dq_block(const Args& a, const Item it, float* sX) {
    typedef Head<HW, VEC> H;
    constexpr int NF = H::NF;
    const int tid = threadIdx.x, lane = tid & 63, l = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hd = a.hd, last = a.S - 1;
    const float* Q0 = a.qkv + (int64_t)it.b * a.S * a.ldq + it.head * hd;
    const float* K0 = Q0 + a.n * hd;
    const float* V0 = K0 + a.n * hd;
    const int q = it.row0 + l, qc = q < last ? q : last;
    const int64_t orow = ((int64_t)it.b * a.S + qc) * a.ldo + it.head * hd;
    f32x4 qf[NF], of[NF];
    H::row(a.dO + orow, hd, g, of);
    H::row(a.o + orow, hd, g, qf);
    float d = 0.f;
#pragma unroll
    for (int t = 0; t < NF; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) d = __builtin_fmaf(of[t][j], qf[t][j], d);
    d = sum_slots(d);
    H::row(Q0 + (int64_t)qc * a.ldq, hd, g, qf);
    const int64_t st = ((int64_t)it.b * a.n + it.head) * a.S;
    if (STORE_DELTA && wave == 0 && g == 0 && q <= last) a.delta[st + q] = d;
    const float L2 = a.lse[st + qc];

    f32x4 acc[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ntiles = it.row0 / 16 + 1;
    for (int t = wave; t < ntiles; t += NW) {
        f32x4 kf[NF], vf[NF];
        const int kr = 16 * t + l;
        const int64_t koff = (int64_t)(kr < last ? kr : last) * a.ldq;
        H::row(K0 + koff, hd, g, kf);
        H::row(V0 + koff, hd, g, vf);
        float kc[4][NF];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 16 * t + 4 * g + j;
            H::cols(K0 + (int64_t)(k < last ? k : last) * a.ldq, hd, l, kc[j]);
        }
        f32x4 s = dot_tile<NF>(kf, qf), dp = dot_tile<NF>(vf, of);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = 16 * t + 4 * g + r;
            s[r] = k <= q && k <= last ? exp2f(s[r] * a.scale2 - L2) * (dp[r] - d) : 0.f;
        }
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i] = mfma(kc[j][i], s[j], acc[i]);
    }
    Merge<HW>::put(sX, acc, wave, l, g);
    __syncthreads();
    const int row = tid >> 4, piece = tid & 15;
    const float w[NW] = {a.scale, a.scale, a.scale, a.scale};
    float x[NF];
    Merge<HW>::get(sX, row, piece, w, x);
    const int qr = it.row0 + row;
    float* const out = a.dqkv + (int64_t)it.b * a.S * a.ldq + it.head * hd;
    const uint64_t again = rows_again(qr <= last && finite_check(x) != 0.f);
    if (qr <= last && !(again >> (lane & 48) & 1)) store_cols<NF>(out + qr * a.ldq, hd, piece, x);
    if (again == 0) return;
    const AttnRows<float> ar{Q0, K0, V0, a.ldq, a.dO + (int64_t)it.b * a.S * a.ldo + it.head * hd, a.ldo, a.S, hd, a.scale, a.scale2};
    for (int r = 0; r < 4; ++r) {
        const int ra = 4 * wave + r, qa = it.row0 + ra; // lane ra holds that row's delta and log-sum-exp
        const float da = __shfl(d, ra, 64), la = __shfl(L2, ra, 64);
        if (again >> (16 * r) & 1) attn_row_dq(ar, qa, lane, la, da, out + qa * a.ldq);
    }
}

template <int HW, bool VEC>
__global__ __launch_bounds__(64 * NW) void attn_f32_dq_kernel(Args a, int nblocks) {
    __shared__ __attribute__((aligned(16))) float sX[merge_floats<HW>()];
    dq_block<HW, VEC, true>(a, item_of(nblocks, false), sX);
}

// backward, dK and dV of 16 keys: sums over the queries q >= k; reads delta (OWN_DELTA: computes it from dO's and O's rows)
template <int HW, bool VEC, bool OWN_DELTA>
__device__ inline void dkv_block(const Args& a, const Item it, float* sX) {
    typedef Head<HW, VEC> H;
    constexpr int NF = H::NF;
    const int tid = threadIdx.x, lane = tid & 63, l = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hd = a.hd, last = a.S - 1;
    const float* Q0 = a.qkv + (int64_t)it.b * a.S * a.ldq + it.head * hd;
    const float* K0 = Q0 + a.n * hd;
    const float* V0 = K0 + a.n * hd;
    const float* O0 = a.dO + (int64_t)it.b * a.S * a.ldo + it.head * hd;
    const float* X0 = OWN_DELTA ? a.o + (int64_t)it.b * a.S * a.ldo + it.head * hd : nullptr; // O
    const int64_t st = ((int64_t)it.b * a.n + it.head) * a.S;
    const int k = it.row0 + l, kc = k < last ? k : last;
    f32x4 kf[NF], vf[NF];
    H::row(K0 + (int64_t)kc * a.ldq, hd, g, kf);
    H::row(V0 + (int64_t)kc * a.ldq, hd, g, vf);
    f32x4 ak[NF], av[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) ak[i] = av[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int ntiles = (a.S + 15) / 16;
    for (int t = it.row0 / 16 + wave; t < ntiles; t += NW) {
        const int qr = 16 * t + l, qrc = qr < last ? qr : last;
        f32x4 qf[NF], of[NF];
        H::row(Q0 + (int64_t)qrc * a.ldq, hd, g, qf);
        H::row(O0 + (int64_t)qrc * a.ldo, hd, g, of);
        float L2[4], dl[4], qc[4][NF], oc[4][NF];
        float d = 0.f; // of query 16 t + l
        if constexpr (OWN_DELTA) {
            f32x4 xf[NF];
            H::row(X0 + (int64_t)qrc * a.ldo, hd, g, xf);
#pragma unroll
            for (int i = 0; i < NF; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) d = __builtin_fmaf(of[i][j], xf[i][j], d);
            d = sum_slots(d);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = 16 * t + 4 * g + j, c = q < last ? q : last;
            L2[j] = a.lse[st + c];
            if constexpr (OWN_DELTA) dl[j] = __shfl(d, 4 * g + j, 64);
            else dl[j] = a.delta[st + c];
            H::cols(Q0 + (int64_t)c * a.ldq, hd, l, qc[j]);
            H::cols(O0 + (int64_t)c * a.ldo, hd, l, oc[j]);
        }
        f32x4 s = dot_tile<NF>(qf, kf), dp = dot_tile<NF>(of, vf); // [query 16 t + 4 g + r][key l]
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int q = 16 * t + 4 * g + r;
            s[r] = k <= q && q <= last ? exp2f(s[r] * a.scale2 - L2[r]) : 0.f;
            dp[r] = s[r] * (dp[r] - dl[r]);
        }
#pragma unroll
        for (int i = 0; i < NF; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                av[i] = mfma(oc[j][i], s[j], av[i]);
                ak[i] = mfma(qc[j][i], dp[j], ak[i]);
            }
    }
    const int row = tid >> 4, piece = tid & 15, krow = it.row0 + row;
    float* out = a.dqkv + ((int64_t)it.b * a.S + (krow < last ? krow : last)) * a.ldq + it.head * hd;
    float x[NF];
    Merge<HW>::put(sX, ak, wave, l, g);
    __syncthreads();
    const float wk[NW] = {a.scale, a.scale, a.scale, a.scale}, wv[NW] = {1.f, 1.f, 1.f, 1.f};
    Merge<HW>::get(sX, row, piece, wk, x);
    float y[NF];
    __syncthreads();
    Merge<HW>::put(sX, av, wave, l, g);
    __syncthreads();
    Merge<HW>::get(sX, row, piece, wv, y);
    const uint64_t again = rows_again(krow <= last && finite_check(x) + finite_check(y) != 0.f);
    if (krow <= last && !(again >> (lane & 48) & 1)) {
        store_cols<NF>(out + a.n * hd, hd, piece, x);
        store_cols<NF>(out + 2 * a.n * hd, hd, piece, y);
    }
    if (again == 0) return;
    const AttnRows<float> ar{Q0, K0, V0, a.ldq, O0, a.ldo, a.S, hd, a.scale, a.scale2};
    for (int r = 0; r < 4; ++r) {
        const int ka = it.row0 + 4 * wave + r;
        float* o = a.dqkv + ((int64_t)it.b * a.S + ka) * a.ldq + it.head * hd;
        if (again >> (16 * r) & 1) attn_row_dkv<OWN_DELTA>(ar, ka, lane, a.lse + st, OWN_DELTA ? nullptr : a.delta + st, o + a.n * hd, o + 2 * a.n * hd, X0);
    }
}

template <int HW, bool VEC>
__global__ __launch_bounds__(64 * NW) void attn_f32_dkv_kernel(Args a, int nblocks) {
    __shared__ __attribute__((aligned(16))) float sX[merge_floats<HW>()];
    dkv_block<HW, VEC, false>(a, item_of(nblocks, true), sX); // the first key blocks meet the most queries
}

// dK, dV and dQ as one launch, while the blocks are few: the chain of a block and the gap between two launches bound these, not
// the matrix cores, and dK/dV does not wait for the delta of the other half.  Forward and backward of an attention, two launches / one:
// 1 x 64 tokens, 4 heads of 64 (16 blocks) 39.8 / 31.1 us, 1 x 200, 4 of 128 92 / 78, 2 x 200, 6 of 80 97 / 85, 2 x 256, 4 of 128 109 / 96,
// 2 x 256, 8 of 64 (256 blocks) 84.4 / 79.1, 2 x 256, 8 of 128 222 / 214, 2 x 256, 12 of 64 (384) 161 / 157; but 2 x 256, 16 of 64 (512)
// 200.5 / 199.7 and 4 x 256, 16 of 32 (1024) 134 / 137, 4 x 512, 8 of 128 (1024) 685 / 774: many blocks pay for the registers of both halves
// and for reading O again.
template <int HW, bool VEC>
__global__ __launch_bounds__(64 * NW) void attn_f32_bwd_kernel(Args a, int nblocks) {
    __shared__ __attribute__((aligned(16))) float sX[merge_floats<HW>()];
    const bool dkv = (int)blockIdx.x < a.n;
    Item it = item_of(nblocks, dkv);
    if (!dkv) it.head -= a.n;
    if (dkv) dkv_block<HW, VEC, true>(a, it, sX);
    else dq_block<HW, VEC, false>(a, it, sX);
}

Args make_args(const AttnCoreDesc& c) {
    Args a{};
    a.qkv = (const float*)c.qkv, a.ldq = c.ldq;
    a.o = (const float*)c.o, a.o_out = (float*)c.o_out, a.dO = (const float*)c.dO, a.ldo = c.ldo;
    a.lse = c.lse, a.delta = c.delta, a.dqkv = (float*)c.dqkv;
    a.S = c.S, a.n = c.n, a.hd = c.hd;
    a.scale = 1.f / sqrtf((float)c.hd), a.scale2 = a.scale * 1.44269504088896340736f;
    return a;
}

template <int HW, bool VEC>
int fwd_t(const AttnCoreDesc& c, int nblocks, hipStream_t s) {
    ProfileScope ps("attn_core_fwd", s);
    attn_f32_fwd_kernel<HW, VEC><<<item_grid(nblocks, c.n, c.Bt), 64 * NW, 0, s>>>(make_args(c), nblocks);
    return launch_status();
}
// both launches as one, see attn_f32_bwd_kernel; few enough blocks to lie along the grid's slowest axis
constexpr int kMergedBlocks = 384;
static_assert(kMergedBlocks <= kSlowAxis, "heads along the fastest axis");
bool merged_backward(const AttnCoreDesc& c, int nblocks) { return (int64_t)nblocks * c.n * c.Bt <= kMergedBlocks; }

template <int HW, bool VEC>
int bwd_t(const AttnCoreDesc& c, int nblocks, hipStream_t s) {
    const dim3 grid = item_grid(nblocks, c.n, c.Bt);
    if (merged_backward(c, nblocks)) {
        ProfileScope ps("attn_core_bwd", s);
        attn_f32_bwd_kernel<HW, VEC><<<item_grid(nblocks, 2 * c.n, c.Bt), 64 * NW, 0, s>>>(make_args(c), nblocks);
        return launch_status();
    }
    {
        ProfileScope ps("attn_core_bwd_dq", s);
        attn_f32_dq_kernel<HW, VEC><<<grid, 64 * NW, 0, s>>>(make_args(c), nblocks);
        const int rc = launch_status();
        if (rc != SDP_OK) return rc;
    }
    ProfileScope ps("attn_core_bwd_dkv", s); // reads the delta written by the dQ kernel
    attn_f32_dkv_kernel<HW, VEC><<<grid, 64 * NW, 0, s>>>(make_args(c), nblocks);
    return launch_status();
}

template <class F>
int by_width(const AttnCoreDesc& c, F f) {
    if (c.hd < 1 || c.hd > 128) return SDP_ERR_UNSUPPORTED;
    const int nblocks = (int)(((int64_t)c.S + 15) / 16);
    const bool vec = c.hd % 4 == 0 && c.ldq % 4 == 0 && c.ldo % 4 == 0 && aligned16(c.qkv) && (!c.o || aligned16(c.o)) &&
                     (!c.dO || aligned16(c.dO));
    return f(vec, nblocks);
}

} // namespace

int attn_f32_fwd(const AttnCoreDesc& c, hipStream_t s) {
    return by_width(c, [&](bool vec, int nb) {
        if (!vec) return c.hd <= 64 ? fwd_t<64, false>(c, nb, s) : fwd_t<128, false>(c, nb, s);
        if (c.hd <= 32) return fwd_t<32, true>(c, nb, s);
        if (c.hd <= 64) return fwd_t<64, true>(c, nb, s);
        return c.hd <= 96 ? fwd_t<96, true>(c, nb, s) : fwd_t<128, true>(c, nb, s);
    });
}
int attn_f32_bwd(const AttnCoreDesc& c, hipStream_t s) {
    return by_width(c, [&](bool vec, int nb) {
        if (!vec) return c.hd <= 64 ? bwd_t<64, false>(c, nb, s) : bwd_t<128, false>(c, nb, s);
        if (c.hd <= 32) return bwd_t<32, true>(c, nb, s);
        if (c.hd <= 64) return bwd_t<64, true>(c, nb, s);
        return c.hd <= 96 ? bwd_t<96, true>(c, nb, s) : bwd_t<128, true>(c, nb, s);
    });
}

} // namespace sdp
