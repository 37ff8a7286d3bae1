// One worker's attention block under head-level masks (the paper's Sec. 4.1: the neuron-level variant of
// Sec. 3.2 masks attention heads on W_Q, W_K, W_V and W_O), forward masking (Sec. 3.1): the block is
// evaluated at the gated parameters, i.e. as the smaller dense block made of the worker's ph heads.  Under
// backward masking the block runs on all H heads without gather lists, and only the weight-gradient
// contraction is restricted to the held heads' rows (row gather on its left operand).
//
// With E = ph * hd, rows_qkv = the 3 E rows of [Wq; Wk; Wv] that belong to the held heads and rows_o the E
// rows of WoT (columns of W_O):
//   forward   qkv   : [Q | K | V] = X . Wqkv[rows_qkv]^T      (T x 3E, depth d; rows gathered in the load)
//             core  : O_h = softmax_causal(Q_h K_h^T / sqrt(hd)) V_h, per sequence and held head
//             out   : Y = O . WoT[rows_o]                     (T x d, depth E)
//   backward  dO = dY . WoT[rows_o]^T (T x E);  core backward -> dQ, dK, dV (T x 3E);
//             dWqkv[rows_qkv] = dQKV^T . X, dWoT[rows_o] = O^T . dY (depth T);  dX = dQKV . Wqkv[rows_qkv]
// The contractions are the ones of the MLP path (same kernels, other shapes).  The core is written here:
// causal attention on 32x32x16 bf16 MFMA tiles for heads of 64, 96 or 128 columns (wider and narrower ones take the next
// of these widths), with the running-maximum formulation of the softmax (logits in base 2), so that no T x T matrix is
// stored.  Heads of 65 .. 128 used to run the plain core: one sequence of 1500 tokens, 4 of 8 heads of 128, forward and
// backward of the block 20.0 ms then, 0.15 ms on the wide MFMA core.
//
// Accumulator convention.  v_mfma_f32_32x32x16 computes D[m][n] += sum_k A[m][k] B[k][n]; lane L supplies
// A[L % 32][8 (L / 32) + e] and B[8 (L / 32) + e][L % 32], e = 0..7, and holds D[8 q + 4 (L / 32) + r][L % 32]
// in element 4 q + r.  Every product below puts the index that owns per-row softmax statistics on n, so that
// a lane keeps one query (or one key) and its statistics are plain per-lane scalars.  The probabilities then
// feed the next product straight from the accumulator registers: elements 8 s .. 8 s + 7 of a 32-wide tile
// are, for this lane, the depth indices {16 s + 4 (L / 32) + r} and {16 s + 8 + 4 (L / 32) + r}, and the other
// operand is read from LDS in that same order with two transposing reads (ds_read_tr16_b64), which turn a
// row-major [depth][column] tile into the per-lane layout of an A operand.
#include "sdp_attn_rule.h"
#include "sdp_attn_rows.h"
#include "sdp_transpose.h"

#include <cmath>
#include <type_traits>

namespace sdp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

constexpr int HD = 64;              // narrowest width of the MFMA core
// Widths of the core: HW = 64, 96 or 128 columns per head.  An LDS tile row holds HW bf16 + 16 bytes: consecutive rows
// then start 4 (an odd multiple of 4) banks apart, so the 16 lanes that a ds_read_b128 serves together hit every bank once.
constexpr int row_bytes(int hw) { return hw * 2 + 16; }
constexpr float kSlack = 8.f;      // forward: how far a query's maximum may run ahead of its reference exponent
constexpr int NW = 4;               // waves per workgroup of the KW = 1 form

// A workgroup's waves share out the work in one of two ways (KW = waves along the walked axis):
//   KW = 1: four blocks of 32 rows (queries, or keys in the dK/dV kernel), every wave walks all tiles of the other axis.
//           The tiles are staged once for the workgroup.
//   KW = 4, 8: one block of 32 rows; wave w walks the 32-row tiles w, w + KW, ... of the other axis, which it stages for
//           itself (no barrier in the loop), and the partial results are added at the end through LDS.  Four times
//           the workgroups with a quarter (an eighth) of the chain each, for four times the reads of the other axis.
template <int KW>
struct Split {
    static_assert(KW == 1 || KW == 4 || KW == 8, "all waves on one axis");
    static constexpr int ROWS = KW == 1 ? 32 * NW : 32; // rows per workgroup
    static constexpr int THREADS = 64 * (KW == 1 ? NW : KW);
};

// Heads wider than 64 take the probabilities (and their gradients) into the second products as two bf16 terms, value =
// hi + lo, i.e. with 16 bits of mantissa: the plain core that served them held these in fp32.  Heads up to 64 take them
// as one bf16 term.
constexpr bool two_terms(int hw) { return hw > HD; }

struct CoreArgs {
    const uint16_t* qkv; // [T][ldq]: Q | K | V of the held heads, head i at columns i * hd of each part
    int64_t ldq;
    const uint16_t* o;   // [T][ldo] attention output (forward: written; backward: read)
    uint16_t* o_out;
    const uint16_t* dO;  // [T][ldo]
    int64_t ldo;
    float* lse;          // [Bt][ph][S]: base-2 log-sum-exp of the scaled logits
    float* delta;        // [Bt][ph][S]: sum_h dO[t][h] O[t][h]
    uint16_t* dqkv;      // [T][ldq]
    int S, ph;
    int hd;              // columns a head takes in qkv, o, dO, dqkv: HW, or a smaller multiple of 8 when HW > 64
    float scale, scale2; // 1 / sqrt(head width), and that times log2(e)
};

__device__ inline uint32_t pack_bf16(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

// acc + the two bf16 halves of w (v_dot2c_f32_bf16 against a pair of ones)
__device__ inline float pair_sum(uint32_t w, float acc) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), ones, acc, false);
}

// elements 8 s .. 8 s + 7 of an accumulator tile as a bf16 operand
__device__ inline bf16x8 pack_operand(const f32x16& a, int s) {
    const u32x4 v = {pack_bf16(a[8 * s], a[8 * s + 1]), pack_bf16(a[8 * s + 2], a[8 * s + 3]),
                     pack_bf16(a[8 * s + 4], a[8 * s + 5]), pack_bf16(a[8 * s + 6], a[8 * s + 7])};
    return __builtin_bit_cast(bf16x8, v);
}

// what pack_operand's rounding left out, as a second operand
__device__ inline bf16x8 pack_rest(const f32x16& a, int s, bf16x8 hi) {
    const u32x4 h = __builtin_bit_cast(u32x4, hi);
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        v[i] = pack_bf16(a[8 * s + 2 * i] - __uint_as_float(h[i] << 16), a[8 * s + 2 * i + 1] - __uint_as_float(h[i] & 0xFFFF0000u));
    return __builtin_bit_cast(bf16x8, v);
}

// orders this wave's LDS accesses around it: what one lane wrote another one reads, within the wave
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// operand whose depth runs along a tile row: row `row` of the tile, depth 16 s + 8 lhi .. + 7
template <int HW>
__device__ inline bf16x8 frag_rows(const unsigned char* tile, int row, int s, int lhi) {
    return __builtin_bit_cast(bf16x8, *(const u32x4*)(tile + row * row_bytes(HW) + 32 * s + 16 * lhi));
}

// A operand whose depth runs down the tile rows: for lane L, column col0 + L % 32 and the rows
// krow + 4 (L / 32) + e (e = 0..3), then krow + 8 + 4 (L / 32) + e.  Within each block of 16 lanes a
// transposing read hands lane n the e-th 16-bit element (e = 0..3) of what lane 4 e + n / 4 addressed,
// at position n % 4 of its 8 bytes: the 16 lanes address 4 rows x 4 groups of 4 columns.
template <int HW>
__device__ inline bf16x8 frag_cols(const unsigned char* tile, int krow, int col0, int lane) {
    constexpr int RSB = row_bytes(HW);
    const int gi = lane >> 4, li = lane & 15;
    const unsigned char* p = tile + (krow + 4 * (gi >> 1) + (li >> 2)) * RSB + (col0 + 16 * (gi & 1) + 4 * (li & 3)) * 2;
    const s16x4 h0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p);
    const s16x4 h1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 8 * RSB));
    const u32x2 a = __builtin_bit_cast(u32x2, h0), b = __builtin_bit_cast(u32x2, h1);
    return __builtin_bit_cast(bf16x8, u32x4{a[0], a[1], b[0], b[1]});
}

// The 16-byte pieces of a ROWS-row x HW-column tile that thread `tid` of a workgroup of NW waves moves from
// global memory to LDS through registers.  Rows are clamped to the last valid one (such rows only meet masked
// logits); columns from hd on (HW > 64 only) become zeros.  `g` is uniform over the workgroup and the tile's first
// row moves it by 64-bit scalar arithmetic; the per-thread part of the address is a 32-bit byte offset inside the
// tile, one multiply and add per piece: 63 rows of kMaxLd elements stay below 4 GiB, taller tiles take 64-bit offsets.
constexpr int64_t kMaxHeads = 65535;
template <int NW, int HW, int ROWS = 64>
struct TileMover {
    static constexpr int CPR = HW == HD ? 8 : 16;      // pieces per row (HW = 96: the last 4 of 16 move nothing)
    static constexpr int PER = ROWS * CPR / (64 * NW); // pieces per thread and tile
    static_assert(ROWS * CPR % (64 * NW) == 0 && 64 * NW % CPR == 0, "a thread's pieces share one column");
    static constexpr int64_t kMaxLd = 3 * kMaxHeads * HW; // Q | K | V
    typedef std::conditional_t<(ROWS * kMaxLd * 2 < ((int64_t)1 << 32)), uint32_t, uint64_t> Offset;
    u32x4 v[PER];
    __device__ void fetch(const uint16_t* g, uint32_t ld, int row0, int last_row, int hd, int tid) {
        const int r0 = row0 < last_row ? row0 : last_row, rmax = last_row - r0;
        const unsigned char* base = (const unsigned char*)(g + (int64_t)r0 * ld);
        int col = tid % CPR;
        if (HW > HD) col = col * 8 < hd ? col : 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            int row = tid / CPR + 64 * NW / CPR * i;
            row = row < rmax ? row : rmax;
            v[i] = *(const u32x4*)(base + ((Offset)row * ld + (uint32_t)col * 8u) * 2u);
        }
    }
    __device__ void stash(unsigned char* tile, int hd, int tid) const {
        const int col = tid % CPR;
        if (HW % 64 != 0 && col >= HW / 8) return;
        const bool pad = HW > HD && col * 8 >= hd;
#pragma unroll
        for (int i = 0; i < PER; ++i)
            *(u32x4*)(tile + (tid / CPR + 64 * NW / CPR * i) * row_bytes(HW) + col * 16) = pad ? u32x4{0u, 0u, 0u, 0u} : v[i];
    }
    // dot products of the tile's rows with those of another tile (of one wave): the CPR lanes of a group hold rows
    // group + 64 / CPR i; lane i of the group, i < PER, returns row dot_row
    __device__ static int dot_row(int tid) { return tid / CPR + 64 * NW / CPR * (tid % CPR); }
    __device__ float row_dots(const TileMover& o, int hd, int tid) const {
        static_assert(NW == 1 && PER <= CPR, "a lane for every row");
        float out = 0.f;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            float d = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                d = __builtin_fmaf(__uint_as_float(v[i][j] << 16), __uint_as_float(o.v[i][j] << 16), d);
                d = __builtin_fmaf(__uint_as_float(v[i][j] & 0xFFFF0000u), __uint_as_float(o.v[i][j] & 0xFFFF0000u), d);
            }
            if (HW > HD && tid % CPR * 8 >= hd) d = 0.f; // a piece beyond the head
#pragma unroll
            for (int m = 1; m < CPR; m <<= 1) d += __shfl_xor(d, m, 64);
            if (tid % CPR == i) out = d;
        }
        return out;
    }
};

// a row of HW bf16 as the depth-along-row operand of lane (row, lhi): sub-step s holds depth 16 s + 8 lhi .. + 7
template <int HW>
__device__ inline void load_row_operand(const uint16_t* g, int64_t ld, int row, int hd, int lhi, bf16x8 (&f)[HW / 16]) {
#pragma unroll
    for (int s = 0; s < HW / 16; ++s) {
        const int col = 16 * s + 8 * lhi;
        const bool pad = HW > HD && col >= hd;
        const u32x4 v = *(const u32x4*)(g + (int64_t)row * ld + (pad ? 0 : col));
        f[s] = __builtin_bit_cast(bf16x8, pad ? u32x4{0u, 0u, 0u, 0u} : v);
    }
}

// accumulator tiles D[h][row] (32-row blocks of h) -> out[row][32 j + 8 q + 4 lhi + r], scaled, 8-byte stores
template <int HW>
__device__ inline void store_rows(uint16_t* out_row, const f32x16 (&acc)[HW / 32], float f, int hd, int lhi) {
#pragma unroll
    for (int j = 0; j < HW / 32; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (HW == HD || 32 * j + 8 * q < hd) *(u32x2*)(out_row + 32 * j + 8 * q + 4 * lhi) =
                u32x2{pack_bf16(acc[j][4 * q] * f, acc[j][4 * q + 1] * f), pack_bf16(acc[j][4 * q + 2] * f, acc[j][4 * q + 3] * f)};
}

__device__ inline float other_half(float x) { return __shfl_xor(x, 32, 64); }

// Heads wider than 64: rows whose result is not finite are computed again, pair by pair (sdp_attn_rows.h): the plain core that
// served them read no masked pair and split no operand.  Heads up to 64 have always multiplied masked pairs by zero.
constexpr bool rows_again(int hw) { return two_terms(hw); }

// 0 when every element of the tiles times f is finite, else NaN
template <int N>
__device__ inline float finite_check(const f32x16 (&acc)[N], float f) {
    float c = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) c += acc[j][e] * f * 0.f;
    return c;
}
// of a wave's 32 rows (lane % 32): those of which either half is bad
__device__ inline uint32_t bad_rows(bool bad) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(bad);
    return (uint32_t)m | (uint32_t)(m >> 32);
}

// 2^x for x <= 0 (or -inf): the hardware instruction alone; results below the normal range may flush to zero
__device__ inline float exp2_neg(float x) { return __builtin_amdgcn_exp2f(x); }

// KW > 1: LDS of one wave, its two 32-row tiles and 64 statistics; after the loop its partial result, 32 rows of HW
// floats (rows 16 bytes longer, so that both the writes by row and the reads along a row hit every bank), and the statistics.
constexpr int wave_lds(int hw) { return 64 * row_bytes(hw) + 256; }
constexpr int part_row(int hw) { return hw + 4; }
static_assert(32 * part_row(HD) * 4 + 256 <= wave_lds(HD) && 32 * part_row(128) * 4 + 256 <= wave_lds(128), "fits the tiles");

// KW > 1: one flag per row of the workgroup's block, in what a wave's LDS has left beyond its partial result and statistics:
// set where store_parts met a value that is not finite.
constexpr int FLAGS = 32 * 4;
static_assert(32 * part_row(96) * 4 + 256 + FLAGS <= wave_lds(96) && 32 * part_row(128) * 4 + 256 + FLAGS <= wave_lds(128), "fits the tiles");
template <int HW>
__device__ inline uint32_t* row_flags(unsigned char* lds) { return (uint32_t*)(lds + wave_lds(HW) - FLAGS); }

// accumulator tiles D[h][row] -> the wave's partial result
template <int HW>
__device__ inline void put_part(unsigned char* mine, const f32x16 (&acc)[HW / 32], int l32, int lhi) {
    float* row = (float*)mine + l32 * part_row(HW);
#pragma unroll
    for (int j = 0; j < HW / 32; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(f32x4*)(row + 32 * j + 8 * q + 4 * lhi) = f32x4{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
}

// sum over the waves of f[w] x partial result, as bf16 rows of `out` (row0 + 0 .. 31, those below S); weights(row, f)
// fills f.  Columns from hd on are left alone.  Rows with a value that is not finite are flagged (rows_again).
template <int HW, int KW, class W>
__device__ inline void store_parts(unsigned char* lds, uint16_t* out, int64_t ld, int row0, int S, int hd, int tid, W weights) {
    constexpr int PIECES = 32 * HW / 4, THREADS = Split<KW>::THREADS;
#pragma unroll
    for (int i = 0; i < (PIECES + THREADS - 1) / THREADS; ++i) {
        const int e = tid + THREADS * i, row = e / (HW / 4), c = e % (HW / 4) * 4;
        if (PIECES % THREADS != 0 && e >= PIECES) break;
        float f[KW];
        weights(row, f);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < KW; ++w) {
            const f32x4 x = *(const f32x4*)((const float*)(lds + w * wave_lds(HW)) + row * part_row(HW) + c);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = __builtin_fmaf(x[r], f[w], v[r]);
        }
        if (row0 + row < S && (HW == HD || c < hd)) {
            *(u32x2*)(out + (int64_t)(row0 + row) * ld + c) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            if constexpr (rows_again(HW))
                if (v[0] * 0.f + v[1] * 0.f + v[2] * 0.f + v[3] * 0.f != 0.f) row_flags<HW>(lds)[row] = 1;
        }
    }
}

// The rows to compute again, each by one wave: `again` holds a wave's own rows (KW = 1), or the flags in LDS say which
// (KW > 1; called by all waves, after store_parts).
template <int HW, int KW, class F>
__device__ inline void each_row_again(unsigned char* lds, uint32_t again, int wave, int lane, F f) {
    if constexpr (KW != 1) {
        __syncthreads(); // the flags, and the values that these replace
        again = (uint32_t)__builtin_amdgcn_ballot_w64(lane < 32 && row_flags<HW>(lds)[lane & 31] != 0) &
                ((KW == 4 ? 0x11111111u : 0x01010101u) << wave);
    }
    while (again) {
        f(__builtin_ctz(again));
        again &= again - 1;
    }
}

// Whether a wave fetches a tile beyond its last one rather than branch around the fetch.  KW > 1: the partial results' barrier
// waits for that tile.  Heads of 96, with the branch: 2 x 512 to 1 x 2048 tokens, 8 heads 1.5 to 5 us of 86 to 194 less; heads of
// 128, KW = 4: 1 to 1.5 us of 84 to 148; but KW = 8, which has no register to spare, 1 us more, and heads of 64 the same.
constexpr bool always_fetch(int hw, int kw) { return kw == 1 || hw == HD || (hw == 128 && kw == 8); }

// ---------------------------------------------------------------------------------------------------
// Forward.  A wave keeps a block of 32 queries as register operands and walks key/value tiles up to the diagonal.
// KW = 1: tiles of 64 keys, double-buffered in LDS (one barrier per tile): while tile t is used, tile t + 1 moves from
// registers into the other buffer and tile t + 2 is fetched from memory.  KW > 1: the wave's own tiles of 32 keys,
// single-buffered; the next one is in flight in registers.
// ---------------------------------------------------------------------------------------------------
template <int HW, int KW>
constexpr int fwd_lds() { return KW == 1 ? 4 * 64 * row_bytes(HW) : KW * wave_lds(HW); }

template <int HW, int KW>
__device__ inline void attn_fwd_block(const CoreArgs& a, const int q0, const int head, const int b, unsigned char* lds) {
    constexpr int KS = HW / 16, JB = HW / 32; // depth steps of a logit, 32-column blocks of the output
    constexpr int TR = KW == 1 ? 64 : 32;     // keys per tile
    constexpr int TILE = TR * row_bytes(HW);
    const int hd = HW == HD ? HD : a.hd;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S;
    const uint16_t* gQ = a.qkv + (int64_t)b * S * a.ldq + head * hd;
    const uint16_t* gK = gQ + a.ph * hd;
    const uint16_t* gV = gK + a.ph * hd;
    const int qrow0 = KW == 1 ? q0 + 32 * wave : q0, qrow = qrow0 + l32;
    bf16x8 qf[KS];
    load_row_operand<HW>(gQ, a.ldq, qrow < S ? qrow : S - 1, hd, lhi, qf);

    // tile t holds the keys first + step t ..
    const int first = KW == 1 ? 0 : TR * wave, step = TR * KW;
    const int kv_end = q0 + Split<KW>::ROWS < S ? q0 + Split<KW>::ROWS : S;
    const int ntiles = kv_end > first ? (kv_end - first + step - 1) / step : 0;
    f32x16 acc[JB];
    // KW > 1: a wave's first tile may hold no key of some queries; the reference then starts from the lowest finite value
    float m = KW == 1 ? -INFINITY : -3.402823466e38f, lsum = 0.f;
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

    TileMover<KW == 1 ? NW : 1, HW, TR> pk, pv;
    const int mt = KW == 1 ? tid : lane; // the mover's thread
    unsigned char* const mine = lds + wave * wave_lds(HW);
    const uint32_t ld = (uint32_t)a.ldq;
    pk.fetch(gK, ld, first, S - 1, hd, mt);
    pv.fetch(gV, ld, first, S - 1, hd, mt);
    // fetches and stashes run unconditionally where always_fetch says so (rows are clamped, and a tile beyond the last one is
    // never read): no branch, hence no register copies, around the loop-carried pieces
    if constexpr (KW == 1) {
        pk.stash(lds, hd, mt);
        pv.stash(lds + 2 * TILE, hd, mt);
        pk.fetch(gK, ld, step, S - 1, hd, mt);
        pv.fetch(gV, ld, step, S - 1, hd, mt);
        __syncthreads();
    }
    for (int t = 0; t < ntiles; ++t) {
        const unsigned char *tK, *tV;
        if constexpr (KW == 1) {
            tK = lds + (t & 1) * TILE, tV = tK + 2 * TILE;
            // the other buffer was last read before the barrier that ended step t - 1
            pk.stash(lds + ((t + 1) & 1) * TILE, hd, mt);
            pv.stash(lds + (2 + ((t + 1) & 1)) * TILE, hd, mt);
            pk.fetch(gK, ld, step * (t + 2), S - 1, hd, mt);
            pv.fetch(gV, ld, step * (t + 2), S - 1, hd, mt);
        } else {
            tK = mine, tV = mine + TILE;
            pk.stash(mine, hd, mt);
            pv.stash(mine + TILE, hd, mt);
            if (always_fetch(HW, KW) || t + 1 < ntiles) {
                pk.fetch(gK, ld, first + step * (t + 1), S - 1, hd, mt);
                pv.fetch(gV, ld, first + step * (t + 1), S - 1, hd, mt);
            }
            wave_sync();
        }
        const int kv0 = first + step * t;
        if (kv0 <= qrow0 + 31) { // wave-uniform: otherwise every key lies after the wave's queries
            // logits, transposed: sc[tb] = D[key 32 tb + ..][query]
            f32x16 sc[TR / 32];
#pragma unroll
            for (int tb = 0; tb < TR / 32; ++tb)
#pragma unroll
                for (int e = 0; e < 16; ++e) sc[tb][e] = 0.f;
#pragma unroll
            for (int tb = 0; tb < TR / 32; ++tb)
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    sc[tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<HW>(tK, 32 * tb + l32, s, lhi), qf[s], sc[tb], 0, 0, 0);
            if (kv0 + TR - 1 > qrow0 || kv0 + TR > S) { // wave-uniform: some logits of this tile are masked
#pragma unroll
                for (int tb = 0; tb < TR / 32; ++tb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int key = kv0 + 32 * tb + 8 * (e >> 2) + 4 * lhi + (e & 3);
                        if (key > qrow || key >= S) sc[tb][e] = -INFINITY;
                    }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int tb = 0; tb < TR / 32; ++tb)
#pragma unroll
                for (int e = 0; e < 16; ++e) mx = fmaxf(mx, sc[tb][e]);
            mx = fmaxf(mx, other_half(mx));
            // m is the reference the exponents are taken against, in units of the scaled base-2 logits (the
            // scale rides in the multiply-add).  It follows the running maximum lazily: only when a query's
            // maximum has grown by more than kSlack is the reference moved and the accumulators rescaled, so
            // probabilities stay below 2^kSlack and the multiplies of the rescale run on few tiles (with KW = 1 the
            // first one always: it holds key 0, which no query masks, so m is finite from then on).
            const float m_cand = mx * a.scale2;
            if (__builtin_amdgcn_ballot_w64(m_cand > m + kSlack) != 0) { // wave-uniform
                const float m_new = m_cand > m + kSlack ? m_cand : m;
                const float alpha = exp2_neg(m - m_new);
                m = m_new;
                lsum *= alpha;
#pragma unroll
                for (int j = 0; j < JB; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[j][e] *= alpha;
            }
            // One term: the sum runs over the rounded probabilities, the ones the second product sees, two per
            // instruction.  Two terms: over the probabilities themselves.
            bf16x8 pf[TR / 32][2]; // probabilities as operands: [key block][depth half]
            float ps = 0.f;
#pragma unroll
            for (int tb = 0; tb < TR / 32; ++tb)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    u32x4 w;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float p0 = exp2_neg(__builtin_fmaf(sc[tb][8 * h + 2 * i], a.scale2, -m));
                        const float p1 = exp2_neg(__builtin_fmaf(sc[tb][8 * h + 2 * i + 1], a.scale2, -m));
                        w[i] = pack_bf16(p0, p1);
                        if constexpr (two_terms(HW)) {
                            sc[tb][8 * h + 2 * i] = p0, sc[tb][8 * h + 2 * i + 1] = p1;
                            ps += p0 + p1;
                        } else {
                            ps = pair_sum(w[i], ps);
                        }
                    }
                    pf[tb][h] = __builtin_bit_cast(bf16x8, w);
                }
            lsum += ps;
            // O^T[h][query] += sum_key V[key][h] P[query][key]
#pragma unroll
            for (int tb = 0; tb < TR / 32; ++tb)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    bf16x8 rest;
                    if constexpr (two_terms(HW)) rest = pack_rest(sc[tb], s, pf[tb][s]);
#pragma unroll
                    for (int j = 0; j < JB; ++j) {
                        const bf16x8 vfr = frag_cols<HW>(tV, 32 * tb + 16 * s, 32 * j, lane);
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr, pf[tb][s], acc[j], 0, 0, 0);
                        if constexpr (two_terms(HW)) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr, rest, acc[j], 0, 0, 0);
                    }
                }
        }
        // tile t is released (KW = 1: and tile t + 1 is in place)
        if constexpr (KW == 1) __syncthreads(); else wave_sync();
    }
    const float l = lsum + other_half(lsum);
    uint16_t* const out = a.o_out + (int64_t)b * S * a.ldo + head * hd;
    float* const lse = a.lse + ((int64_t)b * a.ph + head) * S;
    uint32_t again = 0;
    if constexpr (KW == 1) {
        if constexpr (rows_again(HW)) again = bad_rows(qrow < S && finite_check(acc, 1.f / l) != 0.f);
        if (qrow < S && !(again >> l32 & 1)) {
            store_rows<HW>(out + (int64_t)qrow * a.ldo, acc, 1.f / l, hd, lhi);
            if (lhi == 0) lse[qrow] = m + log2f(l);
        }
    } else {
        put_part<HW>(mine, acc, l32, lhi);
        constexpr int STAT = 32 * part_row(HW) * 4; // [32] references, [32] sums
        ((float*)(mine + STAT))[lane] = lhi == 0 ? m : l;
        if (rows_again(HW) && tid < 32) row_flags<HW>(lds)[tid] = 0;
        __syncthreads();
        store_parts<HW, KW>(lds, out, a.ldo, q0, S, hd, tid, [&](int row, float (&f)[KW]) {
            float top = -INFINITY, sum = 0.f;
#pragma unroll
            for (int w = 0; w < KW; ++w) top = fmaxf(top, ((const float*)(lds + w * wave_lds(HW) + STAT))[row]);
#pragma unroll
            for (int w = 0; w < KW; ++w) {
                const float* st = (const float*)(lds + w * wave_lds(HW) + STAT);
                f[w] = exp2_neg(st[row] - top);
                sum = __builtin_fmaf(f[w], st[32 + row], sum);
            }
#pragma unroll
            for (int w = 0; w < KW; ++w) f[w] /= sum;
        });
        if (tid < 32 && q0 + tid < S) {
            float top = -INFINITY, sum = 0.f;
#pragma unroll
            for (int w = 0; w < KW; ++w) top = fmaxf(top, ((const float*)(lds + w * wave_lds(HW) + STAT))[tid]);
#pragma unroll
            for (int w = 0; w < KW; ++w) {
                const float* st = (const float*)(lds + w * wave_lds(HW) + STAT);
                sum = __builtin_fmaf(exp2_neg(st[tid] - top), st[32 + tid], sum);
            }
            lse[q0 + tid] = top + log2f(sum);
        }
    }
    if constexpr (rows_again(HW))
        each_row_again<HW, KW>(lds, again, wave, lane, [&](int r) {
            const AttnRows<uint16_t> ar{gQ, gK, gV, a.ldq, nullptr, 0, S, hd, a.scale, a.scale2};
            attn_row_fwd(ar, qrow0 + r, lane, out + (int64_t)(qrow0 + r) * a.ldo, lse + qrow0 + r);
        });
}

// Causal rows differ in length: block i of a sequence meets i + 1 blocks of keys, and at the sizes this
// block runs at every workgroup of a launch is resident at once (about three per CU), so nothing evens the
// work out afterwards.  One block per workgroup, and the blocks are dealt to the workgroup ids so that ids
// congruent modulo the number of CUs -- which the dispatcher places on the same CU, one pass after the other
// -- get a long, a short and a middling block: ranks in the order "longest first" run forwards in even passes
// and backwards in odd ones.  Launches with more passes than fit at once start the long blocks first.
__device__ inline void causal_item(int L, int nitems, int nbh, int nblocks, int ph, int& blk, int& head, int& b) {
    constexpr int W = 256;
    const int pass = L / W, base = pass * W;
    const int width = nitems - base < W ? nitems - base : W;
    const int w = L - base;
    const int r = (pass & 1) ? base + (width - 1 - w) : base + w;
    blk = nblocks - 1 - r / nbh;
    const int bh = r % nbh;
    head = bh % ph, b = bh / ph;
}

// The core's launches carry transposes that the contractions after them read (WoT in the forward pass, Wqkv beside dQ; for
// plain weight gradients X, dY, O beside dQ and dQ beside dK/dV as well) as workgroups from `nitems` on: the core moves little
// memory, and the blocks of a causal sequence end at different times.  With X, dY, O and dQ among them, on launches of their own:
// block of 4 x 2048 tokens, 12 heads of 64 464 us, this way 438; 24 heads of 50, 12 held 690 -> 658.
constexpr int side_tiles(int lds) { return lds / kTransposeLds < 4 ? lds / kTransposeLds : 4; }

// A launch's workgroups in one order.  One axis of a grid holds fewer than 2^32 threads (2^24 workgroups); with more
// workgroups the second axis counts rows of kGridRow, the last of which may be partly beyond them.
constexpr int kGridRow = 1 << 23;
__device__ inline int workgroup_id() { return (int)(blockIdx.y * kGridRow + blockIdx.x); }
inline dim3 workgroup_grid(int64_t n) {
    return n < 2 * kGridRow ? dim3((unsigned)n) : dim3(kGridRow, (unsigned)((n + kGridRow - 1) / kGridRow));
}
template <int LDS, int THREADS>
__device__ inline void carried(const SideJobs& side, int w, unsigned char* lds) {
    constexpr int HALVES = THREADS / 256, PER = side_tiles(LDS / HALVES), ALL = PER * HALVES;
    if (w >= (side.end[kMaxTransposeJobs - 1] + ALL - 1) / ALL) return;
    if constexpr (HALVES == 1) {
        side_transposes<PER, true>(side, w, lds, threadIdx.x);
    } else {
        const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
        side_transposes<PER, true>(side, w * HALVES + half, lds + half * PER * kTransposeLds, threadIdx.x & 255);
    }
}

// waves per SIMD the registers are allotted for.  KW = 1, heads of 64: 3 beat 2 (86 -> 77 us at 4 x 2048 tokens, 12 heads)
// and 4 spill.  KW = 4: the wide heads take the registers of one or two waves.
constexpr int waves_fwd(int hw, int kw) { return kw == 1 ? (hw == HD ? 3 : 2) : 2; }
constexpr int waves_dq(int hw, int kw) { return kw == 1 ? (hw == HD ? 3 : 2) : (kw == 8 || hw == HD ? 2 : 1); }
constexpr int waves_dkv(int hw, int kw) { return kw != 4 || hw == HD ? 2 : 1; }

template <int HW, int KW>
__global__ __launch_bounds__(Split<KW>::THREADS) __attribute__((amdgpu_waves_per_eu(waves_fwd(HW, KW), waves_fwd(HW, KW))))
void attn_fwd_kernel(CoreArgs a, int nblocks, int nbh, SideJobs side) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[fwd_lds<HW, KW>()];
    const int nitems = nblocks * nbh;
    const int id = workgroup_id();
    if (id >= nitems) return carried<sizeof(lds), Split<KW>::THREADS>(side, id - nitems, lds);
    int blk, head, b;
    causal_item(id, nitems, nbh, nblocks, a.ph, blk, head, b);
    attn_fwd_block<HW, KW>(a, blk * Split<KW>::ROWS, head, b, lds);
}

// ---------------------------------------------------------------------------------------------------
// Backward, dQ (and delta).  Same walk as the forward: wave w keeps its 32 queries' Q and dO rows as
// register operands; P is recomputed from the stored log-sum-exp.
//   dP[q][k] = dO[q] . V[k];  dZ = P (dP - delta[q]);  dQ[q] = scale sum_k dZ[q][k] K[k]
// ---------------------------------------------------------------------------------------------------
template <int HW, int KW>
constexpr int dq_lds() { return KW == 1 ? 2 * 64 * row_bytes(HW) : KW * wave_lds(HW); }

template <int HW, int KW, bool STORE_DELTA = true>
__device__ inline void attn_bwd_dq_block(const CoreArgs& a, const int q0, const int head, const int b, unsigned char* lds) {
    constexpr int KS = HW / 16, JB = HW / 32;
    constexpr int TR = KW == 1 ? 64 : 32; // keys per tile
    const int hd = HW == HD ? HD : a.hd;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S;
    const uint16_t* gQ = a.qkv + (int64_t)b * S * a.ldq + head * hd;
    const uint16_t* gK = gQ + a.ph * hd;
    const uint16_t* gV = gK + a.ph * hd;
    const int qrow0 = KW == 1 ? q0 + 32 * wave : q0, qrow = qrow0 + l32;
    const int qc = qrow < S ? qrow : S - 1;
    bf16x8 qf[KS], dof[KS];
    load_row_operand<HW>(gQ, a.ldq, qc, hd, lhi, qf);
    const int64_t orow = ((int64_t)b * S + qc) * a.ldo + head * hd;
    load_row_operand<HW>(a.dO + orow, 0, 0, hd, lhi, dof);
    float delta = 0.f;
    {
        bf16x8 of[KS];
        load_row_operand<HW>(a.o + orow, 0, 0, hd, lhi, of);
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) delta += (float)dof[s][e] * (float)of[s][e];
        delta += other_half(delta);
    }
    const int64_t stat = ((int64_t)b * a.ph + head) * S;
    if (STORE_DELTA && qrow < S && lhi == 0 && (KW == 1 || wave == 0)) a.delta[stat + qrow] = delta;
    const float L2 = a.lse[stat + qc];

    const int first = KW == 1 ? 0 : TR * wave, step = TR * KW;
    const int kv_end = q0 + Split<KW>::ROWS < S ? q0 + Split<KW>::ROWS : S;
    const int ntiles = kv_end > first ? (kv_end - first + step - 1) / step : 0;
    f32x16 acc[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

    TileMover<KW == 1 ? NW : 1, HW, TR> pk, pv;
    const int mt = KW == 1 ? tid : lane;
    unsigned char* const sK = KW == 1 ? lds : lds + wave * wave_lds(HW);
    unsigned char* const sV = sK + TR * row_bytes(HW);
    const uint32_t ld = (uint32_t)a.ldq;
    pk.fetch(gK, ld, first, S - 1, hd, mt);
    pv.fetch(gV, ld, first, S - 1, hd, mt);
    for (int t = 0; t < ntiles; ++t) {
        if constexpr (KW == 1) __syncthreads(); else wave_sync();
        pk.stash(sK, hd, mt);
        pv.stash(sV, hd, mt);
        if constexpr (KW == 1) __syncthreads(); else wave_sync();
        if (always_fetch(HW, KW) || t + 1 < ntiles) {
            pk.fetch(gK, ld, first + step * (t + 1), S - 1, hd, mt); // rows are clamped
            pv.fetch(gV, ld, first + step * (t + 1), S - 1, hd, mt);
        }
        const int kv0 = first + step * t;
        if (kv0 > qrow0 + 31) continue;
        const bool edge = kv0 + TR - 1 > qrow0 || kv0 + TR > S;
#pragma unroll
        for (int tb = 0; tb < TR / 32; ++tb) {
            f32x16 sc, dp;
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[e] = 0.f, dp[e] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<HW>(sK, 32 * tb + l32, s, lhi), qf[s], sc, 0, 0, 0);
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<HW>(sV, 32 * tb + l32, s, lhi), dof[s], dp, 0, 0, 0);
            }
            if (edge) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int key = kv0 + 32 * tb + 8 * (e >> 2) + 4 * lhi + (e & 3);
                    if (key > qrow || key >= S) sc[e] = -INFINITY;
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[e] = exp2_neg(__builtin_fmaf(sc[e], a.scale2, -L2)) * (dp[e] - delta);
            // dQ^T[h][query] += sum_key K[key][h] dZ[query][key]
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 zf = pack_operand(sc, s);
                bf16x8 rest;
                if constexpr (two_terms(HW)) rest = pack_rest(sc, s, zf);
#pragma unroll
                for (int j = 0; j < JB; ++j) {
                    const bf16x8 kfr = frag_cols<HW>(sK, 32 * tb + 16 * s, 32 * j, lane);
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr, zf, acc[j], 0, 0, 0);
                    if constexpr (two_terms(HW)) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr, rest, acc[j], 0, 0, 0);
                }
            }
        }
    }
    uint16_t* const out = a.dqkv + (int64_t)b * S * a.ldq + head * hd;
    uint32_t again = 0;
    if constexpr (KW == 1) {
        if constexpr (rows_again(HW)) again = bad_rows(qrow < S && finite_check(acc, a.scale) != 0.f);
        if (qrow < S && !(again >> l32 & 1)) store_rows<HW>(out + (int64_t)qrow * a.ldq, acc, a.scale, hd, lhi);
    } else {
        wave_sync();
        put_part<HW>(sK, acc, l32, lhi);
        if (rows_again(HW) && tid < 32) row_flags<HW>(lds)[tid] = 0;
        __syncthreads();
        store_parts<HW, KW>(lds, out, a.ldq, q0, S, hd, tid, [&](int, float (&f)[KW]) {
#pragma unroll
            for (int w = 0; w < KW; ++w) f[w] = a.scale;
        });
    }
    if constexpr (rows_again(HW))
        each_row_again<HW, KW>(lds, again, wave, lane, [&](int r) {
            const AttnRows<uint16_t> ar{gQ, gK, gV, a.ldq, a.dO + (int64_t)b * S * a.ldo + head * hd, a.ldo, S, hd, a.scale, a.scale2};
            // lane r holds that row's statistics
            attn_row_dq(ar, qrow0 + r, lane, __shfl(L2, r, 64), __shfl(delta, r, 64), out + (int64_t)(qrow0 + r) * a.ldq);
        });
}

template <int HW, int KW>
__global__ __launch_bounds__(Split<KW>::THREADS) __attribute__((amdgpu_waves_per_eu(waves_dq(HW, KW), waves_dq(HW, KW))))
void attn_bwd_dq_kernel(CoreArgs a, int nblocks, int nbh, SideJobs side) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[dq_lds<HW, KW>()];
    const int nitems = nblocks * nbh;
    const int id = workgroup_id();
    if (id >= nitems) return carried<sizeof(lds), Split<KW>::THREADS>(side, id - nitems, lds);
    int blk, head, b;
    causal_item(id, nitems, nbh, nblocks, a.ph, blk, head, b);
    attn_bwd_dq_block<HW, KW>(a, blk * Split<KW>::ROWS, head, b, lds);
}

// ---------------------------------------------------------------------------------------------------
// Backward, dK and dV.  A wave keeps 32 keys of one (sequence, head) (K and V rows) as register operands
// and walks query tiles from the diagonal to the end of the sequence; Q, dO and the per-query statistics of a tile
// are staged in LDS.
//   dV[k] = sum_q P[q][k] dO[q];   dK[k] = scale sum_q dZ[q][k] Q[q]
// ---------------------------------------------------------------------------------------------------
// At HW = 128 a wave's accumulators (128 registers), K rows (32), one 32 x 32 block of logits and of logit gradients
// (32) leave no room for its V rows (32) and the pieces of 64 staged queries (32) under the 256 registers of two waves
// per SIMD: the workgroup's V rows then stay in LDS and are read from there per block, and a tile has 32 queries.  At
// HW = 96 the shorter tile is enough.  (KW = 4 runs one wave per SIMD there: 512 registers, all operands kept.  KW = 8, two
// waves per SIMD and the pieces of two whole tiles in every wave's registers, keeps the block's V rows in LDS at HW = 96, its K and
// V rows at HW = 128, behind a barrier of their own.)
template <int HW, int KW>
struct DkvShape {
    static constexpr bool kVInLds = HW == 128 ? KW != 4 : HW == 96 && KW == 8, kKInLds = HW == 128 && KW == 8;
    static constexpr int QT = HW == HD && KW == 1 ? 64 : 32; // queries per tile
    static constexpr int ROWS_BYTES = Split<KW>::ROWS * row_bytes(HW);
    static constexpr int LOOP = KW == 1 ? 2 * QT * row_bytes(HW) + 2 * QT * 4 : KW * wave_lds(HW);
    static constexpr int LDS = LOOP + (kVInLds + kKInLds) * ROWS_BYTES;
    static_assert(LDS <= 160 * 1024, "LDS of one CU");
};

// OWN_DELTA: the queries' delta is computed from their dO and O rows as the tile is staged (every wave its own tile), in the place
// of what the dQ kernel has left.  O's rows are fetched a tile ahead like the others; KW = 8 has no registers for them and
// fetches them into those that staging has freed (wide heads).  KW = 8 is at the limit of 256 registers: heads above 96 spill 13 of them
// in dK/dV alone (56 bytes of scratch a lane), 15 in the one launch with dQ; heads of 65 to 96 one and 9.
template <int HW, int KW, bool OWN_DELTA = false>
__device__ inline void attn_bwd_dkv_block(const CoreArgs& a, const int k0, const int head, const int b, unsigned char* lds) {
    using Shape = DkvShape<HW, KW>;
    static_assert(!OWN_DELTA || KW > 1, "a wave's own tile");
    constexpr bool kAhead = OWN_DELTA && KW == 4;
    constexpr int KS = HW / 16, JB = HW / 32, QT = Shape::QT;
    constexpr bool kVInLds = Shape::kVInLds, kKInLds = Shape::kKInLds;
    const int hd = HW == HD ? HD : a.hd;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = a.S;
    const uint16_t* gQ = a.qkv + (int64_t)b * S * a.ldq + head * hd;
    const uint16_t* gK = gQ + a.ph * hd;
    const uint16_t* gV = gK + a.ph * hd;
    const uint16_t* gO = a.dO + (int64_t)b * S * a.ldo + head * hd;
    const int64_t stat = ((int64_t)b * a.ph + head) * S;
    const int krow0 = KW == 1 ? k0 + 32 * wave : k0, krow = krow0 + l32;
    const int kc = krow < S ? krow : S - 1;
    unsigned char* const sQ = KW == 1 ? lds : lds + wave * wave_lds(HW);
    unsigned char* const sO = sQ + QT * row_bytes(HW);
    float* const sL = (float*)(sO + QT * row_bytes(HW)); // log-sum-exp of the tile's queries, then delta
    float* const sD = sL + QT;
    unsigned char* const sV = lds + Shape::LOOP;
    unsigned char* const sK = sV + Shape::ROWS_BYTES;
    const int own_row = KW == 1 ? 32 * wave + l32 : l32; // of sV, sK
    bf16x8 kf[kKInLds ? 1 : KS], vf[kVInLds ? 1 : KS];
    if constexpr (!kKInLds) load_row_operand<HW>(gK, a.ldq, kc, hd, lhi, kf);
    if constexpr (kVInLds) {
        TileMover<Split<KW>::THREADS / 64, HW, Split<KW>::ROWS> mv, mk;
        mv.fetch(gV, (uint32_t)a.ldq, k0, S - 1, hd, tid);
        if constexpr (kKInLds) mk.fetch(gK, (uint32_t)a.ldq, k0, S - 1, hd, tid);
        mv.stash(sV, hd, tid);
        if constexpr (kKInLds) mk.stash(sK, hd, tid);
        // Every wave reads rows that all of them have put away.  KW = 1: after the barriers of the first tile; KW > 1 has none in
        // its loop.
        if constexpr (KW > 1) __syncthreads();
    } else {
        load_row_operand<HW>(gV, a.ldq, kc, hd, lhi, vf);
    }

    f32x16 acc_k[JB], acc_v[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc_k[j][e] = 0.f, acc_v[j][e] = 0.f;

    // tile t holds the queries QT (t0 + KW t) ..; t0 lies at the diagonal, which lies inside the sequence (k0 < S)
    const int t0 = k0 / QT + (KW == 1 ? 0 : wave), tend = (S + QT - 1) / QT;
    const int ntiles = tend > t0 ? (tend - t0 + KW - 1) / KW : 0;
    TileMover<KW == 1 ? NW : 1, HW, QT> pq, po, px; // px: O, for delta
    const uint16_t* gX = OWN_DELTA ? a.o + (int64_t)b * S * a.ldo + head * hd : nullptr;
    const int mt = KW == 1 ? tid : lane;
    const uint32_t ldq32 = (uint32_t)a.ldq, ldo32 = (uint32_t)a.ldo;
    // per-query statistics of a tile: threads 0 .. QT - 1 carry the log-sum-exp, QT .. 2 QT - 1 delta
    const float* gstat = (OWN_DELTA || mt < QT ? a.lse : a.delta) + stat;
    const int sq = mt % QT;
    auto stat_of = [&](int q) { return gstat[q < S ? q : S - 1]; };
    pq.fetch(gQ, ldq32, QT * t0, S - 1, hd, mt);
    po.fetch(gO, ldo32, QT * t0, S - 1, hd, mt);
    if constexpr (kAhead) px.fetch(gX, ldo32, QT * t0, S - 1, hd, mt);
    float pstat = stat_of(QT * t0 + sq);
    for (int t = 0; t < ntiles; ++t) {
        if constexpr (KW == 1) __syncthreads(); else wave_sync();
        pq.stash(sQ, hd, mt);
        po.stash(sO, hd, mt);
        if constexpr (OWN_DELTA) {
            if constexpr (!kAhead) px.fetch(gX, ldo32, QT * (t0 + KW * t), S - 1, hd, mt);
            if (mt < QT) sL[mt] = pstat;
            const float d = po.row_dots(px, hd, mt); // of the tile's row that this lane is to put away
            if (mt % TileMover<1, HW, QT>::CPR < TileMover<1, HW, QT>::PER) sD[po.dot_row(mt)] = d;
        } else {
            if (mt < 2 * QT) sL[mt] = pstat;
        }
        if constexpr (KW == 1) __syncthreads(); else wave_sync();
        // the next tile (rows are clamped)
        const int qt0 = QT * (t0 + KW * t), next = qt0 + QT * KW;
        if (always_fetch(HW, KW) || t + 1 < ntiles) {
            pq.fetch(gQ, ldq32, next, S - 1, hd, mt);
            po.fetch(gO, ldo32, next, S - 1, hd, mt);
            if constexpr (kAhead) px.fetch(gX, ldo32, next, S - 1, hd, mt);
            pstat = stat_of(next + sq);
        }
        if (qt0 + QT - 1 < krow0) continue; // wave-uniform: every query of the tile lies before the wave's keys
        const bool edge = qt0 < krow0 + 31 || qt0 + QT > S;
#pragma unroll
        for (int tb = 0; tb < QT / 32; ++tb) {
            // sc = D[query 32 tb + ..][key], dp likewise
            f32x16 sc, dp;
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[e] = 0.f, dp[e] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                bf16x8 k, v;
                if constexpr (kKInLds) k = frag_rows<HW>(sK, own_row, s, lhi);
                else k = kf[s];
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<HW>(sQ, 32 * tb + l32, s, lhi), k, sc, 0, 0, 0);
                if constexpr (kVInLds) v = frag_rows<HW>(sV, own_row, s, lhi);
                else v = vf[s];
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_rows<HW>(sO, 32 * tb + l32, s, lhi), v, dp, 0, 0, 0);
            }
            if (edge) { // a branch of its own: only the tiles on the diagonal and the ragged last one pay for it
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int query = qt0 + 32 * tb + 8 * (e >> 2) + 4 * lhi + (e & 3);
                    if (krow > query || query >= S) sc[e] = -INFINITY;
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 l4 = *(const f32x4*)(sL + 32 * tb + 8 * q + 4 * lhi);
                const f32x4 d4 = *(const f32x4*)(sD + 32 * tb + 8 * q + 4 * lhi);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float z = sc[4 * q + r];
                    const float p = exp2_neg(__builtin_fmaf(z, a.scale2, -l4[r]));
                    sc[4 * q + r] = p;
                    dp[4 * q + r] = p * (dp[4 * q + r] - d4[r]);
                }
            }
            // dV^T[h][key] += sum_query dO[query][h] P[query][key];  dK^T[h][key] += sum_query Q[query][h] dZ[query][key]
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const bf16x8 pf = pack_operand(sc, s), zf = pack_operand(dp, s);
                bf16x8 pr, zr;
                if constexpr (two_terms(HW)) pr = pack_rest(sc, s, pf), zr = pack_rest(dp, s, zf);
#pragma unroll
                for (int j = 0; j < JB; ++j) {
                    const bf16x8 ofr = frag_cols<HW>(sO, 32 * tb + 16 * s, 32 * j, lane);
                    acc_v[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ofr, pf, acc_v[j], 0, 0, 0);
                    if constexpr (two_terms(HW)) acc_v[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ofr, pr, acc_v[j], 0, 0, 0);
                    const bf16x8 qfr = frag_cols<HW>(sQ, 32 * tb + 16 * s, 32 * j, lane);
                    acc_k[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qfr, zf, acc_k[j], 0, 0, 0);
                    if constexpr (two_terms(HW)) acc_k[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qfr, zr, acc_k[j], 0, 0, 0);
                }
            }
        }
    }
    uint16_t* const out = a.dqkv + (int64_t)b * S * a.ldq + head * hd;
    uint32_t again = 0;
    if constexpr (KW == 1) {
        if constexpr (rows_again(HW)) again = bad_rows(krow < S && finite_check(acc_k, a.scale) + finite_check(acc_v, 1.f) != 0.f);
        if (krow < S && !(again >> l32 & 1)) {
            uint16_t* row = out + (int64_t)krow * a.ldq;
            store_rows<HW>(row + a.ph * hd, acc_k, a.scale, hd, lhi);
            store_rows<HW>(row + 2 * a.ph * hd, acc_v, 1.f, hd, lhi);
        }
    } else {
#pragma unroll
        for (int part = 1; part <= 2; ++part) { // dK, then dV
            const float f1 = part == 1 ? a.scale : 1.f;
            if (part == 1) wave_sync(); else __syncthreads();
            put_part<HW>(sQ, part == 1 ? acc_k : acc_v, l32, lhi);
            if (rows_again(HW) && part == 1 && tid < 32) row_flags<HW>(lds)[tid] = 0;
            __syncthreads();
            store_parts<HW, KW>(lds, out + part * a.ph * hd, a.ldq, k0, S, hd, tid, [&](int, float (&f)[KW]) {
#pragma unroll
                for (int w = 0; w < KW; ++w) f[w] = f1;
            });
        }
    }
    if constexpr (rows_again(HW))
        each_row_again<HW, KW>(lds, again, wave, lane, [&](int r) {
            const AttnRows<uint16_t> ar{gQ, gK, gV, a.ldq, gO, a.ldo, S, hd, a.scale, a.scale2};
            uint16_t* row = out + (int64_t)(krow0 + r) * a.ldq;
            attn_row_dkv<OWN_DELTA>(ar, krow0 + r, lane, a.lse + stat, OWN_DELTA ? nullptr : a.delta + stat, row + a.ph * hd, row + 2 * a.ph * hd, gX);
        });
}

template <int HW, int KW>
__global__ __launch_bounds__(Split<KW>::THREADS) __attribute__((amdgpu_waves_per_eu(waves_dkv(HW, KW), waves_dkv(HW, KW))))
void attn_bwd_dkv_kernel(CoreArgs a, int nblocks, int nbh, SideJobs side) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[DkvShape<HW, KW>::LDS];
    const int nitems = nblocks * nbh;
    const int id = workgroup_id();
    if (id >= nitems) return carried<sizeof(lds), Split<KW>::THREADS>(side, id - nitems, lds);
    int blk, head, b;
    causal_item(id, nitems, nbh, nblocks, a.ph, blk, head, b);
    // key block i meets the query blocks i .. n - 1: the first key blocks are the long ones
    attn_bwd_dkv_block<HW, KW>(a, (nblocks - 1 - blk) * Split<KW>::ROWS, head, b, lds);
}

// dK, dV and dQ as one launch, where the walked axis is split: either alone leaves CUs idle, and what a launch costs between two
// kernels is a sixteenth of such a call.  dK/dV then takes delta from dO and O itself.  Forward and backward of an attention, two
// launches / one, heads up to 64: 2 x 256 tokens, 6 heads of 64 47 / 42.7 us, 1 x 64, 4 of 50 44 / 39, 4 x 100, 12 of 50 50.5 / 46,
// 1 x 1024, 12 of 64 80.5 / 75.7, 2 x 1024, 12 122 / 119 (core_merged_backward has the lines).
// Wider heads run one workgroup a CU, so that a block of keys and one of queries, longest first, take turns in the order of the
// workgroups; up to as many blocks of 32 rows as the first half of them fills the CUs (KW = 8 256, KW = 4 224): 1 x 64 tokens, 4 heads
// of 128 49.9 / 40.9, 1 x 512, 4 67 / 55.8, 1 x 1500, 4 105 / 92.6, 1 x 1024, 8 (256 blocks, KW = 8) 106.8 / 101.9, 1 x 155, 13 of 96
// 77.5 / 68.1, 2 x 200, 8 of 128 69.4 / 62; but 2 x 256, 16 (256, KW = 4) 114.3 / 115.7, 1 x 1100, 8 of 96 (280) 103.8 / 110.6, 2 x 1024,
// 12 of 128 (768) 244 / 270: the re-read of O and the longer tail of a launch of several rounds cost more than the gap there.
template <int HW, int KW>
__global__ __launch_bounds__(Split<KW>::THREADS) __attribute__((amdgpu_waves_per_eu(waves_dkv(HW, KW), waves_dkv(HW, KW))))
void attn_bwd_kernel(CoreArgs a, int nblocks, int nbh, SideJobs side) {
    constexpr int LDS = dq_lds<HW, KW>() > DkvShape<HW, KW>::LDS ? dq_lds<HW, KW>() : DkvShape<HW, KW>::LDS;
    __shared__ __attribute__((aligned(16))) unsigned char lds[LDS];
    const int nitems = nblocks * nbh;
    const int id = workgroup_id();
    if (id >= 2 * nitems) return carried<sizeof(lds), Split<KW>::THREADS>(side, id - 2 * nitems, lds);
    int blk, head, b;
    const bool dkv = HW == HD ? id < nitems : (id & 1) == 0;
    causal_item(HW != HD ? id >> 1 : dkv ? id : id - nitems, nitems, nbh, nblocks, a.ph, blk, head, b);
    if (dkv) attn_bwd_dkv_block<HW, KW, true>(a, (nblocks - 1 - blk) * Split<KW>::ROWS, head, b, lds);
    else attn_bwd_dq_block<HW, KW, false>(a, blk * Split<KW>::ROWS, head, b, lds);
}

enum CoreKernel { CORE_FWD, CORE_DQ, CORE_DKV, CORE_BWD };
template <int HW, int KW>
int launch_core(CoreKernel which, const CoreArgs& a, int nbh, const SideJobs& side, hipStream_t s) {
    const int nblocks = (a.S + Split<KW>::ROWS - 1) / Split<KW>::ROWS;
    auto grid = [&](int lds, int kernels = 1) {
        constexpr int HALVES = Split<KW>::THREADS / 256;
        const int per = side_tiles(lds / HALVES) * HALVES;
        return workgroup_grid((int64_t)nblocks * nbh * kernels + (side.end[kMaxTransposeJobs - 1] + per - 1) / per);
    };
    if constexpr (KW > 1) {
        constexpr int LDS = dq_lds<HW, KW>() > DkvShape<HW, KW>::LDS ? dq_lds<HW, KW>() : DkvShape<HW, KW>::LDS;
        if (which == CORE_BWD) {
            attn_bwd_kernel<HW, KW><<<grid(LDS, 2), Split<KW>::THREADS, 0, s>>>(a, nblocks, nbh, side);
            return launch_status();
        }
    }
    if (which == CORE_BWD) return SDP_ERR_UNSUPPORTED;
    if (which == CORE_FWD) attn_fwd_kernel<HW, KW><<<grid(fwd_lds<HW, KW>()), Split<KW>::THREADS, 0, s>>>(a, nblocks, nbh, side);
    else if (which == CORE_DQ) attn_bwd_dq_kernel<HW, KW><<<grid(dq_lds<HW, KW>()), Split<KW>::THREADS, 0, s>>>(a, nblocks, nbh, side);
    else attn_bwd_dkv_kernel<HW, KW><<<grid(DkvShape<HW, KW>::LDS), Split<KW>::THREADS, 0, s>>>(a, nblocks, nbh, side);
    return launch_status();
}
template <int HW>
int launch_core(CoreKernel which, const CoreArgs& a, int64_t nbh, const SideJobs& side, hipStream_t s) {
    if (core_blocks_128(a.S, nbh) > INT32_MAX / 2) return SDP_ERR_UNSUPPORTED;
    const int kw = core_waves(a.hd, a.S, nbh);
    if constexpr (HW > HD) {
        if (kw == 8) return launch_core<HW, 8>(which, a, (int)nbh, side, s);
    }
    return kw == 4 ? launch_core<HW, 4>(which, a, (int)nbh, side, s) : launch_core<HW, 1>(which, a, (int)nbh, side, s);
}
// the core kernel and, in its launch, n transposes
int launch_core(CoreKernel which, const CoreArgs& a, int64_t nbh, const TransposeJob* jobs, int n, const char* name, hipStream_t s) {
    SideJobs side;
    if (side_jobs(jobs, n, &side) < 0) return SDP_ERR_UNSUPPORTED;
    ProfileScope ps(name, s);
    if (a.hd <= 64) return launch_core<64>(which, a, nbh, side, s);
    if (a.hd <= 96) return launch_core<96>(which, a, nbh, side, s);
    return launch_core<128>(which, a, nbh, side, s);
}

// bf16, out and dX in launches of their own: whether they read the weights as stored (E: the columns of the heads that run).  The core's
// launch carries the transposes of small weights for nothing, and a contraction on copies is up to 1 us shorter; large ones lengthen it.
// Copies / as stored, us, forward pass: 512 tokens, d = 1024, 16 heads of 64 26.6 / 25.3, 64, d = 1536, 24 of 64 24.8 / 23.0; but 2048, d = 256,
// 2 of 64 24.6 / 25.5, 1024, d = 512, 2 of 128 26.0 / 27.2.  Backward: 256, d = 2048, 16 of 128 71.5 / 62.3, 64, d = 1536, 24 of 64 46.2 / 42.6; but
// 512, d = 1200, 12 of 50 43.1 / 46.0, 2048, d = 512, 8 of 64 64.5 / 65.5.  From 2^20 elements of WoT on 99 passes take 2 % less as stored, five
// of them 2 to 4 % more; below 194 take 0.2 % more.
bool worth_as_stored(int64_t E, int64_t d) { return E * d >= (int64_t)1 << 20; }

// rows of [Wq; Wk; Wv] ([3 H hd][d]) and of WoT ([H hd][d]) that belong to the held heads
__global__ void head_rows_kernel(const int32_t* __restrict__ head_idx, int ph, int H, int hd, int32_t* __restrict__ rows_qkv,
                                 int32_t* __restrict__ rows_o) {
    const int E = ph * hd;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 3 * E) return;
    const int part = i / E, rem = i - part * E;
    const int row = head_idx[rem / hd] * hd + rem % hd;
    rows_qkv[i] = part * H * hd + row;
    if (part == 0) rows_o[rem] = row;
}

// Token-contiguous copies, for the plain weight gradients: T tokens, zeros up to the next multiple of 8, and 64 more (see the
// MLP path: rows must not sit a power of two apart).  The room for those of O, X and dY also takes copies of them as they are,
// where an output overwrites them.
int64_t depth_tokens(int64_t T) { return (T + 7) / 8 * 8; }
int64_t ld_tokens(int64_t T, int d, int E) { return line_ld(depth_tokens(T) + 64, d > 3 * E ? d : 3 * E); }

// Columns a head takes in the saved tensors.  Bf16 heads narrower than 64 (the paper's 500M / 1B models have width
// 50) are padded to 64 with zero features: a zero feature of Q and K adds nothing to a
// logit, a zero feature of V gives a zero feature of O, and every gradient of a zero feature is zero.  The padding
// is made once, on the weights (pad_heads_kernel): the saved Q | K | V and O then carry 64 columns per head, of
// which the last 64 - hd are zero.  Wider bf16 heads are saved as they are and run the MFMA core of the next width
// (64, 96, 128), which sets the missing columns to zero as it stages them; fp32 heads go through the fp32 core (sdp_attn_f32.hip).
int core_width(int dtype, int hd) { return dtype == SDP_BF16 && hd <= HD ? HD : hd; }
bool mfma_core(int dtype) { return dtype == SDP_BF16; }
size_t esize(int dtype) { return dtype == SDP_F32 ? 4 : 2; }

// What a padded pass needs of its weights, one launch.  blockIdx.y = 0 .. 3: Wq, Wk, Wv, WoT of the n run heads, each padded
// to hw rows: out[(i hw + r)][:] = r < hd ? in[(heads ? heads[i] : i) hd + r][:] : 0 for i < n, r < hw (Wp [3][n hw][ldp], WoP
// [n hw][ldp]); d % 8 == 0, 16 bytes per thread.  blockIdx.y = 4 (backward): row lists of the weight-gradient launch, for
// padded row m = i hw + r of the ph held heads
//   gather[m]  = held[i] hw + r             (row of the all-heads operand, backward masking)
//   scatter[m] = r < hd ? (full ? held[i] : i) hd + r : -1     (output row; padding rows are dropped)
// (Three launches before, of 5 to 6 us each.)
struct PadArgs {
    const uint16_t *Wqkv, *WoT;
    uint16_t *Wp, *WoP;
    const int32_t *heads, *held; // null: every head, in order
    int n, ph, H, hd, hw, d, full;
    int64_t ldp; // of Wp, WoP
    int32_t *gather, *scatter;
};
__global__ __launch_bounds__(256) void pad_heads_kernel(PadArgs a) {
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y;
    if (y == 4) {
        if (i >= a.ph * a.hw) return;
        const int m = (int)i, k = m / a.hw, r = m % a.hw, h = a.held ? a.held[k] : k;
        a.gather[m] = h * a.hw + r;
        a.scatter[m] = r < a.hd ? (a.full ? h : k) * a.hd + r : -1;
        return;
    }
    const int chunks = a.d / 8;
    if (i >= (int64_t)a.n * a.hw * chunks) return;
    const int row = (int)(i / chunks), c = (int)(i % chunks);
    const int head = row / a.hw, r = row % a.hw;
    const int z = y < 3 ? y : 0;
    const uint16_t* in = (y < 3 ? a.Wqkv : a.WoT) + (int64_t)z * a.H * a.hd * a.d;
    uint16_t* out = (y < 3 ? a.Wp : a.WoP) + (int64_t)z * a.n * a.hw * a.ldp;
    u32x4_t v = {0u, 0u, 0u, 0u};
    if (r < a.hd) v = *(const u32x4_t*)(in + ((int64_t)(a.heads ? a.heads[head] : head) * a.hd + r) * a.d + c * 8);
    *(u32x4_t*)(out + (int64_t)row * a.ldp + c * 8) = v;
}

int check(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph) {
    if (mode != SDP_MASK_FORWARD && mode != SDP_MASK_BACKWARD) return SDP_ERR_INVALID_ARG;
    if (dtype != SDP_BF16 && dtype != SDP_F32) return SDP_ERR_INVALID_ARG;
    if (Bt < 1 || S < 1 || d < 1 || H < 1 || hd < 1) return SDP_ERR_INVALID_ARG;
    if (hd > 128) return SDP_ERR_UNSUPPORTED;
    if (ph < 1 || ph > H) return SDP_ERR_SHAPE;
    if (dtype == SDP_BF16 && (d % 8 || (hd > HD && hd % 8))) return SDP_ERR_SHAPE; // 16-byte rows; heads up to 64 are padded
    if (Bt > 65535 || H > kMaxHeads) return SDP_ERR_SHAPE;
    const int hw = core_width(dtype, hd);
    if ((int64_t)Bt * S >= ((int64_t)1 << 31) || (int64_t)Bt * S * 3 * H * hw >= ((int64_t)1 << 40)) return SDP_ERR_SHAPE;
    // padded heads: a sequence's rows span less than 4 GiB
    if (mfma_core(dtype) && hd <= HD && (int64_t)S * 3 * H * hw * 2 >= ((int64_t)1 << 32)) return SDP_ERR_SHAPE;
    return SDP_OK;
}

// heads the forward pass and the core run on: the held ones (forward masking) or all of them (backward masking)
int heads_run(int mode, int H, int ph) { return mode == SDP_MASK_FORWARD ? ph : H; }

// rows of the weight copies in the workspace: WoC [d][E], Wc [d][3 E], Wp [3 E][d], WoP [E][d]
int64_t ld_weights(size_t e, int64_t width, int64_t rows) { return e == 2 ? line_ld(width, rows) : width; }

struct FwdWs {
    int32_t *rows_qkv, *rows_o;
    void *WoC, *Wp, *WoP; // Wp, WoP: padded copies of the run heads' rows of Wqkv / WoT (padded head widths only)
    size_t bytes;
};
FwdWs fwd_ws(char* w, size_t e, int d, int E, bool padded) {
    FwdWs r;
    size_t off = 0;
    auto take = [&](size_t n) { char* p = w ? w + off : nullptr; off += round_up(n, 256); return p; };
    r.rows_qkv = (int32_t*)take((size_t)3 * E * 4);
    r.rows_o = (int32_t*)take((size_t)E * 4);
    r.WoC = take((size_t)d * ld_weights(e, E, d) * e);
    r.Wp = padded ? take((size_t)3 * E * ld_weights(e, d, 3 * E) * e) : nullptr;
    r.WoP = padded ? take((size_t)E * ld_weights(e, d, 3 * E) * e) : nullptr;
    r.bytes = off;
    return r;
}

// whether the four weight gradients are one MFMA launch that reads dQKV, O, X and dY as they are
bool direct_dw(int dtype, int d, int E) { return dtype == SDP_BF16 && gemm_depth_major_ld(3 * (int64_t)E) && gemm_depth_major_ld(d); }

struct BwdWs {
    int32_t *rows_qkv, *rows_o;
    void *dO, *dQKV, *dQKVt, *Ot, *Xt, *dYt, *Wc, *split, *Wp, *WoP;
    float* delta;
    size_t bytes;
};
// E = width the core runs on, Eh = width of the held heads (equal under forward masking), both in padded columns
BwdWs bwd_ws(char* w, size_t e, int64_t T, int d, int E, int Eh, int64_t stats, bool padded) {
    BwdWs r;
    size_t off = 0;
    auto take = [&](size_t n) { char* p = w ? w + off : nullptr; off += round_up(n, 256); return p; };
    const int64_t ldt = ld_tokens(T, d, E);
    r.rows_qkv = (int32_t*)take((size_t)3 * Eh * 4);
    r.rows_o = (int32_t*)take((size_t)Eh * 4);
    r.dO = take((size_t)T * E * e);
    r.dQKV = take((size_t)T * 3 * E * e);
    r.delta = (float*)take((size_t)stats * 4);
    r.dQKVt = e == 2 && !direct_dw(SDP_BF16, d, E) ? take((size_t)3 * E * ldt * e) : nullptr;
    r.Ot = take((size_t)E * ldt * e);
    r.Xt = take((size_t)d * ldt * e);
    r.dYt = take((size_t)d * ldt * e);
    r.Wc = take((size_t)d * ld_weights(e, 3 * E, d) * e);
    const size_t sp = e == 2 ? gemm_split_ws_bytes(Eh, d, (int)depth_tokens(T), 4) : 0; // partial sums of the batched weight-gradient launch
    r.split = sp ? take(sp) : nullptr;
    r.Wp = padded ? take((size_t)3 * E * ld_weights(e, d, 3 * E) * e) : nullptr;
    r.WoP = padded ? take((size_t)E * ld_weights(e, d, 3 * E) * e) : nullptr;
    r.bytes = off;
    return r;
}

// rows: the weight-gradient launch's lists as well
int pad_heads(const PadArgs& a, bool rows, hipStream_t s) {
    ProfileScope ps("attn_pad_w", s);
    const int64_t total = (int64_t)a.n * a.hw * (a.d / 8); // d >= 8: no fewer threads than list rows when n >= ph
    pad_heads_kernel<<<dim3((unsigned)((total + 255) / 256), rows ? 5 : 4), 256, 0, s>>>(a);
    return launch_status();
}

int run(int dtype, const GemmDesc& g, hipStream_t s) {
    if (dtype == SDP_F32) return gemm_f32(g, s);
    return gemm_mfma_supported(g) ? gemm_mfma_bf16(g, s) : gemm_simple(g, s);
}

int head_rows(const int32_t* head_idx, int ph, int H, int hd, int32_t* rows_qkv, int32_t* rows_o, hipStream_t s) {
    ProfileScope ps("attn_rows", s);
    const int n = 3 * ph * hd;
    head_rows_kernel<<<(n + 255) / 256, 256, 0, s>>>(head_idx, ph, H, hd, rows_qkv, rows_o);
    return launch_status();
}

} // namespace
} // namespace sdp

using namespace sdp;

extern "C" int sdp_masked_attn_saved_head_width(int dtype, int hd) {
    if ((dtype != SDP_BF16 && dtype != SDP_F32) || hd < 1 || hd > 128) return 0;
    return core_width(dtype, hd);
}

extern "C" size_t sdp_masked_attn_fwd_workspace_bytes(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph) {
    if (check(mode, dtype, Bt, S, d, H, hd, ph) != SDP_OK) return 0;
    const int hw = core_width(dtype, hd);
    return fwd_ws(nullptr, esize(dtype), d, heads_run(mode, H, ph) * hw, hw != hd).bytes;
}

extern "C" size_t sdp_masked_attn_bwd_workspace_bytes(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph) {
    if (check(mode, dtype, Bt, S, d, H, hd, ph) != SDP_OK) return 0;
    const int hr = heads_run(mode, H, ph), hw = core_width(dtype, hd);
    return bwd_ws(nullptr, esize(dtype), (int64_t)Bt * S, d, hr * hw, ph * hw, (int64_t)Bt * hr * S, hw != hd).bytes;
}

extern "C" int sdp_masked_attn_fwd(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph, const void* X,
                                   const void* Wqkv, const void* WoT, const int32_t* head_idx_k, void* Y, void* QKV_save,
                                   void* O_save, float* LSE_save, void* ws, size_t ws_bytes, void* stream) {
    if (mode == SDP_MASK_BACKWARD) ph = H; // the forward pass is the dense block; the list is not looked at
    int rc = check(mode, dtype, Bt, S, d, H, hd, ph);
    if (rc != SDP_OK) return rc;
    if (!X || !Wqkv || !WoT || !Y || !QKV_save || !O_save || !LSE_save) return SDP_ERR_INVALID_ARG;
    if (mode == SDP_MASK_FORWARD && !head_idx_k) return SDP_ERR_INVALID_ARG;
    for (const void* q : {X, Wqkv, WoT, (const void*)Y, (const void*)QKV_save, (const void*)O_save, (const void*)LSE_save})
        if (!aligned16(q)) return SDP_ERR_INVALID_ARG;
    if (!ws || !aligned16(ws) || ws_bytes < sdp_masked_attn_fwd_workspace_bytes(mode, dtype, Bt, S, d, H, hd, ph))
        return SDP_ERR_WORKSPACE;
    return attn_fwd_impl(mode, dtype, Bt, S, d, H, hd, ph, X, Wqkv, WoT, head_idx_k, Y, QKV_save, O_save, LSE_save, nullptr,
                         ws, (hipStream_t)stream);
}

int sdp::attn_fwd_impl(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph, const void* X, const void* Wqkv,
                       const void* WoT, const int32_t* head_idx_k, void* Y, void* QKV_save, void* O_save, float* LSE_save,
                       const void* residual, void* ws, hipStream_t s) {
    if (mode == SDP_MASK_BACKWARD) ph = H;
    int rc;
    const bool gathered = mode == SDP_MASK_FORWARD;
    const int hw = core_width(dtype, hd); // columns per head in the saved tensors
    const bool padded = hw != hd;
    const int T = Bt * S, E = ph * hw;
    const FwdWs w = fwd_ws((char*)ws, esize(dtype), d, E, padded);
    const int64_t ldp = padded ? ld_weights(2, d, 3 * E) : d, ldo = ld_weights(esize(dtype), E, d); // rows of Wp / WoP, of WoC

    // rows of the held heads: bf16 from the list of heads itself, fp32 from lists of rows
    const HeadList heads = dtype == SDP_BF16 ? head_list(hd, ph, H) : HeadList{};
    if (gathered && dtype == SDP_F32) {
        rc = head_rows(head_idx_k, ph, H, hd, w.rows_qkv, w.rows_o, s);
        if (rc != SDP_OK) return rc;
    }
    const int32_t* rows_qkv = !gathered || padded ? nullptr : dtype == SDP_BF16 ? head_idx_k : w.rows_qkv;
    const int32_t* rows_o = !gathered || padded ? nullptr : dtype == SDP_BF16 ? head_idx_k : w.rows_o;
    if (padded) { // the run heads' rows of W_Q, W_K, W_V and W_O, each head padded to hw rows
        const PadArgs pa{(const uint16_t*)Wqkv, (const uint16_t*)WoT, (uint16_t*)w.Wp, (uint16_t*)w.WoP,
                         gathered ? head_idx_k : nullptr, nullptr, ph, ph, H, hd, hw, d, 0, ldp, nullptr, nullptr};
        rc = pad_heads(pa, false, s);
        if (rc != SDP_OK) return rc;
    }

    GemmDesc pj;
    pj.name = "attn_qkv";
    pj.M = T, pj.N = 3 * E, pj.K = d;
    pj.A = X, pj.lda = d;
    pj.B = padded ? w.Wp : Wqkv, pj.ldb = ldp;
    if (rows_qkv) pj.b_gather = rows_qkv, pj.b_rows = (int64_t)3 * H * hd, pj.heads = heads;
    pj.epilogue = EPI_STORE;
    pj.C = QKV_save, pj.ldc = 3 * E;
    rc = run(dtype, pj, s);
    if (rc != SDP_OK) return rc;

    GemmDesc op;
    op.name = "attn_out";
    op.M = T, op.N = d, op.K = E;
    op.A = O_save, op.lda = E;
    op.epilogue = EPI_STORE;
    op.C = Y, op.ldc = d;
    op.R = residual, op.ldr = d;
    // bf16: WoT as it is stored (padded: its copy) where the contraction takes it so and no output takes its place
    GemmDesc as_stored = op;
    as_stored.B = padded ? w.WoP : WoT, as_stored.ldb = ldp, as_stored.b_km = 1;
    as_stored.b_gather = rows_o, as_stored.b_rows = rows_o ? (int64_t)H * hd : E, as_stored.heads = heads;
    const bool stored = dtype == SDP_BF16 && worth_as_stored(E, d) && gemm_reads_as_stored(as_stored) &&
                        (padded || !overlap({{Y, (size_t)T * d * 2}, {O_save, (size_t)T * E * 2}, {LSE_save, (size_t)Bt * ph * S * 4}},
                                            {{WoT, (size_t)H * hd * d * 2}}));

    if (mfma_core(dtype)) {
        CoreArgs a{};
        a.qkv = (const uint16_t*)QKV_save, a.ldq = 3 * E;
        a.o_out = (uint16_t*)O_save, a.ldo = E;
        a.lse = LSE_save;
        a.S = S, a.ph = ph, a.hd = hw;
        a.scale = 1.f / sqrtf((float)hd), a.scale2 = a.scale * 1.44269504088896340736f;
        const TransposeJob wt{padded ? w.WoP : WoT, w.WoC, ldp, ldo, rows_o, E, d, heads};
        rc = launch_core(CORE_FWD, a, (int64_t)ph * Bt, &wt, stored ? 0 : 1, "attn_core_fwd", s);
    } else {
        AttnCoreDesc c;
        c.qkv = QKV_save, c.ldq = 3 * E, c.o_out = O_save, c.ldo = E, c.lse = LSE_save;
        c.Bt = Bt, c.S = S, c.n = ph, c.hd = hd;
        rc = attn_f32_fwd(c, s);
    }
    if (rc != SDP_OK) return rc;
    if (stored) return run(dtype, as_stored, s);

    // fp32 reads WoT itself: an output that takes its place needs a copy
    const int32_t* wo_rows = rows_o;
    if (dtype == SDP_F32 && overlap({{Y, (size_t)T * d * 4}}, {{WoT, (size_t)H * hd * d * 4}})) {
        rc = copy_rows_f32((const float*)WoT, wo_rows, E, d, (float*)w.WoC, "attn_wt_fwd", s);
        if (rc != SDP_OK) return rc;
        WoT = w.WoC, wo_rows = nullptr;
    }
    if (dtype == SDP_BF16) op.B = w.WoC, op.ldb = ldo;
    else op.B = WoT, op.ldb = d, op.b_km = 1, op.b_gather = wo_rows, op.b_rows = wo_rows ? (int64_t)H * hd : E;
    return run(dtype, op, s);
}

extern "C" int sdp_masked_attn_bwd(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph, const void* X,
                                   const void* dY, const void* Wqkv, const void* WoT, const int32_t* head_idx_k,
                                   const void* QKV_save, const void* O_save, const float* LSE_save, void* dX, void* dWqkv,
                                   void* dWoT, int dw_layout, void* ws, size_t ws_bytes, void* stream) {
    int rc = check(mode, dtype, Bt, S, d, H, hd, ph);
    if (rc != SDP_OK) return rc;
    if (dw_layout != SDP_DW_COMPACT && dw_layout != SDP_DW_SCATTER) return SDP_ERR_INVALID_ARG;
    if (!X || !dY || !Wqkv || !WoT || !head_idx_k || !QKV_save || !O_save || !LSE_save || !dX || !dWqkv || !dWoT)
        return SDP_ERR_INVALID_ARG;
    for (const void* q : {X, dY, Wqkv, WoT, QKV_save, O_save, (const void*)LSE_save, (const void*)dX, (const void*)dWqkv,
                          (const void*)dWoT})
        if (!aligned16(q)) return SDP_ERR_INVALID_ARG;
    if (!ws || !aligned16(ws) || ws_bytes < sdp_masked_attn_bwd_workspace_bytes(mode, dtype, Bt, S, d, H, hd, ph))
        return SDP_ERR_WORKSPACE;
    return attn_bwd_impl(mode, dtype, Bt, S, d, H, hd, ph, X, dY, Wqkv, WoT, head_idx_k, QKV_save, O_save, LSE_save, dX,
                         dWqkv, dWoT, dw_layout, nullptr, true, ws, (hipStream_t)stream);
}

int sdp::attn_bwd_impl(int mode, int dtype, int Bt, int S, int d, int H, int hd, int ph, const void* X, const void* dY,
                       const void* Wqkv, const void* WoT, const int32_t* head_idx_k, const void* QKV_save,
                       const void* O_save, const float* LSE_save, void* dX, void* dWqkv, void* dWoT, int dw_layout,
                       const void* dx_residual, bool want_dw, void* ws, hipStream_t s) {
    int rc;
    const bool gathered = mode == SDP_MASK_FORWARD;
    const int hr = heads_run(mode, H, ph);
    const int hw = core_width(dtype, hd);
    const bool padded = hw != hd;
    const int T = Bt * S, E = hr * hw, Eh = ph * hw; // width the core runs on, width of the held heads (padded columns)
    const BwdWs w = bwd_ws((char*)ws, esize(dtype), T, d, E, Eh, (int64_t)Bt * hr * S, padded);
    const int64_t ldp = padded ? ld_weights(2, d, 3 * E) : d, ldw = ld_weights(esize(dtype), 3 * E, d); // rows of Wp / WoP, of Wc
    // no list under backward masking: every head is held (ph = H), no row gather and no scatter are needed
    const bool all_heads = !gathered && head_idx_k == nullptr;

    if (padded) {
        // with the rows of the held heads in the padded operands, and where each of them goes (padding rows: nowhere)
        const PadArgs pa{(const uint16_t*)Wqkv, (const uint16_t*)WoT, (uint16_t*)w.Wp, (uint16_t*)w.WoP,
                         gathered ? head_idx_k : nullptr, head_idx_k, hr, ph, H, hd, hw, d, dw_layout == SDP_DW_SCATTER, ldp, w.rows_o,
                         w.rows_qkv};
        rc = pad_heads(pa, want_dw, s);
        if (rc != SDP_OK) return rc;
    } else if (!all_heads && dtype == SDP_F32) {
        rc = head_rows(head_idx_k, ph, H, hd, w.rows_qkv, w.rows_o, s);
        if (rc != SDP_OK) return rc;
    }
    // rows of the held heads: padded, the lists just made; bf16, from the list of heads itself; fp32, lists of rows
    const HeadList heads = dtype == SDP_BF16 && !padded ? head_list(hd, ph, H) : HeadList{};
    const int32_t* rows_qkv = dtype == SDP_BF16 && !padded ? head_idx_k : w.rows_qkv;
    const int32_t* rows_o = dtype == SDP_BF16 && !padded ? head_idx_k : w.rows_o;

    // bf16: the four weight gradients share one shape (Eh x d, depth T): dWq, dWk, dWv from the three column blocks of dQKV and
    // X, dWoT from O and dY; one batched launch fills the CUs four times better than four would, and reads all of these as
    // they are stored, depth-major.  (With token-contiguous copies, made beside the core and, of dK and dV, in a launch of their
    // own: block of 4 x 2048 tokens, 12 of 24 heads of 64 432 us, this way 398; 12 of 24 heads of 50, backward masking 666, 610;
    // both ways on one box, of which others are up to 5 % slower.)
    // Under backward masking the blocks hold all heads and the launch reads the held heads' columns only: the gradient is
    // computed on the mask.
    const int64_t part = (int64_t)(dw_layout == SDP_DW_SCATTER ? H * hd : ph * hd) * d; // elements of one weight gradient
    GemmDesc wg;
    const bool direct = want_dw && direct_dw(dtype, d, E);
    if (dtype == SDP_BF16 && want_dw) {
        wg.name = "attn_dw";
        wg.M = Eh, wg.N = d, wg.K = T;
        wg.a_km = wg.b_km = 1;
        wg.lda = 3 * E, wg.ldb = d;
        if (!gathered && !all_heads) wg.a_gather = rows_o, wg.a_rows = E, wg.a_gather_chunks = 1; // heads of a multiple of 8
        wg.epilogue = EPI_STORE;
        wg.ldc = d;
        // rows of the held heads inside each matrix; padded heads: w.rows_o = the held heads' columns of the operands, w.rows_qkv =
        // output rows (-1: dropped)
        wg.c_scatter = padded ? w.rows_qkv : dw_layout == SDP_DW_SCATTER && !all_heads ? rows_o : nullptr;
        wg.heads = heads;
        if (padded && !gathered) wg.a_gather = w.rows_o, wg.a_rows = E, wg.a_gather_chunks = 1;
        wg.nbatch = 4;
        for (int i = 0; i < 3; ++i)
            wg.Ab[i] = (const uint16_t*)w.dQKV + (int64_t)i * E, wg.Bb[i] = X, wg.Cb[i] = (uint16_t*)dWqkv + (size_t)i * part;
        wg.Ab[3] = O_save, wg.ldab[3] = E, wg.Bb[3] = dY, wg.Cb[3] = dWoT;
        wg.split_ws = w.split;
    }

    GemmDesc go;
    go.name = "attn_dout";
    go.M = T, go.N = E, go.K = d;
    go.A = dY, go.lda = d;
    go.B = padded ? w.WoP : WoT, go.ldb = ldp;
    if (gathered && !padded) go.b_gather = rows_o, go.b_rows = (int64_t)H * hd, go.heads = heads;
    go.epilogue = EPI_STORE;
    go.C = w.dO, go.ldc = E;
    rc = run(dtype, go, s);
    if (rc != SDP_OK) return rc;

    GemmDesc dx;
    dx.name = "attn_dx";
    dx.M = T, dx.N = d, dx.K = 3 * E;
    dx.A = w.dQKV, dx.lda = 3 * E;
    dx.epilogue = EPI_STORE;
    dx.C = dX, dx.ldc = d;
    dx.R = dx_residual, dx.ldr = d;
    // bf16: Wqkv as it is stored (padded: its copy) where the contraction takes it so and no output takes its place
    const bool listed = gathered && !padded;
    const size_t dwp_b = want_dw ? (size_t)part * 2 : 0;
    GemmDesc as_stored = dx;
    as_stored.B = padded ? w.Wp : Wqkv, as_stored.ldb = ldp, as_stored.b_km = 1;
    as_stored.b_gather = listed ? rows_qkv : nullptr, as_stored.b_rows = listed ? (int64_t)3 * H * hd : 3 * E, as_stored.heads = heads;
    const bool apart = dtype == SDP_BF16 &&
                       (padded || !overlap({{dX, (size_t)T * d * 2}, {dWqkv, 3 * dwp_b}, {dWoT, dwp_b}}, {{Wqkv, (size_t)3 * H * hd * d * 2}}));
    // and in the launch of the weight gradients, where dX does not take the place of what those read
    const bool pair = direct && apart && gemm_pairs(as_stored, wg) &&
                      !overlap({{dX, (size_t)T * d * 2}}, {{X, (size_t)T * d * 2}, {dY, (size_t)T * d * 2}, {O_save, (size_t)T * E * 2}});
    const bool stored = pair || (apart && worth_as_stored(E, d) && gemm_reads_as_stored(as_stored));
    if (mfma_core(dtype)) {
        CoreArgs a{};
        a.qkv = (const uint16_t*)QKV_save, a.ldq = 3 * E;
        a.o = (const uint16_t*)O_save, a.dO = (const uint16_t*)w.dO, a.ldo = E;
        a.lse = const_cast<float*>(LSE_save), a.delta = w.delta;
        a.dqkv = (uint16_t*)w.dQKV;
        a.S = S, a.ph = hr, a.hd = hw;
        a.scale = 1.f / sqrtf((float)hd), a.scale2 = a.scale * 1.44269504088896340736f;
        // Wqkv's rows for dX; token-contiguous copies for the plain weight gradients
        const int64_t ldt = ld_tokens(T, d, E);
        const TransposeJob beside_dq[4] = {{padded ? w.Wp : Wqkv, w.Wc, ldp, ldw, listed ? rows_qkv : nullptr, 3 * E, d, heads},
                                           {O_save, w.Ot, E, ldt, nullptr, T, E},
                                           {X, w.Xt, d, ldt, nullptr, T, d},
                                           {dY, w.dYt, d, ldt, nullptr, T, d}};
        const TransposeJob beside_dkv{w.dQKV, w.dQKVt, 3 * E, ldt, nullptr, T, E}; // dQ
        const int skip = stored ? 1 : 0; // dX needs no copy of Wqkv
        const bool one = core_merged_backward(a.hd, a.S, (int64_t)hr * Bt) && (direct || !want_dw);
        rc = launch_core(one ? CORE_BWD : CORE_DQ, a, (int64_t)hr * Bt, beside_dq + skip, (want_dw && !direct ? 4 : 1) - skip,
                         one ? "attn_core_bwd" : "attn_core_bwd_dq", s);
        // reads the delta written by the dQ kernel
        if (rc == SDP_OK && !one) rc = launch_core(CORE_DKV, a, (int64_t)hr * Bt, &beside_dkv, want_dw && !direct ? 1 : 0, "attn_core_bwd_dkv", s);
        if (rc != SDP_OK) return rc;
    } else {
        AttnCoreDesc c;
        c.qkv = QKV_save, c.ldq = 3 * E, c.o = O_save, c.dO = w.dO, c.ldo = E;
        c.lse = const_cast<float*>(LSE_save), c.delta = w.delta, c.dqkv = w.dQKV;
        c.Bt = Bt, c.S = S, c.n = hr, c.hd = hd;
        rc = attn_f32_bwd(c, s);
        if (rc != SDP_OK) return rc;
    }

    const int32_t* w_rows = gathered ? w.rows_qkv : nullptr;
    if (dtype == SDP_F32) {
        // What follows reads Wqkv, X, dY and O_save as they are; where an output takes the place of one of these (dX over dY, a
        // gradient over its weights), copies of them.
        const size_t tok_b = (size_t)T * d * 4, dw_b = (size_t)part * 4;
        const Extent x{X, tok_b}, dy{dY, tok_b}, o{O_save, (size_t)T * E * 4}, wq{Wqkv, (size_t)3 * H * hd * d * 4}, ox{dX, tok_b};
        if (want_dw ? overlap({ox, {dWqkv, 3 * dw_b}, {dWoT, dw_b}}, {x, dy, o, wq}) : overlap({ox}, {wq})) {
            const struct { const void* in; const int32_t* rows; int R, C; void* out; } copies[4] = {
                {Wqkv, w_rows, 3 * E, d, w.Wc}, {X, nullptr, T, d, w.Xt}, {dY, nullptr, T, d, w.dYt}, {O_save, nullptr, T, E, w.Ot}};
            for (int i = 0; i < (want_dw ? 4 : 1); ++i) {
                rc = copy_rows_f32((const float*)copies[i].in, copies[i].rows, copies[i].R, copies[i].C, (float*)copies[i].out,
                                   "attn_copy_bwd", s);
                if (rc != SDP_OK) return rc;
            }
            Wqkv = w.Wc, X = w.Xt, dY = w.dYt, O_save = w.Ot, w_rows = nullptr;
        }
    }

    if (dtype == SDP_BF16 && stored) dx = as_stored;
    else if (dtype == SDP_BF16) dx.B = w.Wc, dx.ldb = ldw;
    else dx.B = Wqkv, dx.ldb = d, dx.b_km = 1, dx.b_gather = w_rows, dx.b_rows = w_rows ? (int64_t)3 * H * hd : 3 * E;
    if (!want_dw) return run(dtype, dx, s);

    if (dtype == SDP_F32) { // every operand as it is stored: dQKV, O, X, dY depth-major, the held heads' columns by their list
        GemmDesc all[3];
        GemmDesc &dw = all[1], &dwo = all[2];
        dw.name = "attn_dw";
        dw.M = Eh, dw.N = d, dw.K = T;
        dw.lda = 3 * E, dw.a_km = 1;
        if (!gathered && !all_heads) dw.a_gather = w.rows_o, dw.a_rows = E, dw.a_gather_chunks = hd % 8 == 0;
        dw.ldb = d, dw.b_km = 1;
        dw.epilogue = EPI_STORE;
        dw.ldc = d;
        dw.c_scatter = dw_layout == SDP_DW_SCATTER && !all_heads ? w.rows_o : nullptr;
        dwo = dw;
        dwo.lda = E;
        dwo.A = O_save, dwo.B = dY, dwo.C = dWoT;
        dw.nbatch = 3;
        for (int i = 0; i < 3; ++i)
            dw.Ab[i] = (const float*)w.dQKV + (int64_t)i * E, dw.Bb[i] = X, dw.Cb[i] = (float*)dWqkv + i * part;
        all[0] = dx;
        rc = gemm_f32_group(all, 3, "attn_dx_dw", s);
        if (rc != SDP_ERR_UNSUPPORTED) return rc;
        rc = gemm_f32(dw, s);
        if (rc == SDP_OK) rc = gemm_f32(dwo, s);
        return rc != SDP_OK ? rc : gemm_f32(dx, s);
    }

    if (direct) {
        // a gradient in the place of X, dY or O: the launch reads copies of those
        const size_t tok_b = (size_t)T * d * 2, dw_b = (size_t)part * 2;
        if (overlap({{dWqkv, 3 * dw_b}, {dWoT, dw_b}}, {{X, tok_b}, {dY, tok_b}, {O_save, (size_t)T * E * 2}})) {
            const struct { const void* in; int C; void* out; } copies[3] = {{X, d, w.Xt}, {dY, d, w.dYt}, {O_save, E, w.Ot}};
            for (const auto& c : copies) { // d % 8 == 0, E % 8 == 0: rows of bf16 as rows of half as many floats
                rc = copy_rows_f32((const float*)c.in, nullptr, T, c.C / 2, (float*)c.out, "attn_copy_bwd", s);
                if (rc != SDP_OK) return rc;
            }
            wg.Bb[0] = wg.Bb[1] = wg.Bb[2] = w.Xt, wg.Bb[3] = w.dYt, wg.Ab[3] = w.Ot;
            if (dx_residual == dY) dx.R = w.dYt;
        }
        if (pair) return gemm_mfma_pair(dx, wg, "attn_dx_dw", s);
        rc = gemm_mfma_bf16(wg, s);
        return rc != SDP_OK ? rc : run(dtype, dx, s);
    }
    // plain weight gradients from token-contiguous copies: dK, dV; the others were made beside the core
    const int64_t ldt = ld_tokens(T, d, E);
    rc = transpose_rows((const uint16_t*)w.dQKV + E, 3 * E, nullptr, T, 2 * E, (uint16_t*)w.dQKVt + (size_t)E * ldt, ldt, "attn_tr_bwd", s);
    if (rc != SDP_OK) return rc;
    wg.nbatch = 0;
    wg.a_km = wg.b_km = 0;
    wg.K = (int)depth_tokens(T); // zeros from T on (transpose_rows_vec_kernel)
    wg.lda = wg.ldb = ldt;
    for (int i = 0; i < 4; ++i) {
        wg.A = i < 3 ? (const uint16_t*)w.dQKVt + (size_t)i * E * ldt : (const uint16_t*)w.Ot;
        wg.B = i < 3 ? w.Xt : w.dYt, wg.C = wg.Cb[i];
        rc = gemm_simple(wg, s);
        if (rc != SDP_OK) return rc;
    }
    return run(dtype, dx, s);
}
