// fp32 contraction on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation), with the SwiGLU
// epilogues: the fp32 path of the masked MLP and of the attention projections.  Any M, N, K >= 1.
//
//   C[M][N] = sum_k A(m,k) B(k,n); each operand is read as it is stored, so no transposed or compacted copy is made:
//     rows   : row r of the operand is contiguous along the depth (optional gather of rows)
//     depth-major : depth step k is contiguous along the rows (B: optional gather of depth steps, which is how a list
//              of neurons or heads restricts a depth; A: optional gather of columns, the same for the weight gradients)
//
// What bounds it: the matrix cores give 157 TFLOP/s (a plain fp32 FMA half of that), i.e. 32 cycles per 16x16x4 tile, so
// operand traffic is cheap here (a wave reads 4 KB of LDS per 512 matrix cycles) and the shapes that use fp32 are small:
// latency, launches and idle CUs decide.  Hence four loops:
//   64 x 64 outputs a workgroup whose operands are split into three bf16 terms (gemm_f32_split_kernel, sdp_f32_split.h): where it is the
//   faster one (split_pays), which takes depth and tiles;
//   64 x 64 outputs a workgroup, pipelined (gemm_f32_pipe_kernel): where these fill the CUs;
//   16 x 16 and 32 x 32 outputs a workgroup, whose four waves split the depth (gemm_f32_wave_kernel): launches of few tiles;
//   32 x 32 with the depth split inside each step of 64 (gemm_f32_kernel): between these; and 64 and 128 wide, the largest launches
//   and those that read a list beyond kListMax where the split does not pay.
// The pipelined and the wave-split loops fill LDS by direct loads, 16 bytes a lane or, where extents or strides are no multiples of 4 or
// columns are gathered, 4; the split and the last move global -> registers -> LDS.
//
// A depth slot is free to stand for any k as long as both operands agree: in a group of 16 depth steps, lane group
// g = lane / 16 takes k = 4 g + j in the j-th of four MFMAs, so an operand stored by rows is one 16-byte LDS read per
// 16 x 16 fragment, a depth-major one four 4-byte reads; row strides of 4 (mod 16) words keep both free of conflicts.
//
// Measured: four workers' steps at T = 256, d = 256, F = 1024, p = 512 (twelve launches a worker with a plain FMA kernel
// and transposed copies before, five with this loop): 2079 -> 165 us, and 139 with the 16 x 16 tiles and dX and the weight
// gradients as one launch (four a worker; 101 us since the host calls are compiled, 99 with gradients in one LDS stage and the index
// without a chain); per launch 5 - 10 us, of which about 4 us is what an empty kernel takes.
// (206 us while every step waited for the newest list entry, computed clamped 64-bit addresses per load and branched around its
// loads, so that the loads in flight could not be counted.)
#include "sdp_internal.h"
#include "sdp_swiglu.h"

#include <cmath>
#include <type_traits>

namespace sdp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct Dev {
    int M, N, K;
    const float *A, *A2, *B, *B2;
    int64_t lda, ldb;
    const int32_t *ag, *bg, *cs;
    int runs; // ag's entries come in runs of eight
    float *C, *C2, *C3;
    int64_t ldc;
    const float *Gin, *Uin;
    int64_t ldg;
    const float* R;
    int64_t ldr;
    int vec_out; // 16-byte epilogue accesses
    int nbatch, tiles_m, tiles_n;
    const float *Ab[kMaxBatch], *Bb[kMaxBatch];
    float* Cb[kMaxBatch];
};

template <int BM_, int BN_, int KSPLIT_>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_, KSPLIT = KSPLIT_; // KSPLIT waves share a tile's depth
    static constexpr int BK = KSPLIT == 1 ? 32 : 16 * KSPLIT;
    static constexpr int WM = KSPLIT == 1 ? BM / 2 : BM, WN = KSPLIT == 1 ? BN / 2 : BN; // a wave's part
    static constexpr int FM = WM / 16, FN = WN / 16;
    static constexpr int AHEAD = BM >= 128 ? 1 : 3; // steps in registers beyond the one in LDS
};

// One operand's tile: R rows (M or N side) x BK depth.
template <int R, int BK, bool DM>
struct Operand {
    static constexpr int LD = DM ? R + 4 : BK + 4;               // LDS row stride in floats
    static constexpr int FLOATS = DM ? BK * LD : R * LD;
    static constexpr int Q = DM ? R / 4 : BK / 4;                // 4-float pieces per LDS row
    static constexpr int PER = R * BK / 4 / 256;                 // pieces per thread
    static constexpr int STEP = 256 / Q;                         // LDS rows between a thread's pieces
};

// Where a thread's pieces of an operand come from.  VEC: 16-byte loads (aligned bases and strides, extents along the
// contiguous axis multiples of 4), else single elements.  Rows beyond the matrix are clamped (their products are never
// stored).  The depth needs no clamp per load: a tile that would reach beyond it starts at K - BK instead and the depth
// steps that an earlier tile has had (all of them, for tiles beyond the last) become zeros on the way to LDS; only a
// depth shorter than one tile clamps, once.  A load's address is then one 64-bit add to a pointer kept per piece: the
// loop has one wave per SIMD on small launches, and address arithmetic would cost it as much as the MFMAs.
template <int R, int BK, bool DM, int SETS, bool VEC>
struct Source {
    typedef Operand<R, BK, DM> Op;
    const float* p[Op::PER]; // each piece's row of the tile at depth 0 (depth-major: its depth step, first column)
    const float* base;
    uint32_t ld;
    const int32_t* kg; // depth-major: gather of depth steps
    int off[4];        // single loads: the piece's elements, relative to p
    int K, q4, r0, col0;
    int kidx[SETS][DM ? Op::PER : 1]; // gathered depth steps of the next tile of each register set

    __device__ int start(int k0) const { // depth at which the tile nominally at k0 is read
        const int last = K > BK ? K - BK : 0;
        return k0 < last ? k0 : last;
    }
    __device__ void init(const float* base_, int64_t ld_, int rows, int row0, int K_, const int32_t* gather_rows,
                         const int32_t* gather_depth, int tid) {
        base = base_, ld = (uint32_t)ld_, K = K_, kg = gather_depth;
        q4 = (tid % Op::Q) * 4, r0 = tid / Op::Q;
        const int kmax = K - 1;
        if constexpr (DM) {
            int col[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int c = row0 + q4 + j;
                c = c < rows ? c : (VEC ? rows - 4 + j : rows - 1);
                col[j] = !VEC && gather_rows ? gather_rows[c] : c;
                off[j] = col[j] - col[0];
            }
            col0 = col[0];
#pragma unroll
            for (int i = 0; i < Op::PER; ++i) {
                const int k = r0 + Op::STEP * i;
                p[i] = base + (int64_t)(k < kmax ? k : kmax) * ld_ + col0;
            }
        } else {
            const int k = VEC ? (q4 < K ? q4 : K - 4) : (q4 < kmax ? q4 : kmax);
#pragma unroll
            for (int j = 0; j < 4; ++j) off[j] = (q4 + j < kmax ? q4 + j : kmax) - k;
#pragma unroll
            for (int i = 0; i < Op::PER; ++i) {
                int r = row0 + r0 + Op::STEP * i;
                r = r < rows ? r : rows - 1;
                p[i] = base + (int64_t)(gather_rows ? gather_rows[r] : r) * ld_ + k;
            }
        }
    }
    __device__ void list(int set, int k0) { // list entries of the tile at depth k0
        if constexpr (DM) {
            if (kg) {
                const int32_t* q = kg + start(k0);
#pragma unroll
                for (int i = 0; i < Op::PER; ++i) {
                    const int k = r0 + Op::STEP * i;
                    kidx[set][i] = q[k < K ? k : K - 1];
                }
            }
        }
    }
    __device__ void fetch(f32x4 (&v)[Op::PER], int set, int k0) {
        const int64_t shift = DM ? (int64_t)start(k0) * ld : start(k0);
#pragma unroll
        for (int i = 0; i < Op::PER; ++i) {
            const float* q = p[i] + shift;
            if (DM && kg) q = base + ((uint64_t)(uint32_t)kidx[set][i] * ld + col0);
            if (VEC) v[i] = *(const f32x4*)q;
            else v[i] = f32x4{q[off[0]], q[off[1]], q[off[2]], q[off[3]]};
        }
    }
    // registers -> LDS
    __device__ void stash(float* lds, const f32x4 (&v)[Op::PER], int k0) const {
#pragma unroll
        for (int i = 0; i < Op::PER; ++i) {
            f32x4 w = v[i];
            if (k0 + BK > K) { // uniform: a shifted or short tile
                const int k = start(k0) + (DM ? r0 + Op::STEP * i : q4);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int kj = DM ? k : k + j;
                    w[j] = kj >= k0 && kj < K ? w[j] : 0.f;
                }
            }
            *(f32x4*)(lds + (r0 + Op::STEP * i) * Op::LD + q4) = w;
        }
    }
};

// fragment of 16 rows at depth 16 t: element j belongs to depth 16 t + 4 g + j
template <int R, int BK, bool DM>
__device__ inline f32x4 fragment(const float* lds, int row, int t, int g) {
    constexpr int LD = Operand<R, BK, DM>::LD;
    if constexpr (DM) {
        const float* p = lds + (16 * t + 4 * g) * LD + row;
        return f32x4{p[0], p[LD], p[2 * LD], p[3 * LD]};
    } else {
        return *(const f32x4*)(lds + row * LD + 16 * t + 4 * g);
    }
}

// columns n .. n + 3 of row m of a matrix of the outputs' extents, zeros outside
__device__ inline f32x4 row_of_four(const Dev& g, const float* base, int64_t ld, int m, int n) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (m >= g.M || n >= g.N) return x;
    const float* p = base + (int64_t)m * ld + n;
    if (g.vec_out) return *(const f32x4*)p;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (n + e < g.N) x[e] = p[e];
    return x;
}

// epilogue of four consecutive columns n .. n + 3 of row m; FROM: those from `lo` on (vec_out: lo - n is a multiple of 4);
// gu: G and U there, where they have been read already
template <int EPI, bool FROM = false>
__device__ inline void emit(const Dev& g, float* gC, int m, int n, f32x4 v, f32x4 v2, int lo = 0, const f32x4* gu = nullptr) {
    if (m >= g.M || n >= g.N || (FROM && n + 3 < lo)) return;
    const int cnt = g.N - n < 4 ? g.N - n : 4;
    auto put = [&](float* base, int64_t row, int64_t ld, f32x4 x) {
        float* p = base + row * ld + n;
        if (g.vec_out) *(f32x4*)p = x;
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < cnt && (!FROM || n + e >= lo)) p[e] = x[e];
        }
    };
    auto get = [&](const float* base, int64_t ld) { return row_of_four(g, base, ld, m, n); };
    if (EPI == EPI_STORE || EPI == EPI_DUAL_ACC) {
        const int64_t row = g.cs ? g.cs[m] : m;
        if (row < 0) return; // dropped row
        if (g.R) v += get(g.R, g.ldr);
        put(gC, row, g.ldc, v);
    } else if (EPI == EPI_SWIGLU_FWD) {
        put(g.C, m, g.ldc, v);
        put(g.C2, m, g.ldc, v2);
        f32x4 act;
#pragma unroll
        for (int e = 0; e < 4; ++e) act[e] = swiglu_fwd<true>(v[e], v2[e]);
        put(g.C3, m, g.ldc, act);
    } else {
        const f32x4 gv = gu ? gu[0] : get(g.Gin, g.ldg), uv = gu ? gu[1] : get(g.Uin, g.ldg);
        f32x4 dg, du, act;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float a, b, c;
            swiglu_bwd<true>(v[e], gv[e], uv[e], a, b, c);
            dg[e] = a, du[e] = b, act[e] = c;
        }
        put(g.C, m, g.ldc, dg);
        put(g.C2, m, g.ldc, du);
        put(g.C3, m, g.ldc, act);
    }
}

template <class C, int EPI, bool ADM, bool BDM, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(Dev g) {
    constexpr int BM = C::BM, BN = C::BN, BK = C::BK, FM = C::FM, FN = C::FN, AHEAD = C::AHEAD;
    constexpr bool kTwoB = EPI == EPI_SWIGLU_FWD;
    typedef Operand<BM, BK, ADM> OA;
    typedef Operand<BN, BK, BDM> OB;
    constexpr int NB = kTwoB ? 2 : 1, STAGE = OA::FLOATS + NB * OB::FLOATS;
    extern __shared__ __attribute__((aligned(16))) float smem[]; // two stages of A, B (, B2)

    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = g.tiles_m * g.tiles_n;
    const int z = blockIdx.x / per, tile = blockIdx.x - z * per;
    const int m0 = (tile % g.tiles_m) * BM, n0 = (tile / g.tiles_m) * BN;
    const float *gA = g.A, *gB = g.B;
    float* gC = g.C;
    if (g.nbatch > 0) {
        gA = z == 0 ? g.Ab[0] : (z == 1 ? g.Ab[1] : (z == 2 ? g.Ab[2] : g.Ab[3]));
        gB = z == 0 ? g.Bb[0] : (z == 1 ? g.Bb[1] : (z == 2 ? g.Bb[2] : g.Bb[3]));
        gC = z == 0 ? g.Cb[0] : (z == 1 ? g.Cb[1] : (z == 2 ? g.Cb[2] : g.Cb[3]));
    }
    const int wrow = C::KSPLIT == 1 ? (wave >> 1) * C::WM : 0, wcol = C::KSPLIT == 1 ? (wave & 1) * C::WN : 0;

    f32x4 acc[NB][FM][FN];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int steps = (g.K + BK - 1) / BK;
#pragma unroll
    for (int pass = 0; pass < (EPI == EPI_DUAL_ACC ? 2 : 1); ++pass) {
        Source<BM, BK, ADM, AHEAD, VEC> sa;
        Source<BN, BK, BDM, AHEAD, VEC> sb, sb2;
        sa.init(pass ? g.A2 : gA, g.lda, g.M, m0, g.K, g.ag, nullptr, tid);
        sb.init(pass ? g.B2 : gB, g.ldb, g.N, n0, g.K, BDM ? nullptr : g.bg, BDM ? g.bg : nullptr, tid);
        if (kTwoB) sb2.init(g.B2, g.ldb, g.N, n0, g.K, BDM ? nullptr : g.bg, BDM ? g.bg : nullptr, tid);
        f32x4 ra[AHEAD][OA::PER], rb[NB][AHEAD][OB::PER];
        auto list = [&](int t, int s) {
            sa.list(s, t * BK);
            sb.list(s, t * BK);
            if (kTwoB) sb2.list(s, t * BK);
        };
        // tile t of the depth into register set s, then the lists of the set's next tile: when those are used, the
        // loads issued after them may still be in flight
        auto fetch = [&](int t, auto set) {
            constexpr int s = decltype(set)::value;
            sa.fetch(ra[s], s, t * BK);
            sb.fetch(rb[0][s], s, t * BK);
            if (kTwoB) sb2.fetch(rb[NB - 1][s], s, t * BK);
            list(t + AHEAD, s);
        };
        auto stash = [&](int t, auto set) {
            constexpr int s = decltype(set)::value;
            float* st = smem + (t & 1) * STAGE;
            sa.stash(st, ra[s], t * BK);
            sb.stash(st + OA::FLOATS, rb[0][s], t * BK);
            if (kTwoB) sb2.stash(st + OA::FLOATS + OB::FLOATS, rb[NB - 1][s], t * BK);
        };
        auto compute = [&](int t) {
            const float* st = smem + (t & 1) * STAGE;
#pragma unroll
            for (int u = 0; u < (C::KSPLIT == 1 ? BK / 16 : 1); ++u) {
                const int kt = C::KSPLIT == 1 ? u : wave;
                f32x4 fa[FM], fb[NB][FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) fa[i] = fragment<BM, BK, ADM>(st, wrow + 16 * i + l16, kt, lg);
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        fb[b][j] = fragment<BN, BK, BDM>(st + OA::FLOATS + b * OB::FLOATS, wcol + 16 * j + l16, kt, lg);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int i = 0; i < FM; ++i)
#pragma unroll
                            for (int j = 0; j < FN; ++j) // B first: a lane then holds 4 consecutive columns of one row
                                acc[b][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[b][j][e], fa[i][e], acc[b][i][j], 0, 0, 0);
            }
        };
        // tile t is in LDS, t + 1 .. t + AHEAD in registers (set of tile t: t % AHEAD).  Everything runs unconditionally:
        // tiles beyond the last are clamped loads and zeros that no step computes on, and without branches the loads in
        // flight are counted exactly.
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) list(s, s);
        typedef std::integral_constant<int, 0> Set0;
        typedef std::integral_constant<int, 1 % AHEAD> Set1;
        typedef std::integral_constant<int, 2 % AHEAD> Set2;
        fetch(0, Set0{});
        if constexpr (AHEAD == 3) {
            fetch(1, Set1{});
            fetch(2, Set2{});
        }
        stash(0, Set0{});
        fetch(AHEAD, Set0{});
        __syncthreads();
        auto step = [&](int t, auto set) { // `set`: register set of tile t + 1
            stash(t + 1, set);
            fetch(t + 1 + AHEAD, set);
            compute(t);
            __syncthreads();
        };
        int t = 0;
        for (; t + 3 <= steps; t += 3) {
            step(t, Set1{});
            step(t + 1, Set2{});
            step(t + 2, Set0{});
        }
        if (t < steps) step(t, Set1{});
        if (t + 1 < steps) step(t + 1, Set2{});
    }

    if constexpr (C::KSPLIT == 1) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                emit<EPI>(g, gC, m0 + wrow + 16 * i + l16, n0 + wcol + 16 * j + 4 * lg, acc[0][i][j], acc[NB - 1][i][j]);
    } else {
        // the waves' depth shares meet in LDS, added in wave order; one thread per 4 columns
        static_assert(BM * BN / 4 == 256 && BN == 32 && C::KSPLIT * BM * (BN + 4) * NB <= 2 * STAGE, "one piece per thread");
        constexpr int RS = BN + 4;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    *(f32x4*)(smem + ((b * C::KSPLIT + wave) * BM + 16 * i + l16) * RS + 16 * j + 4 * lg) = acc[b][i][j];
        __syncthreads();
        const int row = tid / 8, c = (tid % 8) * 4;
        f32x4 s[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            s[b] = *(const f32x4*)(smem + (b * C::KSPLIT * BM + row) * RS + c);
#pragma unroll
            for (int w = 1; w < C::KSPLIT; ++w) s[b] += *(const f32x4*)(smem + ((b * C::KSPLIT + w) * BM + row) * RS + c);
        }
        emit<EPI>(g, gC, m0 + row, n0 + c, s[0], s[NB - 1]);
    }
}

// ---------------------------------------------------------------------------------------------------
// Launches of few tiles: B x B outputs a workgroup (B = 16 or 32), whose four waves take the 32-deep steps w, w + 4, ...
// of the tile's depth, each in LDS stages of its own.  Operands go memory -> LDS by direct loads (16 bytes a lane, 1 KB
// an instruction, no registers, no barrier), `S` steps of every wave in flight; the waves' sums meet in LDS at the end.
// Such a launch is bound by the latency of its loads and by the share of the chip's matrix cores that its tiles reach:
// B = 16 spreads 256 x 256 outputs over all CUs, where the 32 x 32 tile of the other kernel (KSPLIT) takes 64 of them and
// meets at a barrier every 64 depth steps.  B = 32 serves launches of several problems (gemm_f32_group).  More stages than
// two (S = 4) gained nothing and keep a second workgroup off the CU.
//
// LDS of one operand's step, 16-byte chunks:
//   rows        : [B rows][8 chunks of 4 depth steps], chunk c of row r at position c ^ ((r >> 1) & 7)
//   depth-major : [32 depth steps][B / 4 chunks of 4 rows]; depth step 16 t + 4 g + j in LDS row 16 t + 4 j + g, and for
//                 B = 32 chunk c of LDS row q at position c ^ (4 ((q >> 1) & 1))
// A 16 x 16 fragment is one 16-byte read per lane of the first, four 4-byte reads of the second; both free of conflicts.
// ---------------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(1))) const void* glb_void_ptr;
#define SDP_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))
#define SDP_WAIT_LGKMCNT0() __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14))

constexpr int kListMax = 4096; // entries of a gathered depth's list that are kept in LDS

// source of the chunks beyond the depth
__device__ __attribute__((aligned(16))) const float kZero4[4] = {0.f, 0.f, 0.f, 0.f};

// V: 16-byte loads (aligned base and stride, extent along the contiguous axis a multiple of 4), a lane fills a chunk.  Else 4-byte
// ones, a lane fills one float, which also lets a depth-major operand gather its columns (the weight gradients' list of neurons).
template <int B, bool DM, bool V>
struct WaveOperand {
    static constexpr int BYTES = B * 128, SLABS = BYTES / (V ? 1024 : 256); // of one step; direct loads a step
    static constexpr int CPR = DM ? B / 4 : 8;                              // chunks per LDS row
    static constexpr int LPR = V ? CPR : 4 * CPR, RPS = 64 / LPR;           // lanes per LDS row, LDS rows per slab
    // rows: this lane's place in each slab at depth 0; depth-major: its first column (4-byte loads of 32 columns: two, those of the
    // even slabs and those of the odd ones)
    static constexpr int NP = DM ? (!V && B == 32 ? 2 : 1) : SLABS;
    const float* p[NP];
    int k[SLABS]; // depth of that place within a step
    int64_t ld;
    __device__ void init(const float* base, int64_t ld_, int rows, int row0, const int32_t* gather, int lane) {
        ld = ld_;
        const int pos = lane % LPR;
#pragma unroll
        for (int i = 0; i < SLABS; ++i) {
            const int q = RPS * i + lane / LPR; // LDS row
            if constexpr (DM) {
                k[i] = (q & 16) + 4 * (q & 3) + ((q >> 2) & 3);
                if (i < NP) {
                    // the swizzle bit of LDS row q is the same in every slab (in every second one): a slab holds 8 or 16 rows (2 or 4)
                    const int swap = B == 32 ? 4 * ((q >> 1) & 1) : 0; // chunks
                    int c = row0 + (V ? 4 * (pos ^ swap) : pos ^ (4 * swap));
                    c = c < rows ? c : rows - (V ? 4 : 1);
                    p[i] = base + (!V && gather ? gather[c] : c);
                }
            } else {
                const int swap = (q >> 1) & 7;
                int r = row0 + q;
                r = r < rows ? r : rows - 1;
                k[i] = V ? 4 * (pos ^ swap) : pos ^ (4 * swap);
                p[i] = base + (int64_t)(gather ? gather[r] : r) * ld_ + k[i];
            }
        }
    }
    // the direct loads of the step that begins at depth k0, of the operand `other` bytes from this one; list: gathered depth (in
    // LDS), or null
    __device__ void issue(unsigned char* lds, int k0, int K, const int* list, int64_t other = 0) const {
#pragma unroll
        for (int i = 0; i < SLABS; ++i) {
            const int kk = k0 + k[i];
            const float* src;
            if constexpr (DM) {
                const int kc = kk < K ? kk : K - 1;
                src = p[i % NP] + (int64_t)(list ? list[kc] : kc) * ld;
            } else {
                src = p[i] + k0;
            }
            src = (const float*)((const char*)src + other);
            if (kk >= K) src = kZero4;
            if constexpr (V) __builtin_amdgcn_global_load_lds((glb_void_ptr)src, (lds_void_ptr)(lds + 1024 * i), 16, 0, 0);
            else __builtin_amdgcn_global_load_lds((glb_void_ptr)src, (lds_void_ptr)(lds + 256 * i), 4, 0, 0);
        }
    }
    // rows 16 f .. of the tile at depth 16 t of the step: element j belongs to depth 16 t + 4 lg + j
    __device__ static f32x4 fragment(const unsigned char* lds, int f, int t, int l16, int lg) {
        if constexpr (DM) {
            const float* w = (const float*)lds;
            f32x4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int q = 16 * t + 4 * j + lg, col = 16 * f + l16;
                v[j] = w[q * B + (B == 32 ? col ^ (16 * ((q >> 1) & 1)) : col)];
            }
            return v;
        } else {
            const int r = 16 * f + l16;
            return *(const f32x4*)(lds + r * 128 + (((4 * t + lg) ^ ((r >> 1) & 7)) * 16));
        }
    }
};

template <int B, int S, int EPI, bool ADM, bool BDM, bool VA, bool VB>
struct WaveShape {
    static constexpr int NB = EPI == EPI_SWIGLU_FWD ? 2 : 1;
    static constexpr int STAGE = (1 + NB) * B * 128, LOADS = WaveOperand<B, ADM, VA>::SLABS + NB * WaveOperand<B, BDM, VB>::SLABS;
    static constexpr int TILES = 4 * S * STAGE, LDS = TILES + (BDM ? kListMax * 4 : 0);
    static_assert(LDS <= 160 * 1024 && 4 * NB * B * (B + 4) * 4 <= TILES && (S - 1) * LOADS < 64, "fits");
};

template <int B, int S, int EPI, bool ADM, bool BDM, bool VA = true, bool VB = true>
__device__ inline void wave_body(const Dev& g, int block, unsigned char* smem) {
    using Sh = WaveShape<B, S, EPI, ADM, BDM, VA, VB>;
    typedef WaveOperand<B, ADM, VA> OA;
    typedef WaveOperand<B, BDM, VB> OB;
    constexpr int NB = Sh::NB, F = B / 16;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = g.tiles_m * g.tiles_n;
    const int z = block / per, tile = block - z * per;
    const int m0 = (tile % g.tiles_m) * B, n0 = (tile / g.tiles_m) * B;
    const float *gA = g.A, *gB = g.B;
    float* gC = g.C;
    if (g.nbatch > 0) {
        gA = z == 0 ? g.Ab[0] : (z == 1 ? g.Ab[1] : (z == 2 ? g.Ab[2] : g.Ab[3]));
        gB = z == 0 ? g.Bb[0] : (z == 1 ? g.Bb[1] : (z == 2 ? g.Bb[2] : g.Bb[3]));
        gC = z == 0 ? g.Cb[0] : (z == 1 ? g.Cb[1] : (z == 2 ? g.Cb[2] : g.Cb[3]));
    }
    int* list = nullptr;
    if constexpr (BDM) {
        if (g.bg) { // K <= kListMax
            list = (int*)(smem + Sh::TILES);
            for (int i = tid; i < g.K; i += 256) list[i] = g.bg[i];
            __syncthreads();
        }
    }
    OA a;
    OB b[NB];
    a.init(gA, g.lda, g.M, m0, ADM && VA ? nullptr : g.ag, lane);
    b[0].init(gB, g.ldb, g.N, n0, BDM ? nullptr : g.bg, lane);
    if constexpr (NB == 2) b[1].init(g.B2, g.ldb, g.N, n0, g.bg, lane);
    f32x4 acc[NB][F][F];
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j) acc[c][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    unsigned char* const mine = smem + wave * S * Sh::STAGE;
    const int steps = (g.K + 31) / 32;
    {
        // this wave's steps, of both operand pairs in one run (each pair on its own: the loads of its first steps are waited for)
        const int n1 = steps > wave ? (steps - wave + 3) / 4 : 0, n = EPI == EPI_DUAL_ACC ? 2 * n1 : n1;
        const int64_t other_a = EPI == EPI_DUAL_ACC ? (int64_t)((intptr_t)g.A2 - (intptr_t)gA) : 0;
        const int64_t other_b = EPI == EPI_DUAL_ACC ? (int64_t)((intptr_t)g.B2 - (intptr_t)gB) : 0;
        auto issue = [&](int t, int stage) {
            unsigned char* st = mine + stage * Sh::STAGE;
            const bool second = EPI == EPI_DUAL_ACC && t >= n1;
            const int k0 = 32 * (wave + 4 * (second ? t - n1 : t));
            a.issue(st, k0, g.K, nullptr, second ? other_a : 0);
#pragma unroll
            for (int c = 0; c < NB; ++c) b[c].issue(st + OA::BYTES + c * OB::BYTES, k0, g.K, list, second ? other_b : 0);
        };
        for (int t = 0; t < S && t < n; ++t) issue(t, t);
        int stage = 0;
        for (int t = 0; t < n; ++t) {
            // steps issued beyond this one: S - 1, fewer at the end
            const int ahead = n - 1 - t;
            if (ahead >= S - 1) SDP_WAIT_VMCNT((S - 1) * Sh::LOADS);
            else if (S > 2 && ahead == 2) SDP_WAIT_VMCNT(2 * Sh::LOADS);
            else if (S > 1 && ahead == 1) SDP_WAIT_VMCNT(Sh::LOADS);
            else SDP_WAIT_VMCNT(0);
            __builtin_amdgcn_sched_barrier(0);
            const unsigned char* st = mine + stage * Sh::STAGE;
            f32x4 fa[2][F], fb[2][NB][F];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int i = 0; i < F; ++i) fa[u][i] = OA::fragment(st, i, u, l16, lg);
#pragma unroll
                for (int c = 0; c < NB; ++c)
#pragma unroll
                    for (int j = 0; j < F; ++j) fb[u][c][j] = OB::fragment(st + OA::BYTES + c * OB::BYTES, j, u, l16, lg);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (u == 1) { // the whole step has been read: its stage can be filled again
                    SDP_WAIT_LGKMCNT0();
                    __builtin_amdgcn_sched_barrier(0);
                    if (t + S < n) issue(t + S, stage);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int c = 0; c < NB; ++c)
#pragma unroll
                        for (int i = 0; i < F; ++i)
#pragma unroll
                            for (int j = 0; j < F; ++j) // B first: a lane then holds 4 consecutive columns of one row
                                acc[c][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[u][c][j][e], fa[u][i][e], acc[c][i][j], 0, 0, 0);
            }
            stage = stage == S - 1 ? 0 : stage + 1;
        }
    }
    __syncthreads(); // every wave is done with its stages
    constexpr int RS = B + 4;
    float* const sum = (float*)smem;
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
            for (int j = 0; j < F; ++j)
                *(f32x4*)(sum + ((c * 4 + wave) * B + 16 * i + l16) * RS + 16 * j + 4 * lg) = acc[c][i][j];
    __syncthreads();
    if (tid < B * B / 4) {
        const int row = tid / (B / 4), col = (tid % (B / 4)) * 4;
        f32x4 v[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            v[c] = *(const f32x4*)(sum + (c * 4 * B + row) * RS + col);
#pragma unroll
            for (int w = 1; w < 4; ++w) v[c] += *(const f32x4*)(sum + ((c * 4 + w) * B + row) * RS + col);
        }
        emit<EPI>(g, gC, m0 + row, n0 + col, v[0], v[NB - 1]);
    }
}

template <int B, int S, int EPI, bool ADM, bool BDM, bool VA, bool VB>
__global__ __launch_bounds__(256) void gemm_f32_wave_kernel(Dev g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char wave_lds[];
    wave_body<B, S, EPI, ADM, BDM, VA, VB>(g, blockIdx.x, wave_lds);
}

template <int B, int S, int EPI, bool ADM, bool BDM, bool VA = true, bool VB = true>
int launch_wave(Dev g, const char* name, hipStream_t s) {
    typedef WaveShape<B, S, EPI, ADM, BDM, VA, VB> Sh;
    constexpr int LDS = Sh::LDS;
    const int lds = BDM && g.bg ? LDS : Sh::TILES;
    g.tiles_m = (g.M + B - 1) / B, g.tiles_n = (g.N + B - 1) / B;
    const int64_t blocks = (int64_t)g.tiles_m * g.tiles_n * (g.nbatch > 0 ? g.nbatch : 1);
    if (blocks > 0x7FFFFFFF) return SDP_ERR_SHAPE;
    auto kern = gemm_f32_wave_kernel<B, S, EPI, ADM, BDM, VA, VB>;
    static const hipError_t attr = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (attr != hipSuccess) return SDP_ERR_HIP;
    profile_shape(name, B, B, 0, S == 1 ? F32_WAVES_ONE_STAGE : F32_WAVES);
    ProfileScope ps(name, s);
    kern<<<(unsigned)blocks, 256, lds, s>>>(g);
    return launch_status();
}

#include "sdp_f32_split.h"

// ---------------------------------------------------------------------------------------------------
// Pipelined tile: 64 x 64 outputs (of both right operands: 64 x 32 each), four waves of 32 x 32, depth steps of 32 in three LDS stages
// that direct loads fill.  A step is two 16-deep halves; while a wave's MFMAs of one half run, its fragments of the next are read, and
// one barrier a step, between the halves, hands over the stages:
//   first half of step k : MFMAs on (k, 0); reads of (k, 1)
//   wait for the own loads of step k + 1 and the own reads of step k; barrier: step k + 1 has landed, step k is read
//   second half          : MFMAs on (k, 1); reads of (k + 1, 0); loads of step k + 3 into the stage of step k
//
// LDS of an operand's step, 16-byte chunks:
//   rows        : [rows][8 chunks of 4 depth steps], chunk c of row r at position c ^ ((r >> 1) & 7); a fragment is 16 rows, one
//                 16-byte read per lane gives 4 depth steps of it
//   depth-major : [32 depth steps][rows / 4 chunks]; fragment f of a wave's F fragments is its rows F i + f, i = 0 .. 15, so that
//                 one read of F floats per lane and depth step gives all of them.  F = 2: the 128-byte halves of a row trade
//                 places where bit 2 of the depth step is set, which keeps the four lane groups (4 steps apart) off each
//                 other's banks.
// ---------------------------------------------------------------------------------------------------
template <int R, bool DM, bool V>
struct PipeOperand {
    static constexpr int BYTES = R * 128, PER = R / (V ? 32 : 8); // of a step; direct loads of a wave and step
    static constexpr int F = R / 32;                              // fragments of a wave
    static constexpr int LPR = (DM ? R / 4 : 8) * (V ? 1 : 4), RPS = 64 / LPR; // lanes per LDS row, LDS rows per load
    static_assert(64 % LPR == 0, "whole rows a load");
    static constexpr int swap(int k) { return DM ? 8 * (k >> 2 & 1) : 0; } // depth-major: chunk c sits at c ^ swap
    static constexpr int NP = DM ? (swap(4) && !V ? 2 : 1) : PER;
    int64_t off[NP]; // elements from the base: this lane's places at depth 0 (depth-major: its first column, of even and odd loads)
    int k[PER];      // and their depth within a step
    int64_t ld;
    __device__ void init(int64_t ld_, int rows, int row0, const int32_t* gather, int wave, int lane) {
        ld = ld_;
        const int pos = lane % LPR;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int q = RPS * (4 * i + wave) + lane / LPR; // LDS row
            if constexpr (DM) {
                // bit 2 of q: the same for all loads (V: 4 rows a load and wave), or that of i (one row)
                static_assert(V ? RPS == 4 : RPS == 1, "which loads share a swap");
                k[i] = q;
                if (i < NP) {
                    int c = row0 + (V ? 4 * (pos ^ swap(q)) : pos ^ (4 * swap(q)));
                    c = c < rows ? c : rows - (V ? 4 : 1);
                    off[i] = !V && gather ? gather[c] : c;
                }
            } else {
                const int turn = (q >> 1) & 7;
                int r = row0 + q;
                r = r < rows ? r : rows - 1;
                k[i] = V ? 4 * (pos ^ turn) : pos ^ (4 * turn);
                off[i] = (int64_t)(gather ? gather[r] : r) * ld_ + k[i];
            }
        }
    }
    // load i of the step that begins at depth k0; list: gathered depth (in LDS), or null
    __device__ void issue(unsigned char* stage, int wave, int i, const float* base, int k0, int K, const int* list) const {
        const int kk = k0 + k[i];
        const float* src;
        if constexpr (DM) {
            const int kc = kk < K ? kk : K - 1;
            src = base + off[i % NP] + (int64_t)(list ? list[kc] : kc) * ld;
        } else {
            src = base + off[i] + k0;
        }
        if (kk >= K) src = kZero4;
        if constexpr (V) __builtin_amdgcn_global_load_lds((glb_void_ptr)src, (lds_void_ptr)(stage + 1024 * (4 * i + wave)), 16, 0, 0);
        else __builtin_amdgcn_global_load_lds((glb_void_ptr)src, (lds_void_ptr)(stage + 256 * (4 * i + wave)), 4, 0, 0);
    }
    // read r of half h: rows part0 .. of the tile.  fr[f][e] belongs to depth 16 h + 4 lg + e.
    static constexpr int READS = DM ? 4 : F;
    __device__ static void read(const unsigned char* stage, int part0, int h, int r, int l16, int lg, f32x4 (&fr)[F]) {
        if constexpr (DM) {
            const int kk = 16 * h + 4 * lg + r;
            const unsigned char* p = stage + kk * R * 4;
            static_assert(F == 2, "64 rows");
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            const int col = part0 + 2 * l16; // floats; the swap is of 32 floats, the same for all steps of a lane group
            const f32x2 v = *(const f32x2*)(p + (col ^ (32 * (lg & 1))) * 4);
            fr[0][r] = v[0], fr[1][r] = v[1];
        } else {
            const int row = part0 + 16 * r + l16;
            fr[r] = *(const f32x4*)(stage + row * 128 + (((4 * h + lg) ^ ((row >> 1) & 7)) * 16));
        }
    }
};

template <int BM, int BN, int EPI, bool ADM, bool BDM, bool VA, bool VB, bool LIST = BDM>
struct PipeShape {
    static constexpr int NB = EPI == EPI_SWIGLU_FWD ? 2 : 1; // BN columns of each
    typedef PipeOperand<BM, ADM, VA> OA;
    typedef PipeOperand<BN, BDM, VB> OB;
    static constexpr int STAGE = OA::BYTES + NB * OB::BYTES, LOADS = OA::PER + NB * OB::PER;
    static constexpr int RING = 3 * STAGE, LDS = RING + (LIST ? kListMax * 4 : 0);
};

template <int BM, int BN, int EPI, bool ADM, bool BDM, bool VA, bool VB, bool LIST = BDM>
__device__ inline void pipe_body(const Dev& g, int block, unsigned char* smem) {
    using Sh = PipeShape<BM, BN, EPI, ADM, BDM, VA, VB, LIST>;
    typedef typename Sh::OA OA;
    typedef typename Sh::OB OB;
    constexpr int NB = Sh::NB, FM = OA::F, FN = OB::F, L = Sh::LOADS;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = g.tiles_m * g.tiles_n;
    const int z = block / per, tile = block - z * per;
    const int m0 = (tile % g.tiles_m) * BM, n0 = (tile / g.tiles_m) * BN;
    const int pm = (wave >> 1) * (BM / 2), pn = (wave & 1) * (BN / 2); // the wave's part
    const float *gA = g.A, *gB = g.B;
    float* gC = g.C;
    if (g.nbatch > 0) {
        gA = z == 0 ? g.Ab[0] : (z == 1 ? g.Ab[1] : (z == 2 ? g.Ab[2] : g.Ab[3]));
        gB = z == 0 ? g.Bb[0] : (z == 1 ? g.Bb[1] : (z == 2 ? g.Bb[2] : g.Bb[3]));
        gC = z == 0 ? g.Cb[0] : (z == 1 ? g.Cb[1] : (z == 2 ? g.Cb[2] : g.Cb[3]));
    }
    int* list = nullptr;
    if constexpr (LIST) {
        if (g.bg) { // K <= kListMax
            list = (int*)(smem + Sh::RING);
            for (int i = tid; i < g.K; i += 256) list[i] = g.bg[i];
            __syncthreads();
        }
    }
    OA a;
    OB b;
    a.init(g.lda, g.M, m0, ADM && VA ? nullptr : g.ag, wave, lane);
    b.init(g.ldb, g.N, n0, BDM ? nullptr : g.bg, wave, lane);
    f32x4 acc[NB][FM][FN];
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[c][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int n1 = (g.K + 31) / 32, n = EPI == EPI_DUAL_ACC ? 2 * n1 : n1;
    auto issue = [&](int t, int stage, int l) { // load l of step t
        const bool second = EPI == EPI_DUAL_ACC && t >= n1;
        const int k0 = 32 * (second ? t - n1 : t);
        unsigned char* st = smem + stage * Sh::STAGE;
        if (l < OA::PER) a.issue(st, wave, l, second ? g.A2 : gA, k0, g.K, nullptr);
        else if (l < OA::PER + OB::PER) b.issue(st + OA::BYTES, wave, l - OA::PER, second ? g.B2 : gB, k0, g.K, list);
        else b.issue(st + OA::BYTES + OB::BYTES, wave, l - OA::PER - OB::PER, g.B2, k0, g.K, list);
    };
    f32x4 fa[2][FM], fb[2][NB][FN];
    constexpr int NR = OA::READS + NB * OB::READS, NM = 4 * NB * FM * FN; // of a half
    static_assert(NR <= NM && L <= NM, "between the MFMAs");
    auto read_one = [&](int stage, int h, int r) {
        const unsigned char* st = smem + stage * Sh::STAGE;
        if (r < OA::READS) OA::read(st, pm, h, r, l16, lg, fa[h]);
        else if (r < OA::READS + OB::READS) OB::read(st + OA::BYTES, pn, h, r - OA::READS, l16, lg, fb[h][0]);
        else OB::read(st + OA::BYTES + OB::BYTES, pn, h, r - OA::READS - OB::READS, l16, lg, fb[h][NB - 1]);
    };
    // the MFMAs of half h; between them the reads of the other half from `stage` and the loads of step `t`
    auto half = [&](int h, bool reads, int stage, bool loads, int t, int into) {
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const bool rd = reads && m < NR, ldq = loads && m * L / NM != (m + 1) * L / NM;
            if (rd) read_one(stage, h ^ 1, m);
            if (ldq) issue(t, into, m * L / NM);
            if (rd || ldq) __builtin_amdgcn_sched_barrier(0);
            const int e = m / (NB * FM * FN), c = m / (FM * FN) % NB, i = m / FN % FM, j = m % FN;
            // B first: a lane then holds outputs of one row
            acc[c][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[h][c][j][e], fa[h][i][e], acc[c][i][j], 0, 0, 0);
            if (rd || ldq) __builtin_amdgcn_sched_barrier(0);
        }
    };
    int t = 0, stage = 0;
    auto step = [&](auto left_c) { // steps left after this one, at most 3
        constexpr int LEFT = decltype(left_c)::value;
        const int next = stage == 2 ? 0 : stage + 1;
        half(0, true, stage, false, 0, 0);
        if constexpr (LEFT > 0) {
            __builtin_amdgcn_sched_barrier(0);
            SDP_WAIT_VMCNT(LEFT > 1 ? L : 0);
            SDP_WAIT_LGKMCNT0();
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        }
        half(1, LEFT > 0, next, LEFT > 2, t + 3, stage);
        __builtin_amdgcn_sched_barrier(0);
        stage = next, ++t;
    };
#pragma unroll
    for (int j = 0; j < 3; ++j)
        if (j < n) {
#pragma unroll
            for (int l = 0; l < L; ++l) issue(j, j, l);
        }
    __builtin_amdgcn_sched_barrier(0);
    if (n > 2) SDP_WAIT_VMCNT(2 * L); else if (n > 1) SDP_WAIT_VMCNT(L); else SDP_WAIT_VMCNT(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < NR; ++r) read_one(0, 0, r);
    while (t + 3 < n) step(std::integral_constant<int, 3>{});
    if (t + 2 < n) step(std::integral_constant<int, 2>{});
    if (t + 1 < n) step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 0>{});

    // element r of acc[c][i][j]: fragment row l16 of A's i-th, row 4 lg + r of B's j-th
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int m = m0 + pm + (ADM ? FM * l16 + i : 16 * i + l16);
#pragma unroll
        for (int q = 0; q < FN; ++q) {
            f32x4 v[NB];
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                if constexpr (!BDM) v[c] = acc[c][i][q];
                else v[c] = f32x4{acc[c][i][0][2 * q], acc[c][i][1][2 * q], acc[c][i][0][2 * q + 1], acc[c][i][1][2 * q + 1]};
            }
            emit<EPI>(g, gC, m, n0 + pn + (BDM ? 4 * FN * lg + 4 * q : 16 * q + 4 * lg), v[0], v[NB - 1]);
        }
    }
}

template <int BM, int BN, int EPI, bool ADM, bool BDM, bool VA, bool VB>
__global__ __launch_bounds__(256) void gemm_f32_pipe_kernel(Dev g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char pipe_lds[];
    pipe_body<BM, BN, EPI, ADM, BDM, VA, VB>(g, blockIdx.x, pipe_lds);
}

template <int BM, int BN, int EPI, bool ADM, bool BDM, bool VA, bool VB>
int launch_pipe(Dev g, const char* name, hipStream_t s) {
    typedef PipeShape<BM, BN, EPI, ADM, BDM, VA, VB> Sh;
    const int lds = g.bg && BDM ? Sh::LDS : Sh::RING;
    g.tiles_m = (g.M + BM - 1) / BM, g.tiles_n = (g.N + BN - 1) / BN;
    const int64_t blocks = (int64_t)g.tiles_m * g.tiles_n * (g.nbatch > 0 ? g.nbatch : 1);
    if (blocks > 0x7FFFFFFF) return SDP_ERR_SHAPE;
    auto kern = gemm_f32_pipe_kernel<BM, BN, EPI, ADM, BDM, VA, VB>;
    static const hipError_t attr = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, Sh::LDS);
    if (attr != hipSuccess) return SDP_ERR_HIP;
    profile_shape(name, BM, BN, 0, F32_PIPELINED);
    ProfileScope ps(name, s);
    kern<<<(unsigned)blocks, 256, lds, s>>>(g);
    return launch_status();
}

template <class C, int EPI, bool ADM, bool BDM, bool VEC>
int launch(Dev g, const char* name, hipStream_t s) {
    constexpr int STAGE = Operand<C::BM, C::BK, ADM>::FLOATS + (EPI == EPI_SWIGLU_FWD ? 2 : 1) * Operand<C::BN, C::BK, BDM>::FLOATS;
    constexpr int LDS = 2 * STAGE * 4;
    static_assert(LDS <= 160 * 1024, "LDS of one CU");
    g.tiles_m = (g.M + C::BM - 1) / C::BM, g.tiles_n = (g.N + C::BN - 1) / C::BN;
    const int64_t blocks = (int64_t)g.tiles_m * g.tiles_n * (g.nbatch > 0 ? g.nbatch : 1);
    if (blocks > 0x7FFFFFFF) return SDP_ERR_SHAPE;
    auto kern = gemm_f32_kernel<C, EPI, ADM, BDM, VEC>;
    static const hipError_t attr = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (attr != hipSuccess) return SDP_ERR_HIP;
    profile_shape(name, C::BM, C::BN, 0, F32_STAGED);
    ProfileScope ps(name, s);
    kern<<<(unsigned)blocks, 256, LDS, s>>>(g);
    return launch_status();
}

// Launches whose 16 x 16 tiles are resident all at once (two workgroups a CU).  Against the 32 x 32 tile (times with about
// 5 us of event overhead): 256 x 512, depth 256, two operands 10.1 -> 7.5 us; 256 x 256, depth 2 x 512 15.0 -> 9.1; 128 x
// 512, depth 1024 13.3 -> 9.2; but 512 x 512, depth 512 (1024 tiles) 10.4 -> 12.1.
bool few_tiles(const Dev& g) {
    return (int64_t)((g.M + 15) / 16) * ((g.N + 15) / 16) * (g.nbatch > 0 ? g.nbatch : 1) <= 512;
}

// Whether a launch takes the tiles of sdp_f32_split.h instead of the fp32 ones: what either would take, from its rounds of tiles over the
// 256 CUs and its steps of 32 depths.  The figures are kernel times in us, with about 5 of event overhead, of 850 launches of MLP and
// attention passes (T = 64 .. 2400, widths 160 .. 3000, every alignment, listed columns), fitted within 3 to 8 % (rms).
// A round of split tiles takes what two and a half rounds of 32-wide ones do with 16-byte loads, so one loses to two of those and two
// lose to four, but win against three and five: fp32 / split (rounds), down T = 416, d = 1176, p = 1824 30.1 / 35.7 (2 / 1), T = 512,
// d = 1100, p = 1376 35.5 / 30.4 (3 / 1), T = 1518, d = 668, p = 1444 42.3 / 48.1 (4 / 2), T = 1300, d = 800, p = 816 39.5 / 31.1 (6 / 2).  Single
// floats cost the fp32 loops a quarter to all of a step again and the split ones nothing: weight gradients of 699 x 623, 813 deep
// 100.7 / 48.1.  Rows that end off a multiple of four floats cost the split epilogues more, since a lane has single columns of 32 rows; the
// activation gradient's then takes 12 us a round: n = 1407, d = 576, T = 900 27.4 / 39.4, and with single-float loads T = 599, d = 367, n = 799
// 15.4 / 21.9.  Listed columns of the left operand cost them a third of a step: T = 408, d = 676, p = 372 17.2 / 21.6, but T = 2160, d = 460,
// p = 948 138 / 111.
struct LaunchKind {
    int kind; // 0 gate_up, 1 activation gradient, 2 both operands by rows, 3 right one depth-major, 4 both depth-major
    int load; // 16-byte loads: 0 of both operands, 1 of the right one, 2 of neither
    bool rows, listed; // 16-byte stores; listed columns of a depth-major left operand
};
constexpr double kRound32[5][3] = {{1.3, 0, 3.5}, {1, 0, 1.8}, {.6, 0, 1.8}, {1.2, .3, 2.4}, {.5, .4, .1}};
constexpr double kStep32[5][3] = {{.303, 0, .43}, {.161, 0, .232}, {.165, 0, .232}, {.188, .262, .39}, {.184, .265, .352}};
constexpr double kStart64[5][3] = {{8, 0, 8}, {9.7, 0, 12}, {7.5, 0, 12}, {8, 9, 15}, {9, 9, 13}};
constexpr double kStep64[5][3] = {{.61, 0, .745}, {.64, 0, .745}, {.63, 0, .745}, {.70, .80, 1.2}, {.60, .66, .72}};
double fp32_us(const LaunchKind& k, int width, int64_t tiles32, int64_t tiles64, int64_t steps) {
    if (width == 32) return 6.2 + (tiles32 + 255) / 256 * (kRound32[k.kind][k.load] + (kStep32[k.kind][k.load] + (k.listed ? .025 : 0)) * steps);
    const double round = k.kind == 1 ? (k.rows ? .6 : 3) : k.kind == 0 && !k.rows ? 1.3 : 0;
    return kStart64[k.kind][k.load] + (tiles64 + 255) / 256 * (round + kStep64[k.kind][k.load] * steps);
}
constexpr double kSplitRound[5][2] = {{1.3, 4}, {5.5, 12}, {.9, 3}, {1.3, 1.8}, {1, 2}}; // rows, not rows
constexpr double kSplitStart[5] = {5.2, 2, 5, 5.3, 5.2}, kSplitStep[5] = {.446, .425, .452, .46, .474};
constexpr double kTeamsStart[5] = {7.1, 5, 7.1, 7, 7.2}, kTeamsStep[5] = {.455, .455, .46, .495, .567}; // two teams: one round
double split_us(const LaunchKind& k, int64_t tiles64, int64_t steps) {
    const int64_t rounds = (tiles64 + 255) / 256;
    if (k.listed) return rounds == 1 ? 10 + .827 * steps : k.rows ? 4.5 + rounds * (3 + .652 * steps) : rounds * (5.5 + .69 * steps);
    const double round = kSplitRound[k.kind][k.rows ? 0 : 1];
    return rounds == 1 ? kTeamsStart[k.kind] + round + kTeamsStep[k.kind] * steps : kSplitStart[k.kind] + rounds * (round + kSplitStep[k.kind] * steps);
}

// width: of the fp32 tiles that the launch would have
template <int EPI, bool ADM, bool BDM, bool VA, bool VB>
bool split_pays(const Dev& g, int width, int64_t tiles32, int64_t tiles64) {
    constexpr bool VEC = VA && VB, two = EPI == EPI_SWIGLU_FWD;
    const LaunchKind k{two ? 0 : EPI == EPI_SWIGLU_BWD ? 1 : ADM ? 4 : BDM ? 3 : 2, VEC ? 0 : VB ? 1 : 2, g.vec_out != 0, ADM && g.ag};
    // what the tiles need: a whole step, 64 rows of a depth-major operand
    if (g.K < 256 || (ADM && g.M < 64) || (BDM && g.N < 64) || tiles64 > 0x7FFFFF) return false;
    if (two && tiles64 <= 256 && g.K < 320 && (VEC || !k.rows)) return false; // T = 528, d = 280, n = 536 11.9 / 12.6
    // less than a round: where it was measured to pay
    if (tiles64 < 256 && !(two && tiles64 >= 150) && !(tiles64 > 128 && g.K >= 1024) && !(tiles64 >= 128 && !VEC)) return false;
    if (k.kind == 1 && VEC && !k.rows) return false; // 26 launches: 24 slower, by 5 to 44 %
    // 48 launches of listed columns 0.93 to 1.27 of the 64-wide tiles' time.  Runs of columns, heads, are what the fp32 loops read well:
    // T = 1248, d = 704, 9 of 11 heads of 64 88.7 / 111.0, T = 688, d = 960, 9 of 12 of 80 88.7 / 102.1; heads of 50 90.4 / 81.4
    if (k.listed && (width == 64 || g.runs)) return false;
    if (width == 128) return true;
    const int64_t steps = (int64_t)((g.K + 31) / 32) * (EPI == EPI_DUAL_ACC ? 2 : 1);
    return split_us(k, tiles64, steps) < fp32_us(k, width, tiles32, tiles64, steps);
}

// Tile of a launch: the fewest matrix cycles on the busiest CU (rounds of tiles over 256 CUs x tile area), each tile
// weighted by what its loop loses to staging and barriers.  With fewer 64-wide tiles than CUs the 32-wide ones win on
// both counts (T = 256, p = 512, d = 256: 128 tiles whose waves each run a quarter of the depth, against 32).
// Register-staged or pipelined, event times in us: gate_up at T = 1024, d = 256, p = 1500 27.7 (32 wide) / 23.0 (64), T = 2048, d = 1024,
// n = 512 49.0 / 46.8 (both 64), but T = 4096, d = 2048, n = 512 146.9 / 154.7, n = 2048 568 (128) / 596 (128); dact at T = 2048, d = 1024,
// n = 1024 50.4 / 50.1, n = 4096 164 (128) / 194 (128); down at T = 4096, d = 2048, n = 1024 146.5 (128) / 179.0 (128), T = 4096, d = 768, n = 2048
// 124.5 (64) / 137.3 (64); dX there 240 / 267; weight gradients at T = 1024, d = 2048, p = 4000 432 (128) / 498 (128), 453 / 456 (64).  The
// pipelined 128-wide tile had one workgroup a CU for the other's two.  32 x 32, four waves on a step / on a tile's depth: down 17.3 / 15.8,
// attn_dout 9.8 / 8.3 with 256 tiles, but 25.9 / 27.5 with 512 (T = 1000).
// Extents that are no multiples of 4, whole steps before / now: T = 1023, d = 510, F = 2046, p = 1025 610 / 471 us, T = 255, d = 126,
// p = 401 126 / 69, T = 101, d = 301, p = 901 201 / 110, backward masking T = 600, d = 66, p = 900 257 / 130.
template <int EPI, bool ADM, bool BDM, bool VA, bool VB>
int choose(const Dev& g, const char* name, hipStream_t s) {
    constexpr bool VEC = VA && VB;
    constexpr int NB = EPI == EPI_SWIGLU_FWD ? 2 : 1; // the pipelined tiles hold BN / 2 columns of both right operands
    const bool direct = !(BDM && g.bg && g.K > kListMax);
    auto tiles = [&](int bm, int bn) {
        return (int64_t)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * (g.nbatch > 0 ? g.nbatch : 1);
    };
    auto cost = [&](int b, int bn, double weight) {
        const int64_t t = tiles(b, bn);
        if (t * 256 > UINT32_MAX) return HUGE_VAL; // threads of one launch
        return (double)((t + 255) / 256) * b * bn * weight;
    };
    if (direct && few_tiles(g)) return launch_wave<16, 2, EPI, ADM, BDM, VA, VB>(g, name, s); // never split
    // the fp32 tile otherwise: 32, 64 or 128 wide
    const double c128 = cost(128, 128, 1.0), c32 = cost(32, 32, 1.3);
    // single floats: the tiles that direct loads fill, of 64 and 32
    const double c64 = direct ? cost(64, 64 / NB, 1.1) : HUGE_VAL, staged128 = VEC || !direct ? c128 : HUGE_VAL;
    const double staged64 = (VEC && NB == 2) || !direct ? cost(64, 64, 1.1) : HUGE_VAL;
    int width = 64;
    if (c32 < c64 && c32 < staged64 && c32 < staged128) width = 32;
    else if (staged128 <= c64 && staged128 <= staged64) width = 128;
    if (split_pays<EPI, ADM, BDM, VA, VB>(g, width, tiles(32, 32), tiles(64, 64 / NB))) {
        auto go = [&](auto listed) { // listed columns of the left operand
            constexpr bool AG = decltype(listed)::value;
            // two teams, one workgroup a CU, while the tiles leave room for it
            if (tiles(64, 64 / NB) <= 256) return launch_split<2, EPI, ADM, BDM, AG>(g, name, s);
            return launch_split<1, EPI, ADM, BDM, AG>(g, name, s);
        };
        if constexpr (ADM) {
            if (g.ag) return go(std::true_type{});
        }
        return go(std::false_type{});
    }
    if (direct) {
        if (width == 32) {
            if (!VEC || (!ADM && NB == 1 && EPI != EPI_SWIGLU_BWD && tiles(32, 32) <= 256)) return launch_wave<32, 2, EPI, ADM, BDM, VA, VB>(g, name, s);
            return launch<Cfg<32, 32, 4>, EPI, ADM, BDM, true>(g, name, s);
        }
        if constexpr (VEC) {
            if (width == 128) return launch<Cfg<128, 128, 1>, EPI, ADM, BDM, true>(g, name, s);
            if ((BDM && !ADM) || (staged64 <= c64 && tiles(64, 64) > 256)) return launch<Cfg<64, 64, 1>, EPI, ADM, BDM, true>(g, name, s);
        }
        return launch_pipe<64, 64 / NB, EPI, ADM, BDM, VA, VB>(g, name, s);
    }
    if constexpr (BDM) { // a list too long for LDS
        if (width == 32) return launch<Cfg<32, 32, 4>, EPI, ADM, BDM, VEC>(g, name, s);
        if (width == 64) return launch<Cfg<64, 64, 1>, EPI, ADM, BDM, VEC>(g, name, s);
        return launch<Cfg<128, 128, 1>, EPI, ADM, BDM, VEC>(g, name, s); // beyond the split tiles' 2^23, which leave nothing else to it
    }
    return SDP_ERR_INVALID_ARG; // not reached
}
template <int EPI, bool ADM, bool BDM>
int choose(bool va, bool vb, const Dev& g, const char* name, hipStream_t s) {
    if (va && vb) return choose<EPI, ADM, BDM, true, true>(g, name, s);
    if constexpr (BDM) {
        if (vb) return choose<EPI, ADM, BDM, false, true>(g, name, s);
    }
    return choose<EPI, ADM, BDM, false, false>(g, name, s);
}

// kernel arguments of a descriptor; *va, *vb: 16-byte loads can take A, B
int describe(const GemmDesc& d, Dev& g, bool* va_out, bool* vb_out) {
    if (d.M < 1 || d.N < 1 || d.K < 1) return SDP_ERR_SHAPE;
    if (d.nbatch < 0 || d.nbatch > kMaxBatch || d.Cc || d.Ct) return SDP_ERR_UNSUPPORTED;
    g = Dev{};
    g.M = d.M, g.N = d.N, g.K = d.K;
    g.A = (const float*)d.A, g.A2 = (const float*)d.A2, g.B = (const float*)d.B, g.B2 = (const float*)d.B2;
    g.lda = d.lda, g.ldb = d.ldb, g.ag = d.a_gather, g.bg = d.b_gather, g.cs = d.c_scatter, g.runs = d.a_gather_chunks;
    g.C = (float*)d.C, g.C2 = (float*)d.C2, g.C3 = (float*)d.C3, g.ldc = d.ldc;
    g.Gin = (const float*)d.Gin, g.Uin = (const float*)d.Uin, g.ldg = d.ldg;
    g.R = (const float*)d.R, g.ldr = d.ldr;
    g.nbatch = d.nbatch;
    auto al = [](const void* p) { return !p || aligned16(p); };
    bool va = al(d.A) && al(d.A2), vb = al(d.B) && al(d.B2), vo = al(d.C) && al(d.C2) && al(d.C3);
    for (int z = 0; z < d.nbatch; ++z) {
        g.Ab[z] = (const float*)d.Ab[z], g.Bb[z] = (const float*)d.Bb[z], g.Cb[z] = (float*)d.Cb[z];
        va = va && al(d.Ab[z]), vb = vb && al(d.Bb[z]), vo = vo && al(d.Cb[z]);
    }
    // along the contiguous axis: the depth for an operand stored by rows, M or N for a depth-major one
    *va_out = va && d.lda % 4 == 0 && (d.a_km ? d.M : d.K) % 4 == 0 && !(d.a_km && d.a_gather);
    *vb_out = vb && d.ldb % 4 == 0 && (d.b_km ? d.N : d.K) % 4 == 0;
    g.vec_out = vo && d.N % 4 == 0 && d.ldc % 4 == 0 && (!d.R || (al(d.R) && d.ldr % 4 == 0)) &&
                (d.epilogue != EPI_SWIGLU_BWD || (al(d.Gin) && al(d.Uin) && d.ldg % 4 == 0));
    return SDP_OK;
}

// dX (BX x BX tiles, four waves on each) and one or two launches' worth of weight gradients (BW = 32: four waves on a tile;
// 64: pipelined; kOneStage: 32 in one stage; kSplit: 64, sdp_f32_split.h).  VX: 16-byte loads for both operands of dX; WA, WB: for the weight gradients'.
constexpr int kSplit = -64, kOneStage = -32;
template <int BX, int EPIX, int BW, bool VX, bool WA, bool WB>
struct GroupShape {
    typedef WaveShape<BX, 2, EPIX, false, true, VX, VX> X;
    static constexpr int W = BW == 32       ? WaveShape<32, 2, EPI_STORE, true, true, WA, WB>::TILES
                             : BW == kOneStage ? WaveShape<32, 1, EPI_STORE, true, true, WA, WB>::TILES
                             : BW == kSplit ? SplitTile<1, EPI_STORE, true, true, false>::LDS
                                            : PipeShape<64, 64, EPI_STORE, true, true, WA, WB, false>::RING;
    static constexpr int LDS = X::LDS > W ? X::LDS : W;
};
template <int BW, bool WA, bool WB>
__device__ inline void group_gradients(const Dev& w, int b, unsigned char* lds) {
    if constexpr (BW == 32) wave_body<32, 2, EPI_STORE, true, true, WA, WB>(w, b, lds);
    else if constexpr (BW == kOneStage) wave_body<32, 1, EPI_STORE, true, true, WA, WB>(w, b, lds);
    else if constexpr (BW == kSplit && WA) SplitTile<1, EPI_STORE, true, true, false>::run(w, b, lds); // 16-byte loads: columns in order
    else if constexpr (BW == kSplit) {
        if (w.ag) SplitTile<1, EPI_STORE, true, true, true>::run(w, b, lds);
        else SplitTile<1, EPI_STORE, true, true, false>::run(w, b, lds);
    } else pipe_body<64, 64, EPI_STORE, true, true, WA, WB, false>(w, b, lds);
}
template <int BX, int EPIX, int BW, bool VX, bool WA, bool WB>
__global__ __launch_bounds__(256) void gemm_f32_group_kernel(Dev x, Dev w0, Dev w1, int nx, int n0) {
    extern __shared__ __attribute__((aligned(16))) unsigned char group_lds[];
    const int b = blockIdx.x;
    if (b < nx) wave_body<BX, 2, EPIX, false, true, VX, VX>(x, b, group_lds);
    else if (b < nx + n0) group_gradients<BW, WA, WB>(w0, b - nx, group_lds);
    else group_gradients<BW, WA, WB>(w1, b - nx - n0, group_lds);
}

int64_t count_tiles(const Dev& g, int b) {
    return (int64_t)((g.M + b - 1) / b) * ((g.N + b - 1) / b) * (g.nbatch > 0 ? g.nbatch : 1);
}
struct Group {
    Dev x, w0, w1;
    int n; // launches' worth: 2 or 3
    const char *name, *name_x, *name_w; // of the launch; what dX and the weight gradients would be called alone
    hipStream_t s;
};
template <int BX, int EPIX, int BW, bool VX, bool WA, bool WB>
int launch_group(const Group& a) {
    typedef GroupShape<BX, EPIX, BW, VX, WA, WB> Sh;
    Dev x = a.x, w0 = a.w0, w1 = a.w1;
    const int lx = x.bg ? Sh::X::LDS : Sh::X::TILES, lds = lx > Sh::W ? lx : Sh::W;
    auto tiles = [](Dev& g, int b) {
        g.tiles_m = (g.M + b - 1) / b, g.tiles_n = (g.N + b - 1) / b;
        return count_tiles(g, b);
    };
    constexpr int BT = BW == kSplit ? 64 : BW == kOneStage ? 32 : BW;
    const int64_t nx = tiles(x, BX), n0 = tiles(w0, BT), n1 = a.n > 2 ? tiles(w1, BT) : 0;
    if (nx + n0 + n1 > 0x7FFFFFFF) return SDP_ERR_SHAPE;
    auto kern = gemm_f32_group_kernel<BX, EPIX, BW, VX, WA, WB>;
    static const hipError_t attr = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, Sh::LDS);
    if (attr != hipSuccess) return SDP_ERR_HIP;
    profile_shape(a.name_x, BX, BX, 0, F32_WAVES);
    profile_shape(a.name_w, BT, BT, 0, BW == kSplit ? F32_SPLIT : BW == kOneStage ? F32_WAVES_ONE_STAGE : BW == 32 ? F32_WAVES : F32_PIPELINED);
    ProfileScope ps(a.name, a.s);
    kern<<<(unsigned)(nx + n0 + n1), 256, lds, a.s>>>(x, w0, w1, (int)nx, (int)n0);
    return launch_status();
}
template <int BX, int EPIX>
int launch_group(const Group& a, bool vx, bool wa, bool wb) {
    // Weight gradients on 64 x 64 tiles where these are many for the depth of each: a tile's time is its depth's.  32-wide / 64-wide,
    // by tiles of 64 and steps of 32: 768, 4 (T = 128, d = 512, p = 2000) 32.8 / 25.9 us, 360, 16 57.6 / 56.1, an attention's 256, 16
    // 32.6 / 28.7; but 231, 16 (T = 512, d = 448) 37.5 / 47.5, 288, 32 58.4 / 66.8, 96, 16 19.3 / 22.4.
    const int64_t t64 = count_tiles(a.w0, 64) + (a.n > 2 ? count_tiles(a.w1, 64) : 0);
    const bool wide = t64 >= 16 * (int64_t)((a.w0.K + 31) / 32);
    const int64_t all = count_tiles(a.x, BX) + count_tiles(a.w0, 32) + (a.n > 2 ? count_tiles(a.w1, 32) : 0); // of dX's and 32-wide ones
    // Split products from 150 tiles and a depth of 448 on: 64-wide before / split 53.6 / 49.0 (528, 512 deep), 39.2 / 35.7 (288, 434, single
    // floats), 67.0 / 58.7 (432, 835), but 34.4 / 36.0 (384, 400), 15.6 / 17.5 (384, 128); 32-wide / split 33.7 / 29.7 (216, 600), 33.1 / 28.8
    // (195, 698), single floats 48.0 / 31.9 (210, 592).  Not where 32-wide tiles with 16-byte loads nearly fit the chip at once: 31.1 / 34.5
    // (168, 948; 798 tiles in all), 34.1 / 37.2 (153, 1048; 660), but 43.2 / 39.2 (153, 1136; 828).  Not listed columns, whose loads cost the
    // split tiles most, instead of 64-wide ones: T = 468, d = 220, p = 1536 35.6 / 43.9, T = 502, d = 235, p = 1441 51.4 / 57.8; with 32-wide ones
    // T = 558, d = 388, p = 737 43.6 / 35.0.  Nor, with 16-byte loads of the rest, beside more than 400 16-wide tiles of dX (T = 504,
    // d = 216, p = 776 24.7 / 32.0, T = 461, d = 232, p = 796 30.7 / 35.1; with 273, T = 609, d = 112, p = 2249, 46.2 / 36.7) and not heads (512
    // tokens, 3 of 4 of 128 29.6 / 31.0).
    const bool fits = vx && wa && wb && all <= 800;
    const bool listed = a.w0.ag && (wide || (vx && wb && (a.w0.runs || (BX == 16 && count_tiles(a.x, 16) > 400))));
    const bool split = t64 >= 150 && a.w0.K >= 448 && a.w0.M >= 64 && a.w0.N >= 64 && !fits && !listed;
    auto go = [&](auto bw) {
        constexpr int BW = decltype(bw)::value;
        if (vx && wa && wb) return launch_group<BX, EPIX, BW, true, true, true>(a);
        if (vx && wb) return launch_group<BX, EPIX, BW, true, false, true>(a);
        return launch_group<BX, EPIX, BW, false, false, false>(a);
    };
    if (split) return go(std::integral_constant<int, kSplit>{});
    if (wide) return go(std::integral_constant<int, 64>{});
    // 32-wide ones with one LDS stage where the launch then fits the chip at once, three workgroups a CU instead of two, unless dX's depth is
    // so long beside the gradients' that the launch ends with it, slowed down by a third workgroup.  42 shapes of 513 to 768 tiles, forward and
    // backward masking, two stages / one: T = 256, d = 256, p = 512 10.2 / 9.8 us, T = 200, d = 452, p = 140 10.6 / 8.9 and 12.0 / 9.9, T = 592,
    // d = 133, p = 705 31.5 / 26.8 and 33.9 / 26.3 (median 14 % less), but T = 424, d = 121, p = 849 24.5 / 25.2, T = 256, d = 153, p = 861
    // 22.3 / 23.3 and 19.4 / 20.9.  Listed columns (backward masking) load longer: T = 288, d = 217, p = 677 22.1 / 21.9 and 21.6 / 19.8.
    if constexpr (BX == 16) {
        const int64_t depth = (int64_t)a.x.K * (EPIX == EPI_DUAL_ACC ? 2 : 1);
        if (all > 512 && all <= 768 && depth <= (a.w0.ag ? 6 : 4) * (int64_t)a.w0.K) return go(std::integral_constant<int, kOneStage>{});
    }
    return go(std::integral_constant<int, 32>{});
}

} // namespace

int gemm_f32_group(const GemmDesc* d, int n, const char* name, hipStream_t s) {
    if (n < 2 || n > 3) return SDP_ERR_UNSUPPORTED;
    Dev g[3] = {};
    bool va[3] = {true, true, true}, vb[3] = {true, true, true};
    for (int i = 0; i < n; ++i) {
        const int rc = describe(d[i], g[i], &va[i], &vb[i]);
        if (rc != SDP_OK) return rc;
        if (!d[i].b_km || (d[i].b_gather && (i > 0 || d[i].K > kListMax))) return SDP_ERR_UNSUPPORTED;
        if (i == 0 ? d[i].a_km || d[i].nbatch > 0 || (d[i].epilogue != EPI_STORE && d[i].epilogue != EPI_DUAL_ACC)
                   : !d[i].a_km || d[i].epilogue != EPI_STORE)
            return SDP_ERR_UNSUPPORTED;
        // one tile for both launches' worth of weight gradients, chosen from the first's extents
        if (i == 2 && (d[1].M != d[2].M || d[1].N != d[2].N || d[1].K != d[2].K)) return SDP_ERR_UNSUPPORTED;
    }
    // Worth it while d[0] alone leaves room on the chip.  Launches of 512 x 512 outputs, depth 2 x 1376, beside three of
    // 1376 x 512, depth 512: step 114 -> 109 us; 1000 x 512, depth 2 x 1600 (512 tiles of 32 x 32, two on every CU): 209 ->
    // 215 us.
    const bool few = few_tiles(g[0]);
    if (!few && (int64_t)((d[0].M + 31) / 32) * ((d[0].N + 31) / 32) > 256) return SDP_ERR_UNSUPPORTED;
    const Group a{g[0], g[1], g[2], n, name, d[0].name, d[1].name, s};
    const bool vx = va[0] && vb[0], wa = va[1] && va[2], wb = vb[1] && vb[2];
    if (d[0].epilogue == EPI_DUAL_ACC) return few ? launch_group<16, EPI_DUAL_ACC>(a, vx, wa, wb) : launch_group<32, EPI_DUAL_ACC>(a, vx, wa, wb);
    return few ? launch_group<16, EPI_STORE>(a, vx, wa, wb) : launch_group<32, EPI_STORE>(a, vx, wa, wb);
}

int gemm_f32(const GemmDesc& d, hipStream_t s) {
    Dev g;
    bool va, vb;
    const int rc = describe(d, g, &va, &vb);
    if (rc != SDP_OK) return rc;
    switch (d.epilogue) {
    case EPI_STORE:
        if (d.a_km) return d.b_km ? choose<EPI_STORE, true, true>(va, vb, g, d.name, s) : SDP_ERR_UNSUPPORTED;
        return d.b_km ? choose<EPI_STORE, false, true>(va, vb, g, d.name, s) : choose<EPI_STORE, false, false>(va, vb, g, d.name, s);
    case EPI_DUAL_ACC: return d.a_km || !d.b_km ? SDP_ERR_UNSUPPORTED : choose<EPI_DUAL_ACC, false, true>(va, vb, g, d.name, s);
    case EPI_SWIGLU_FWD: return d.a_km || d.b_km ? SDP_ERR_UNSUPPORTED : choose<EPI_SWIGLU_FWD, false, false>(va, vb, g, d.name, s);
    case EPI_SWIGLU_BWD: return d.a_km || d.b_km ? SDP_ERR_UNSUPPORTED : choose<EPI_SWIGLU_BWD, false, false>(va, vb, g, d.name, s);
    }
    return SDP_ERR_INVALID_ARG;
}

} // namespace sdp
