// bf16 MFMA contraction for gfx950 (CDNA4) with the masked-MLP row gather and SwiGLU epilogues fused.
//
//   C[M][N] = sum_k A(m,k) B(k,n),  bf16 operands, fp32 accumulation in v_mfma_f32_16x16x32_bf16.
//   A is stored [M][K], B is stored [N][K] (rows optionally gathered through an index table): both
//   operands are read along the depth, 16 bytes (8 bf16) at a time.
//
// Tile: BM x BN outputs per workgroup, depth step 64, WAVES_M x WAVES_N waves of 64 lanes, each wave
// owning (BM/WAVES_M) x (BN/WAVES_N) outputs as 32 x 32 blocks of four 16 x 16 MFMA tiles.  The flagship shape is
// 256 x 256 with 8 waves: 128 accumulator registers per lane, two waves per SIMD, one workgroup per CU.  Launches that
// it would leave on few CUs take 128-row tiles of 8 waves, or 64 x 64 tiles whose 4 waves each run their own depth steps
// (choose_shape has the rule and the times).
//
// HBM/L2 -> LDS: direct loads (global_load_lds_dwordx4).  One wave instruction moves 64 chunks of
// 16 bytes into 1 KB of consecutive LDS ("slab"); which global chunk a lane fetches is free, so the
// LDS layout below is produced by choosing the global address per lane.  No registers and no
// ds_write instructions are spent on staging.  LDS holds two stages of A and three of B (three and three for the
// 128-row tiles, two and two per wave for the 64 x 64 tile).
//
// Depth-major operands (the weight gradients: dG, dU, Act, Q, K, V gradients, O, X and dY are [T][..] and the depth is T): a
// stage holds 64 depth rows of the tile's columns, and a lane's 8 consecutive k of one column come from two transposing
// LDS reads (ds_read_b64_tr_b16; read_km).  No transposed copies are made of them.
//
// LDS layout of a row-major operand stage, [R rows][64 k] in 16-byte chunks: chunk (r, c) sits at
// r*8 + (c ^ ((r >> 1) & 7)).  A lane's MFMA operand (8 consecutive k of one row) is one chunk, one
// ds_read_b128, and the lanes served together fall on distinct banks.
//
// Main loop of the 256-row tiles: the waves form two groups that alternate between a phase of LDS reads + load issue and a
// phase of MFMAs only, one phase apart, so that on every SIMD one wave computes while the other one
// fetches (see the comment at the loop).  128-row tiles: every wave reads a half step ahead of its MFMAs, with one barrier a
// step.  64 x 64: each wave on its own, no barrier.
//
// The MFMA is issued with the B fragment as its first operand: a lane then holds, for one output
// row m, 4 consecutive columns n.  Epilogues go through LDS: each wave packs 32 x WN outputs as bf16
// into a private LDS strip with 8-byte writes and reads the strip back as 16-byte chunks of whole
// rows, so that every global store (and the loads of the saved pre-activations) is a coalesced
// 16-byte access.  SwiGLU and its backward are applied on the fp32 accumulators before packing; the
// backward epilogue can also write its three outputs transposed (transposing LDS reads of the strip).
//
// Workgroup -> tile mapping is XCD-aware: consecutive workgroup ids go round-robin to the 8 XCDs
// (each with its own L2), so ids are first regrouped per XCD and each XCD then walks a compact
// block of tiles (group_m tile-rows at a time, group_m chosen on the host per shape; in a batched
// launch the problems that share an operand are stacked into one matrix first) whose operand
// tiles are shared through that L2.
//
// Batching: the three weight-gradient contractions of one worker (same M x N x K, different operands)
// run as one launch of 3 x tiles workgroups, so that their few, deep tiles fill the CUs together.
#include "sdp_internal.h"
#include "sdp_swiglu.h"
#include "sdp_transpose.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <array>
#include <cstdlib>
#include <map>
#include <mutex>
#include <type_traits>
#include <vector>

namespace sdp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(1))) const void* glb_void_ptr;

constexpr int BK = 64;
constexpr int NUM_XCD = 8;

struct Dev {
    int M, N, K;
    const uint16_t *A, *A2, *B, *B2;
    int64_t lda, ldb;
    const int32_t *ag, *bg, *cs;
    HeadList heads; // of these three
    uint16_t *C, *C2, *C3;
    int64_t ldc, ldc3; // ldc3: of C3 (SWIGLU_FWD)
    const uint16_t* R; // STORE / DUAL_ACC, single problem: optional residual [M][ldr]
    int64_t ldr;
    const uint16_t *Gin, *Uin;
    int64_t ldg;
    uint16_t *Ct, *Ct2, *Ct3; // SWIGLU_BWD: neuron-major (transposed) copies [column or rank][ldct], optional
    int64_t ldct;
    const int32_t* crank; // encoded rank of every column, or null: every column is listed
    int tiles_m, tiles_n, ntot; // ntot = tiles of all problems of the launch
    int group_m, nbatch;
    int np0; // batched launches: > 0 = the first np0 problems share one B operand and the others another (see tile_of_shared)
    // batched launch (weight gradients): problem z uses Ab[z], Bb[z], Cb[z]
    const uint16_t *Ab[kMaxBatch], *Bb[kMaxBatch];
    uint16_t* Cb[kMaxBatch];
    int64_t ldab[kMaxBatch]; // depth-major A: leading dimension of each problem's
    // OP_DW_SPLIT: the depth is cut into ksplit ranges of ksteps steps; each (range, problem) is a "problem" of
    // the launch and leaves its fp32 partial sums in partial[range][problem][M][N]
    int ksplit, ksteps;
    float* partial;
    // OP_DW_TAIL: ids below n_head are whole tiles (a multiple of the CU count: the full rounds); the `tail` tiles of
    // the last round follow as tail x ksplit items, range after range, each leaving an fp32 tile in
    // partial[range][tail tile][BM][BN].  ntot counts tiles, not ids.
    int n_head, tail;
};

// two fp32 -> packed bf16, round to nearest even (the hardware's v_cvt_pk_bf16_f32)
__device__ inline uint32_t pack_bf16(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ inline u32x2 pack4(float a, float b, float c, float d) { return u32x2{pack_bf16(a, b), pack_bf16(c, d)}; }
__device__ inline float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// source of the chunks that lie beyond the depth of the matrices in a partial last step
__device__ __attribute__((aligned(256))) const uint32_t kZeroChunk[64] = {0};

// Tile order of a batched launch whose problems share B operands (the weight gradients: dG and dU against X, Act against
// dY).  Problems that share B are stacked into one matrix of (problems x tiles_m)
// tile-rows, and each such stack is walked like a single problem: group_m tile-rows at a time, down the rows
// first, then along the tile-columns.  The tiles that run together on one XCD then touch fewer distinct operand
// rows than with the problems interleaved tile by tile.  Per depth range (ksplit > 1: OP_DW_SPLIT) there are two
// stacks, problems [0, np0) and the rest; the ranges follow one another.  `batch` returns range * nbatch + problem.
__host__ __device__ inline void tile_of_shared(int lin, int tiles_m, int tiles_n, int np0, int nbatch, int ksplit,
                                               int group_m, int& batch, int& tile_m, int& tile_n) {
    const int n0 = np0 * tiles_m * tiles_n, n1 = (nbatch - np0) * tiles_m * tiles_n;
    const int range = lin / (n0 + n1);
    lin -= range * (n0 + n1);
    int first_problem = 0, stack = np0;
    if (lin >= n0) lin -= n0, first_problem = np0, stack = nbatch - np0;
    const int rows = stack * tiles_m;
    const int per_group = group_m * tiles_n;
    const int grp = lin / per_group;
    const int first = grp * group_m;
    const int gm = rows - first < group_m ? rows - first : group_m;
    const int in = lin - grp * per_group;
    const int v = first + in % gm;
    tile_n = in / gm;
    batch = range * nbatch + first_problem + v / tiles_m;
    tile_m = v % tiles_m;
    (void)ksplit;
}

// Linear-order position (see the kernel's workgroup -> tile mapping) of id `id` of the full rounds, and of the q-th
// tile of the last round: XCD x owns positions [start_x, start_x + count_x), the first n_head / 8 of them run in
// the full rounds, the rest are its tail tiles; tail tiles are numbered round-robin over the XCDs.
__host__ __device__ inline int head_position(int id, int ntiles) {
    const int x = id % NUM_XCD, j = id / NUM_XCD, base = ntiles / NUM_XCD, rem = ntiles % NUM_XCD;
    return x * base + (x < rem ? x : rem) + j;
}
__host__ __device__ inline int tail_position(int q, int ntiles, int n_head) {
    const int base = ntiles / NUM_XCD, rem = ntiles % NUM_XCD, jh = n_head / NUM_XCD, tb = base - jh;
    const int x = q < NUM_XCD * tb ? q % NUM_XCD : q - NUM_XCD * tb;
    const int i = q < NUM_XCD * tb ? q / NUM_XCD : tb;
    return x * base + (x < rem ? x : rem) + jh + i;
}

// s_waitcnt lgkmcnt(0) alone: this wave's LDS reads have returned
#define SDP_WAIT_LGKMCNT0() __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14))
// s_waitcnt vmcnt(n) alone (expcnt / lgkmcnt left at their maxima), gfx9 encoding
#define SDP_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))

// ---- depth-major operands: LDS stage [64 depth rows][COLS columns], rows without gaps, in granules of 16 columns (32 bytes).
// A fragment (16 columns x 32 depth) is two transposing reads: within each block of 16 lanes such a read hands lane n the e-th
// element (e = 0..3) of what lane 4 e + n / 4 addressed, at position n % 4 of its 8 bytes.  Lane (l16, lq) therefore addresses
// row 8 lq + l16 / 4 (+ 4), columns 4 (l16 % 4) .. of the fragment's granule and gets column l16, depths 8 lq .. 8 lq + 7.
// The 32 lanes served together touch rows {0 .. 3, 8 .. 11} (+ 4, + 16) of one granule column, 32 bytes each: granule g of
// row r sits at g ^ swizzle(r), which puts these 8 pieces on distinct groups of 8 banks.
template <int COLS>
__device__ inline int km_swizzle(int row) {
    static_assert(COLS % 64 == 0, "whole blocks of 4 granules");
    // rows a multiple of 256 bytes apart start on the same bank, odd multiples of 128 bytes alternate between two halves
    return COLS % 128 == 0 ? (row & 3) | ((row >> 3) & 1) << 2 : ((row >> 1) & 1) | ((row >> 3) & 1) << 1;
}
// the row and column of the 16-byte chunk that a direct load puts at chunk position q of the stage
template <int COLS>
__device__ inline void km_chunk(int q, int& row, int& col) {
    row = q / (COLS / 8);
    const int c = q % (COLS / 8);
    col = (((c >> 1) ^ km_swizzle<COLS>(row)) * 2 + (c & 1)) * 8;
}
// byte offset of this lane's first read of the fragment in granule g (depths 0 .. 31)
template <int COLS>
__device__ inline int km_offset(int g, int l16, int lq) {
    const int row = 8 * lq + (l16 >> 2);
    return row * COLS * 2 + (g ^ km_swizzle<COLS>(row)) * 32 + (l16 & 3) * 8;
}
template <int COLS>
__device__ inline bf16x8 read_km(const unsigned char* stage, int offset, int s) {
    const unsigned char* p = stage + offset + s * 32 * COLS * 2;
    const u32x2 a = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p));
    const u32x2 b = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * COLS * 2)));
    return __builtin_bit_cast(bf16x8, u32x4{a[0], a[1], b[0], b[1]});
}

// One direct load: 64 lanes x 16 bytes from base + off (per lane; the zero chunk where `zero`) to 1 KB of LDS at dst.
// kAsm: written out, for the kernels with transposing reads.  The compiler does not tell the stages apart and puts a wait for all
// direct loads in flight in front of every group of such reads (not in front of ordinary ones): 128 x 128 tiles 2 x slower, 128 x 256
// 2.2 x.  The instruction has no output register, reads its address and M0 as it is issued, and is waited for by the loop's own
// counts (SDP_WAIT_VMCNT), which are the same for both forms; the memory clobber keeps LDS accesses on their side of it.
// Its hazards are met inside the block, where the compiler adds no wait states.  A scalar base that the vector unit wrote may be
// read by a memory instruction only five wait states later, but by a scalar move at once: the load takes a copy made here.  That
// move is also the wait state between the write of M0 and the load.  (In the place of an s_nop: no instruction more.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm" // M0 among the clobbers is reserved: nothing else in these kernels holds a value in it
// The LDS address of dst, as that of the workgroup's first byte plus an offset: a 32-bit addition (from a pointer to dst it is a
// 64-bit one, a comparison against null and a selection, three scalar instructions more a load: two workers at T = 512,
// d = 1024, F = 5504 under backward masking 252 -> 248.5 us, T = 256, d = 768, p = 1024 86 -> 83, 2 % at most, larger launches the same).
struct LdsBase {
    unsigned char* first;
    uint32_t address;
};
template <bool kAsm, bool kTail>
__device__ __attribute__((always_inline)) inline void direct_load(const unsigned char* base, uint32_t off, bool zero, unsigned char* dst, LdsBase lds) {
    const unsigned char* src = kTail && zero ? (const unsigned char*)kZeroChunk : base + off;
    if constexpr (!kAsm) {
        __builtin_amdgcn_global_load_lds((glb_void_ptr)src, (lds_void_ptr)dst, 16, 0, 0);
    } else {
        const uint32_t m0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds.address + (uint32_t)(dst - lds.first)));
        if constexpr (kTail) {
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(m0), "v"(src) : "memory", "m0");
        } else {
            const uint64_t a = (uint64_t)base; // the same in all lanes
            const uint64_t u = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32) |
                               (uint32_t)__builtin_amdgcn_readfirstlane((int)a);
            uint64_t copy;
            asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0"
                         : "=&s"(copy) : "s"(m0), "v"(off), "s"(u) : "memory", "m0");
        }
    }
}
#pragma clang diagnostic pop

// MFMA m of a wave's ni x nj accumulator tiles: strips of two A fragments, back and forth along B, so that of two MFMAs in a row one
// operand stays.  Large launches are limited by power, and operands that change cost some: MFMAs alone on N(0, 1) operands
// 2020 TFLOP/s with A kept for four and both changed then, 2075 back and forth without strips, 2095 so; whole passes 1.0 to 1.4 %
// (eight workers at T = 16384, d = 2048, F = 5504, backward masking 19935 -> 19665 us; its contractions take the same cycles at 0.4 to 2.6 % more
// clock, and the same time as before on all-zero operands).  Strips of two B fragments: the same.
struct TileAt {
    int i, j;
};
__device__ constexpr TileAt mfma_order(int ni, int nj, int m) {
    // 128 x 128 tiles, the ones of short launches: one A fragment after the other, as the second one is read last (86 passes of 64 to 3000
    // tokens, d = 256 .. 2048, in strips 0.7 % slower in the median: gate_up 0.5 %, attention projections 2.2 %, weight gradients 1.2 %)
    if (ni == 2 && nj == 4) return {m / nj, m / nj ? nj - 1 - m % nj : m % nj};
    const int strip = m / (2 * nj), r = m % (2 * nj), j = r / 2;
    return {2 * strip + ((r ^ j) & 1), strip % 2 ? nj - 1 - j : j};
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int KM>
struct Geometry {
    static constexpr int NW = WAVES_M * WAVES_N;
    static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    static constexpr int FM = WM / 32, FN = WN / 32;
    static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
    static constexpr bool kWaveDepth = BM == 64; // each wave runs its own depth steps on the whole tile (see the loop)
    // fragments read a half step ahead, one barrier a step (see the loop).  With both operands depth-major also the 256 x 192
    // tile, whose reads are twice as many there: 2048 x 1536 outputs x 3, 8192 deep 170 -> 162 us (the one shape it was timed
    // at); 256 x 256 no faster (135 us both ways at 2664 x 1600 x 3, 5000 deep) and short of registers
    static constexpr bool kPipe = BM == 128 || (KM == 3 && BN == 192);
    static constexpr int A_STAGES = BM == 128 ? 3 : 2; // LDS stages of A; B has three
    // kWaveDepth: two stages of both operands per wave
    static constexpr int RING = kWaveDepth ? 2 * NW * (A_BYTES + B_BYTES) : A_STAGES * A_BYTES + 3 * B_BYTES;
    // epilogue strip: 32 rows x SW columns of bf16, rows padded by 8 bytes
    static constexpr int SW = EPI == EPI_SWIGLU_FWD ? WN / 2 : WN;
    static constexpr int RS = SW * 2 + 8;
    static constexpr int STRIP = 32 * RS;
    static constexpr int NSTRIP = EPI == EPI_SWIGLU_BWD ? 3 : 1; // strips per wave
    static constexpr int RANKTAB = EPI == EPI_SWIGLU_BWD ? SW * 4 : 0; // per wave: output row of each strip column
    static constexpr int WAVE_LDS = NSTRIP * STRIP + RANKTAB;
    static constexpr int LDS = RING > NW * WAVE_LDS ? RING : NW * WAVE_LDS;
    static_assert(LDS <= 160 * 1024, "LDS of one CU");
};

// Transposes carried by a launch (the MLP's gate_up, dact and weight gradients): workgroups from g.ntot on do `side_tiles`
// tiles at a time.
struct NoSide {};
constexpr bool carries_side(int op) { return op == OP_GATE_UP || op == OP_DACT || op == OP_DW; }
// the launches of the attention block, whose lists may be of heads
constexpr bool takes_heads(int op) { return op == OP_DOWN || op == OP_DW || op == OP_DW_SPLIT; }
template <int OP>
using SideArg = std::conditional_t<carries_side(OP), SideJobs, NoSide>;
// tiles each 256 threads of a workgroup take at once: as many as the contraction's LDS holds, at most 8 (64 registers)
constexpr int side_tiles(int threads, int lds) {
    return lds / (threads / 256 * kTransposeLds) < 8 ? lds / (threads / 256 * kTransposeLds) : 8;
}

// One workgroup's tile (id `block` of the launch).  KM: bit 0 = A is depth-major ([K][lda]), bit 1 = B is, bit 2 = B's depth rows
// are listed (b_gather)
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int OP, int KM>
__device__ __attribute__((always_inline)) inline void gemm_tile(const Dev& g, const int block, unsigned char* const smem) {
    using Geo = Geometry<BM, BN, WAVES_M, WAVES_N, EPI, KM>;
    constexpr int NW = Geo::NW, WM = Geo::WM, WN = Geo::WN, FM = Geo::FM, FN = Geo::FN;
    constexpr int A_BYTES = Geo::A_BYTES, B_BYTES = Geo::B_BYTES;
    constexpr bool kFwd = EPI == EPI_SWIGLU_FWD;
    constexpr bool kWaveDepth = Geo::kWaveDepth;
    constexpr bool kAkm = (KM & 1) != 0, kBkm = (KM & 2) != 0, kBList = (KM & 4) != 0;
    static_assert(KM == 0 || EPI == EPI_STORE || (EPI == EPI_DUAL_ACC && !kAkm), "depth-major operands: store epilogues only");
    static_assert(!kBList || (kBkm && !kAkm), "a list of depth rows");
    constexpr int SA = (BM / 8) / NW;  // A slabs (1 KB) per wave per step
    constexpr int SB = (BN / 8) / NW;  // B slabs per wave per step
    static_assert((BM / 8) % NW == 0 && (BN / 8) % NW == 0, "slabs must divide among the waves");
    static_assert(!kFwd || FN % 2 == 0, "gate/up fragments come in pairs");
    const LdsBase lds_base{smem, (uint32_t)(uintptr_t)(lds_void_ptr)smem};
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6); // wave-uniform: keeps what derives from it scalar
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int l16 = lane & 15, lq = lane >> 4; // the MFMA's lane coordinates: index along the 16 rows, depth / output quarter

    // ---- workgroup -> (problem of the batch, tile), XCD-aware ----
    // Ids congruent mod 8 share an XCD: XCD x is given the contiguous range [start_x, start_x + count_x)
    // of a linear order in which the problems of a batch vary fastest, then group_m tile-rows, then the
    // tile-columns: the tiles that run together on one XCD then form a compact block of (problems x
    // tile-rows x tile-columns) whose operand rows are fetched into that XCD's L2 once.
    constexpr bool kTail = OP == OP_DW_TAIL;
    int bid = block;
    bool cut = false;  // OP_DW_TAIL: this workgroup computes one depth range of a tile of the last round
    int tail_part = 0, tail_q = 0;
    if (kTail && bid >= g.n_head) {
        cut = true;
        tail_part = (bid - g.n_head) / g.tail, tail_q = (bid - g.n_head) % g.tail;
        bid = tail_position(tail_q, g.ntot, g.n_head);
    } else {
        bid = head_position(bid, g.ntot);
    }
    constexpr bool kBatched = OP == OP_DW || OP == OP_DW_SPLIT || kTail;
    constexpr bool kSplit = OP == OP_DW_SPLIT;
    const int nb = kBatched ? g.nbatch * (kSplit ? g.ksplit : 1) : 1;
    int tile_m, tile_n, batch;
    if (kBatched && g.np0 > 0) {
        tile_of_shared(bid, g.tiles_m, g.tiles_n, g.np0, g.nbatch, g.ksplit, g.group_m, batch, tile_m, tile_n);
    } else {
        const int per_group = g.group_m * g.tiles_n * nb;
        const int grp = bid / per_group;
        const int first_m = grp * g.group_m;
        const int gm = g.tiles_m - first_m < g.group_m ? g.tiles_m - first_m : g.group_m;
        int in = bid - grp * per_group;
        batch = in % nb;
        in /= nb;
        tile_m = first_m + in % gm;
        tile_n = in / gm;
    }
    const uint16_t* gA = g.A;
    const uint16_t* gB = g.B;
    uint16_t* gC = g.C;
    int64_t lda = g.lda;
    int kpart = 0; // depth range of this workgroup (OP_DW_SPLIT, and the cut tiles of OP_DW_TAIL)
    if (kSplit) kpart = batch / g.nbatch, batch -= kpart * g.nbatch;
    if (kTail) kpart = tail_part;
    if (kBatched) {
        // selected by comparisons: a runtime index into a by-value kernel argument would go through scratch
        static_assert(kMaxBatch == 4, "one comparison per problem");
        gA = batch == 0 ? g.Ab[0] : (batch == 1 ? g.Ab[1] : (batch == 2 ? g.Ab[2] : g.Ab[3]));
        gB = batch == 0 ? g.Bb[0] : (batch == 1 ? g.Bb[1] : (batch == 2 ? g.Bb[2] : g.Bb[3]));
        if (kAkm) lda = batch == 0 ? g.ldab[0] : (batch == 1 ? g.ldab[1] : (batch == 2 ? g.ldab[2] : g.ldab[3]));
        gC = batch == 0 ? g.Cb[0] : (batch == 1 ? g.Cb[1] : (batch == 2 ? g.Cb[2] : g.Cb[3]));
    }
    const int m0 = tile_m * BM;
    const int n0 = kFwd ? tile_n * (BN / 2) : tile_n * BN; // SWIGLU_FWD: BN columns = BN/2 neurons x {gate, up}
    // SWIGLU_BWD with neuron-major copies: the encoded rank of each of this wave's output columns (at most two
    // per lane), fetched now so that the epilogue does not wait for it; a column outside the matrix counts as
    // not listed
    int crank_pre[2] = {-1, -1};
    if (EPI == EPI_SWIGLU_BWD && g.Ct) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = n0 + Geo::WN * wn + 64 * h + lane;
            if (64 * h < Geo::WN && c < g.N) crank_pre[h] = g.crank ? g.crank[c] : c;
        }
    }

    // ---- depth steps; a partial last step (K % 64 != 0, K % 8 == 0) reads its missing chunks from a
    // zero buffer, so that every step issues the same loads and runs all four MFMA sub-steps ----
    const int nk_all = (g.K + BK - 1) / BK;
    const bool ranged = kSplit || (kTail && cut);
    const int kt0 = ranged ? kpart * g.ksteps : 0; // first depth step of this workgroup
    const int nk1 = ranged ? (nk_all - kt0 < g.ksteps ? nk_all - kt0 : g.ksteps) : nk_all;
    const int nk = EPI == EPI_DUAL_ACC ? 2 * nk1 : nk1;

    // Accumulators: the wave's WM x WN outputs as 16 x 16 tiles of v_mfma_f32_16x16x32_bf16, grouped by 32 x 32
    // blocks (i, j): acc[i][j][q] is the tile with rows 32 i + 16 (q >> 1) .. and columns 32 j + 16 (q & 1) ..
    // (the 16 x 16 x 32 form sustains a higher clock than 32 x 32 x 16 on random operands: the same flops draw
    // less power)
    f32x4 acc[FM][FN][4];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[i][j][q] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto read_tile_frags = [&](const unsigned char* sa, const unsigned char* sb, int s, bf16x8* fa, bf16x8* fb) {
        const int off = (((4 * s + lq) ^ ((l16 >> 1) & 7)) * 16) + l16 * 128;
#pragma unroll
        for (int i = 0; i < BM / 16; ++i) {
            if constexpr (kAkm) fa[i] = read_km<BM>(sa, km_offset<BM>(i, l16, lq), s);
            else fa[i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(sa + i * 2048 + off));
        }
#pragma unroll
        for (int j = 0; j < BN / 16; ++j) {
            if constexpr (kBkm) fb[j] = read_km<BN>(sb, km_offset<BN>(j, l16, lq), s);
            else fb[j] = __builtin_bit_cast(bf16x8, *(const u32x4*)(sb + j * 2048 + off));
        }
    };
    // Offsets of a direct load's source within a depth step, and the step's depth rows / chunks it takes.  Indices beyond the
    // matrix are clamped to the last valid ones: such lanes fetch valid memory whose products only reach outputs that are
    // never stored.  Row-major: slab s of 1 KB holds tile rows 8 s .. 8 s + 7, lane -> row 8 s + lane / 8, stored chunk
    // position lane % 8.  Depth-major: chunk positions 64 s .. (km_chunk).
    // Row (depth-major: column) indices -> places in the stored matrix; the look-ups of a wave's slabs in flight together.
    constexpr bool kHeads = takes_heads(OP);
    auto look_up = [&](const int32_t* list, auto& idx) __attribute__((always_inline)) {
        if (!list) return;
        if (!kHeads || g.heads.width == 0) {
            for (int& i : idx) i = list[i];
        } else {
            for (int& i : idx) i = listed_row(list, g.heads, i);
        }
    };
    // slabs first, first + stride, ..
    auto sources_a = [&](int first, int stride, auto& off, auto& k) __attribute__((always_inline)) {
        constexpr int N = sizeof(off) / sizeof(off[0]);
        int idx[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int slab = first + stride * i;
            if constexpr (kAkm) {
                int col;
                km_chunk<BM>(64 * slab + lane, k[i], col);
                idx[i] = m0 + col < g.M ? m0 + col : g.M - 8; // M % 8 == 0, and a list moves whole chunks
            } else {
                const int r = 8 * slab + (lane >> 3);
                k[i] = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
                idx[i] = m0 + r < g.M ? m0 + r : g.M - 1;
            }
        }
        look_up(g.ag, idx);
#pragma unroll
        for (int i = 0; i < N; ++i) off[i] = (uint32_t)((kAkm ? k[i] * lda + idx[i] : idx[i] * lda + k[i]) * 2);
    };
    auto sources_b = [&](int first, int stride, auto& off, auto& k) __attribute__((always_inline)) {
        constexpr int N = sizeof(off) / sizeof(off[0]);
        int idx[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int slab = first + stride * i;
            if constexpr (kBkm) {
                int col;
                km_chunk<BN>(64 * slab + lane, k[i], col);
                idx[i] = n0 + col < g.N ? n0 + col : g.N - 8;
            } else {
                const int r = 8 * slab + (lane >> 3), n = kFwd ? n0 + (r % (BN / 2)) : n0 + r;
                k[i] = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
                idx[i] = n < g.N ? n : g.N - 1;
            }
        }
        if (!kBkm) look_up(g.bg, idx);
#pragma unroll
        for (int i = 0; i < N; ++i) off[i] = (uint32_t)((kBList ? idx[i] : kBkm ? k[i] * g.ldb + idx[i] : idx[i] * g.ldb + k[i]) * 2);
    };
    // listed depth rows: the byte offset of each row, in LDS behind the stages, to a whole number of steps
    uint32_t* const list = (uint32_t*)(smem + Geo::LDS);
    if constexpr (kBList) {
        // eight look-ups of a thread in flight together, without a branch among them: one after the other, 4000 rows cost a
        // workgroup of 256 threads 7 us
        constexpr int NT = NW * 64, U = 8;
        const int end = (g.K + BK - 1) / BK * BK;
        auto fill = [&](auto row_of) __attribute__((always_inline)) {
            for (int i0 = tid; i0 < end; i0 += U * NT) {
                int row[U];
#pragma unroll
                for (int u = 0; u < U; ++u) row[u] = row_of(i0 + u * NT < g.K ? i0 + u * NT : g.K - 1);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (i0 + u * NT < end) list[i0 + u * NT] = (uint32_t)row[u] * (uint32_t)(g.ldb * 2);
            }
        };
        if (!kHeads || g.heads.width == 0) fill([&](int i) __attribute__((always_inline)) { return g.bg[i]; });
        else fill([&](int i) __attribute__((always_inline)) { return head_row(g.bg, g.heads, i); });
        __syncthreads();
    }
    // what depth step k0 / 64 adds to an operand's base
    auto step_a = [&](int k0) __attribute__((always_inline)) { return kAkm ? (int64_t)k0 * lda * 2 : (int64_t)k0 * 2; };
    auto step_b = [&](int k0) __attribute__((always_inline)) { return kBList ? 0 : kBkm ? (int64_t)k0 * g.ldb * 2 : (int64_t)k0 * 2; };
    // and to the offsets of its chunks of B at depths k: read before the first of the loads that take them, as the written-out
    // loads keep their order with LDS reads
    auto listed = [&](int k0, const auto& k, auto& off) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < (int)(sizeof(off) / sizeof(off[0])); ++i) off[i] = kBList ? list[k0 + k[i]] : 0u;
    };
    if constexpr (kWaveDepth) {
        // ---- main loop of the 64-row tiles: wave w runs the depth steps w, w + NW, ... on the whole tile, in two LDS stages
        // of its own (no barrier); the partial tiles are then added through LDS, in wave order, every wave taking the part
        // whose epilogue it runs.  What such a launch lacks is not matrix-core time but workgroups, and its time is the
        // chain of loads of one tile: this runs NW x 2 steps of it at a time.
        static_assert(!kFwd, "no gate / up pairing inside a 64-column tile");
        constexpr int TM = BM / 16, TN = BN / 16; // fragments of the tile
        uint32_t a_off[BM / 8], b_off[BN / 8];
        int a_k[BM / 8], b_k[BN / 8];
        sources_a(0, 1, a_off, a_k);
        sources_b(0, 1, b_off, b_k);
        f32x4 part[TM][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) part[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        unsigned char* const mine = smem + wave * 2 * (A_BYTES + B_BYTES);
        auto issue = [&](int kt, int stage, auto tail_c) {
            constexpr bool TAIL = decltype(tail_c)::value;
            const bool second = EPI == EPI_DUAL_ACC && kt >= nk1;
            const int k0 = (kt0 + (second ? kt - nk1 : kt)) * BK;
            const unsigned char* abase = (const unsigned char*)(second ? g.A2 : gA) + step_a(k0);
            const unsigned char* bbase = (const unsigned char*)(second ? g.B2 : gB) + step_b(k0);
            unsigned char* st = mine + stage * (A_BYTES + B_BYTES);
            uint32_t row[BN / 8];
            listed(k0, b_k, row);
#pragma unroll
            for (int i = 0; i < BM / 8; ++i) {
                direct_load<KM != 0, TAIL>(abase, a_off[i], k0 + a_k[i] >= g.K, st + i * 1024, lds_base);
            }
#pragma unroll
            for (int j = 0; j < BN / 8; ++j) {
                direct_load<KM != 0, TAIL>(bbase, b_off[j] + row[j], k0 + b_k[j] >= g.K, st + A_BYTES + j * 1024, lds_base);
            }
        };
        // only the last step of an operand pair may end beyond the depth, and only its loads compare (T = 1000, d = 2048, p = 4128:
        // dX 77 -> 66 us, down 43 -> 40); a depth of whole steps has a loop of its own that does not ask (weight gradients of 256 x 1024,
        // 4096 deep 8.4 -> 8.2 us; two workers at T = 512, d = 1600, p = 1024 123 -> 120.5)
        auto issue_step = [&](int kt, int stage, auto whole_c) {
            const int last = nk_all - 1 - kt0;
            if (!decltype(whole_c)::value && (kt == last || (EPI == EPI_DUAL_ACC && kt == nk1 + last))) issue(kt, stage, std::true_type{});
            else issue(kt, stage, std::false_type{});
        };
        auto run = [&](auto whole_c) {
            if (wave < nk) issue_step(wave, 0, whole_c);
            if (wave + NW < nk) issue_step(wave + NW, 1, whole_c);
            int stage = 0;
            for (int kt = wave; kt < nk; kt += NW, stage ^= 1) {
                if (kt + NW < nk) SDP_WAIT_VMCNT(BM / 8 + BN / 8); else SDP_WAIT_VMCNT(0);
                __builtin_amdgcn_sched_barrier(0);
                const unsigned char* st = mine + stage * (A_BYTES + B_BYTES);
                bf16x8 ta[2][TM], tb[2][TN];
                read_tile_frags(st, st + A_BYTES, 0, ta[0], tb[0]);
                read_tile_frags(st, st + A_BYTES, 1, ta[1], tb[1]);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (h == 1) { // both halves have been read: the stage can be filled again
                        SDP_WAIT_LGKMCNT0();
                        __builtin_amdgcn_sched_barrier(0);
                        if (kt + 2 * NW < nk) issue_step(kt + 2 * NW, stage, whole_c);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            part[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tb[h][j], ta[h][i], part[i][j], 0, 0, 0);
                }
            }
        };
        if (g.K % BK == 0) run(std::true_type{}); else run(std::false_type{});
        __syncthreads(); // every wave is done with its stages
        f32x4* const parts = (f32x4*)smem; // [wave][fragment][lane]
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) parts[((wave * TM + i) * TN + j) * 64 + lane] = part[i][j];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int tm = WM / 16 * wm + 2 * i + (q >> 1);
                    const int tn = WN / 16 * wn + 2 * j + (q & 1);
                    f32x4 v = parts[(tm * TN + tn) * 64 + lane];
#pragma unroll
                    for (int w = 1; w < NW; ++w) v += parts[((w * TM + tm) * TN + tn) * 64 + lane];
                    acc[i][j][q] = v;
                }
    } else {
    // ---- per-lane global source of every slab this wave fills: byte offsets from a uniform base
    uint32_t a_off[SA], b_off[SB];
    int a_k[SA], b_k[SB]; // depth offset of this lane's chunk inside a step
    sources_a(wave, NW, a_off, a_k);
    sources_b(wave, NW, b_off, b_k);

    // LDS: the A stages, then a ring of three B stages
    unsigned char* const lds_a = smem;
    unsigned char* const lds_b = smem + Geo::A_STAGES * A_BYTES;

    // loads [first, last) of the SA (resp. SB) slabs of depth step kt; TAIL: the step may end beyond the depth.  Only the last
    // step of an operand pair does, and only its loads compare (with the compare and two selects on every load: 3208 deep
    // instead of 3200 cost a 128 x 192 tile 13 us of 26, a 256 x 192 one 3 of 42).
    auto issue_a = [&](int kt, int slot, auto tail_c, int first, int last) __attribute__((always_inline)) {
        constexpr bool TAIL = decltype(tail_c)::value;
        const bool second = EPI == EPI_DUAL_ACC && kt >= nk1;
        const int k0 = (kt0 + (second ? kt - nk1 : kt)) * BK;
        const int krem = g.K - k0;
        unsigned char* sa = lds_a + slot * A_BYTES;
        const unsigned char* abase = (const unsigned char*)(second ? g.A2 : gA) + step_a(k0);
#pragma unroll
        for (int i = 0; i < SA; ++i) {
            if (i < first || i >= last) continue;
            direct_load<KM != 0, TAIL>(abase, a_off[i], a_k[i] >= krem, sa + (wave + NW * i) * 1024, lds_base);
        }
    };
    uint32_t b_row[SB]; // listed depth rows: of the next loads of B
    auto list_b = [&](int kt) __attribute__((always_inline)) { listed(((EPI == EPI_DUAL_ACC && kt >= nk1) ? kt - nk1 : kt) * BK, b_k, b_row); };
    auto issue_b = [&](int kt, int slot, auto tail_c, int first, int last) __attribute__((always_inline)) {
        constexpr bool TAIL = decltype(tail_c)::value;
        const bool second = EPI == EPI_DUAL_ACC && kt >= nk1;
        const int k0 = (kt0 + (second ? kt - nk1 : kt)) * BK;
        const int krem = g.K - k0;
        unsigned char* sb = lds_b + slot * B_BYTES;
        const unsigned char* bbase0 = (const unsigned char*)(second ? g.B2 : gB) + step_b(k0);
        const unsigned char* bbase1 = (const unsigned char*)g.B2 + step_b(k0);
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            if (i < first || i >= last) continue;
            // SWIGLU_FWD: tile rows BN/2.. hold the up-projection rows (second matrix)
            const bool up = kFwd && 8 * (wave + NW * i) >= BN / 2;
            direct_load<KM != 0, TAIL>(up ? bbase1 : bbase0, b_off[i] + (kBList ? b_row[i] : 0u), b_k[i] >= krem, sb + (wave + NW * i) * 1024, lds_base);
        }
    };

    // B tile row where fragment j of this wave starts (wave-uniform)
    int bfrag[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        if (kFwd)
            bfrag[j] = (j & 1) * (BN / 2) + (WN / 2) * wn + 32 * (j >> 1);
        else
            bfrag[j] = WN * wn + 32 * j;
    }

    // ---- LDS read addresses.  Everything that depends on the lane is folded into a few byte
    // offsets; fragment index, depth sub-step and stage only add compile-time constants.
    // row tile: chunk (r, c) at r*8 + (c ^ ((r >> 1) & 7)); for r = base + lane%16 with base a
    // multiple of 16 the XOR term is (lane%16 >> 1) & 7 for every fragment.  A fragment is 16 rows x 32 depth:
    // lane (l16, lq) takes row l16, depth chunk 4 s + lq of the 32-deep sub-step s; the 16 lanes of one lq hit
    // every 16-byte slot of a 256-byte bank row once.
    int row_off[BK / 32];
#pragma unroll
    for (int s = 0; s < BK / 32; ++s) row_off[s] = (((4 * s + lq) ^ ((l16 >> 1) & 7)) * 16) + l16 * 128;
    const int a_base = WM * wm * 128;

    // fragment reads of sub-step s: A fragment i = rows 16 i .. of the wave's A rows, B fragment j = rows 16 j .. likewise
    int a_km[kAkm ? 2 * FM : 1], b_km[kBkm ? 2 * FN : 1]; // depth-major: this lane's offset of every fragment
    if constexpr (kAkm) {
#pragma unroll
        for (int i = 0; i < 2 * FM; ++i) a_km[i] = km_offset<BM>(WM * wm / 16 + i, l16, lq);
    }
    if constexpr (kBkm) {
#pragma unroll
        for (int j = 0; j < 2 * FN; ++j) b_km[j] = km_offset<BN>(bfrag[j >> 1] / 16 + (j & 1), l16, lq);
    }
    auto read_a = [&](const unsigned char* sa, int s, int i) __attribute__((always_inline)) {
        if constexpr (kAkm) return read_km<BM>(sa, a_km[i], s);
        else return __builtin_bit_cast(bf16x8, *(const u32x4*)(sa + a_base + i * 16 * 128 + row_off[s]));
    };
    auto read_b = [&](const unsigned char* sb, int s, int j) __attribute__((always_inline)) {
        if constexpr (kBkm) return read_km<BN>(sb, b_km[j], s);
        else return __builtin_bit_cast(bf16x8, *(const u32x4*)(sb + (bfrag[j >> 1] + 16 * (j & 1)) * 128 + row_off[s]));
    };
    // B fragment first: the accumulator tile is then indexed [n][m] in the MFMA's own layout, i.e. lane (l16, lq)
    // holds, for output row m = l16 of the tile, its columns n = 4 lq + r in element r.
    auto mfma_one = [&](bf16x8 a, bf16x8 b, int i, int j) __attribute__((always_inline)) {
        f32x4& c = acc[i >> 1][j >> 1][2 * (i & 1) + (j & 1)];
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a, c, 0, 0, 0);
    };
    auto barrier = [&]() __attribute__((always_inline)) { // the bare instruction: loads of later steps stay in flight across it
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    using std::false_type;
    using std::integral_constant;
    using std::true_type;

    if constexpr (Geo::kPipe) {
        // ---- main loop of the 128-row tiles (and see kPipe).  A depth step is two 32-deep halves; while a wave's MFMAs of one half run, its
        // fragments of the next half are read and its share of later steps' loads is issued between them, at most one of
        // either per MFMA.  One barrier a step, between the halves:
        //   first half of step k: MFMAs on (k, 0); reads of (k, 1); loads of B for step k + 2
        //   wait for the own loads of step k + 1 and the own reads of step k; barrier: step k + 1 has landed, step k is read
        //   second half: MFMAs on (k, 1); reads of (k + 1, 0); loads of A for step k + 3 (256 rows: two stages of A, k + 2)
        // A and B have three stages each; the stage of step k is filled again from that barrier on.  The phases of the
        // 256-row tiles (four barriers a step) cost such a tile more than its 8 to 16 MFMAs a phase: 4096 x 1200 outputs,
        // 3200 deep, chip at full clock, 128 x 192 tiles 39.7 -> 32.3 us, 128 x 128 57.7 -> 43.6, 128 x 256 38.4 -> 35.5
        // (256 x 192 tiles 43.0 -> 46.5: those keep the phases).  The loads issued all at once after the barrier, in front of the
        // MFMAs: 43.9 instead of 40.6 (at a lower clock).  Four or five stages: no faster.  A step's halves shared out between
        // two groups of waves, whose tiles are then twice as high (three eighths fewer LDS reads): 33.
        constexpr int NA = Geo::A_STAGES, S = 3, L = SA + SB; // stages of A and of B
        constexpr int NM = 4 * FM * FN, NR = 2 * FM + 2 * FN; // MFMAs and fragment reads of a half step
        static_assert(NR <= NM, "one read per MFMA");
        bf16x8 fa[2][2 * FM], fb[2][2 * FN];
        auto read_one = [&](int sa, int sb, int h, int r) __attribute__((always_inline)) {
            if (r < 2 * FN) fb[h][r] = read_b(lds_b + sb * B_BYTES, h, r);
            else fa[h][r - 2 * FN] = read_a(lds_a + sa * A_BYTES, h, r - 2 * FN);
        };
        // the MFMAs of half h; between them the reads of the other half from stages sa, sb and `nload` loads
        auto half_step = [&](int h, bool reads, int sa, int sb, int nload, auto load) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const bool rd = reads && m < NR;
                bool ld = false;
                if (rd) read_one(sa, sb, h ^ 1, m);
#pragma unroll
                for (int l = 0; l < nload; ++l)
                    if ((2 * l + 1) * NM / (2 * nload) == m) load(l), ld = true;
                if (rd || ld) __builtin_amdgcn_sched_barrier(0);
                const TileAt t = mfma_order(2 * FM, 2 * FN, m);
                mfma_one(fa[h][t.i], fb[h][t.j], t.i, t.j);
                if (rd || ld) __builtin_amdgcn_sched_barrier(0);
            }
        };
        int kt = 0, slot = 0, prev = S - 1, slot_a = 0; // B's stages of steps kt and kt - 1, A's of step kt
        // R: steps left after this one, at most S; TA / TB: the step of the loads of A / B may end beyond the depth
        auto step = [&](auto r_c, auto ta_c, auto tb_c) __attribute__((always_inline)) {
            constexpr int R = decltype(r_c)::value;
            if (kBList && R >= S - 1) list_b(kt + S - 1);
            half_step(0, true, slot_a, slot, R >= S - 1 ? SB : 0, [&](int l) __attribute__((always_inline)) { issue_b(kt + S - 1, prev, tb_c, l, l + 1); });
            if constexpr (R > 0) {
                // the loads younger than step kt + 1's
                constexpr int in_flight = NA == S ? (R >= S ? S - 2 : R - 1) * L : R > 1 ? SB : 0;
                __builtin_amdgcn_sched_barrier(0);
                SDP_WAIT_VMCNT(in_flight);
                SDP_WAIT_LGKMCNT0();
                barrier();
            }
            const int next = slot == S - 1 ? 0 : slot + 1, next_a = slot_a == NA - 1 ? 0 : slot_a + 1;
            half_step(1, R > 0, next_a, next, R >= NA ? SA : 0, [&](int l) __attribute__((always_inline)) { issue_a(kt + NA, slot_a, ta_c, l, l + 1); });
            __builtin_amdgcn_sched_barrier(0);
            prev = slot, slot = next, slot_a = next_a, ++kt;
        };
#pragma unroll
        for (int j = -S; j < 0; ++j) { // what the steps before the first would have issued; B of step S - 1 follows in step 0
            if (j + NA >= 0 && j + NA < nk) issue_a(j + NA, j + NA, true_type{}, 0, SA);
            if (j + S < nk && j < -1) {
                if (kBList) list_b(j + S);
                issue_b(j + S, j + S, true_type{}, 0, SB);
            }
        }
        if (nk >= S) SDP_WAIT_VMCNT(SA + SB + (NA == S ? SA : 0)); else SDP_WAIT_VMCNT(0);
        barrier();
#pragma unroll
        for (int r = 0; r < NR; ++r) read_one(0, 0, 0, r);
        constexpr integral_constant<int, S> full{};
        if constexpr (EPI == EPI_DUAL_ACC) { // the first pair of operands ends with step nk1 - 1
            while (kt + S < nk1 - 1) step(full, false_type{}, false_type{});
            if (kt + S == nk1 - 1) step(full, true_type{}, false_type{});
            if (kt + S == nk1) step(full, false_type{}, true_type{});
        }
        while (kt + S < nk - 1) step(full, false_type{}, false_type{});
        if (kt + S == nk - 1) step(full, integral_constant<bool, NA == S>{}, false_type{});
        if (kt == nk - 3) step(integral_constant<int, 2>{}, true_type{}, true_type{});
        if (kt == nk - 2) step(integral_constant<int, 1>{}, true_type{}, true_type{});
        step(integral_constant<int, 0>{}, true_type{}, true_type{});
    } else {
    bf16x8 fa[2 * FM], fb[2 * FN];
    auto read_half = [&](const unsigned char* sa, const unsigned char* sb, int h) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2 * FM; ++i) fa[i] = read_a(sa, h, i);
#pragma unroll
        for (int j = 0; j < 2 * FN; ++j) fb[j] = read_b(sb, h, j);
    };

    // ---- main loop of the 256-row tiles: two wave groups in alternating phases.
    // Group 0 = the first half of the waves, group 1 = the second half; the hardware places wave w of
    // a workgroup on SIMD w % 4, so every SIMD holds one wave of each group.  A depth step is cut into
    // two 32-deep halves.  Each wave alternates a READ phase (the 2 (FM + FN) fragment
    // reads of one half from LDS, plus its share of the direct loads of later steps) with a COMPUTE
    // phase (the 4 FM FN MFMAs of that half, at raised priority), and the two groups are one phase
    // apart: while one wave of a SIMD computes, the other one reads.  One wave alone keeps the matrix
    // core busy, so the MFMA stream never waits for LDS or for the load unit.  Every phase ends with a
    // workgroup barrier (plain s_barrier: the waits it needs are stated explicitly, and loads of later
    // steps stay in flight across it).
    //   phase 4 k     : group 0 reads (k, half 0), issues the loads of A for step k + 1
    //   phase 4 k + 1 : group 0 computes (k, 0);  group 1 reads (k, 0), issues A(k + 1)
    //   phase 4 k + 2 : group 0 reads (k, 1), issues the loads of B for step k + 2;  group 1 computes (k, 0)
    //   phase 4 k + 3 : group 0 computes (k, 1);  group 1 reads (k, 1), issues B(k + 2)
    // A has two LDS stages and B three.  Stage contents of step k are read in phases 4 k .. 4 k + 3;
    // loads into the stages of step k - 1 are issued from phase 4 k on, after the barrier that ends
    // phase 4 k - 1, before which every wave has waited for its own LDS reads.  Before that same
    // barrier every wave waits until its loads for step k have landed (loads complete in issue
    // order; only the newest SB, B of step k + 1, may still be in flight).
    const int grp = wave / (NW / 2);
    auto compute_half = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int m = 0; m < 4 * FM * FN; ++m) {
            const TileAt t = mfma_order(2 * FM, 2 * FN, m);
            mfma_one(fa[t.i], fb[t.j], t.i, t.j);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    int kt = 0, slot = 0;
    // IA / IB: step kt + 1 / kt + 2 exists; TA / TB: it may end beyond the depth
    auto step = [&](auto ia_c, auto ta_c, auto ib_c, auto tb_c) __attribute__((always_inline)) {
        constexpr bool IA = decltype(ia_c)::value;
        constexpr bool IB = decltype(ib_c)::value;
        const unsigned char* sa = lds_a + (kt & 1) * A_BYTES;
        const unsigned char* sb = lds_b + slot * B_BYTES;
        const int slot2 = slot == 0 ? 2 : slot - 1; // (kt + 2) % 3
        // READ (kt, 0)
        read_half(sa, sb, 0);
        if (IA) issue_a(kt + 1, (kt + 1) & 1, ta_c, 0, SA);
        SDP_WAIT_LGKMCNT0();
        barrier();
        // COMPUTE (kt, 0)
        compute_half();
        barrier();
        // READ (kt, 1)
        read_half(sa, sb, 1);
        if (IB) issue_b(kt + 2, slot2, tb_c, 0, SB);
        SDP_WAIT_LGKMCNT0();
        if (grp == 1) {
            if (IB) SDP_WAIT_VMCNT(SB); else SDP_WAIT_VMCNT(0);
        }
        barrier();
        // COMPUTE (kt, 1)
        compute_half();
        if (grp == 0) {
            if (IB) SDP_WAIT_VMCNT(SB); else SDP_WAIT_VMCNT(0);
        }
        barrier();
        slot = slot == 2 ? 0 : slot + 1;
        ++kt;
    };
    issue_a(0, 0, true_type{}, 0, SA);
    issue_b(0, 0, true_type{}, 0, SB);
    if (nk > 1) {
        issue_b(1, 1, true_type{}, 0, SB);
        SDP_WAIT_VMCNT(SB);
    } else {
        SDP_WAIT_VMCNT(0);
    }
    barrier();
    if (grp == 1) barrier(); // group 1 runs one phase behind
    if constexpr (EPI == EPI_DUAL_ACC) { // the first pair of operands ends with step nk1 - 1
        while (kt + 3 < nk1) step(true_type{}, false_type{}, true_type{}, false_type{});
        if (kt + 3 == nk1) step(true_type{}, false_type{}, true_type{}, true_type{});
        if (kt + 2 == nk1) step(true_type{}, true_type{}, true_type{}, false_type{});
    }
    while (kt + 3 < nk) step(true_type{}, false_type{}, true_type{}, false_type{});
    if (kt + 2 < nk) step(true_type{}, false_type{}, true_type{}, true_type{});
    if (kt + 1 < nk) step(true_type{}, true_type{}, false_type{}, false_type{});
    step(false_type{}, false_type{}, false_type{}, false_type{});
    if (grp == 0) barrier();
    }
    }

    // ================================ epilogue ================================
    // acc[i][j][q][r] = C(m, n),  m = m0 + WM wm + 32 i + 16 (q >> 1) + l16,
    //                             n = n0 + (column base of block j) + 16 (q & 1) + 4 lq + r.
    if constexpr (kSplit) {
        // fp32 partial sums of this depth range, 16 bytes (4 columns) per store; N % 8 == 0
        float* P = g.partial + ((int64_t)kpart * g.nbatch + batch) * g.M * g.N;
#pragma unroll
        for (int i = 0; i < FM; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int m = m0 + WM * wm + 32 * i + 16 * (q >> 1) + l16;
                    const int n = n0 + WN * wn + 32 * j + 16 * (q & 1) + 4 * lq;
                    if (m < g.M && n < g.N) *(f32x4*)(P + (int64_t)m * g.N + n) = acc[i][j][q];
                }
        }
        return;
    }
    if constexpr (kTail) {
        if (cut) {
            // fp32 partial tile of this depth range, tile-local [BM][BN]; rows and columns outside the matrix hold
            // what the clamped operand rows gave and are never read back
            float* P = g.partial + ((int64_t)tail_part * g.tail + tail_q) * (BM * BN);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *(f32x4*)(P + (WM * wm + 32 * i + 16 * (q >> 1) + l16) * BN + WN * wn + 32 * j + 16 * (q & 1) + 4 * lq) =
                            acc[i][j][q];
            return;
        }
    }
    __syncthreads(); // all waves are done with the operand tiles: LDS becomes per-wave strips
    constexpr int SW = Geo::SW, RS = Geo::RS;
    constexpr int CPR = SW / 8;               // 16-byte chunks per strip row
    constexpr int NCH = 32 * CPR;             // chunks per strip
    unsigned char* strip0 = smem + wave * Geo::WAVE_LDS;
    const int wcol0 = kFwd ? n0 + (WN / 2) * wn : n0 + WN * wn; // first output column of this wave's strips

    // one packed 8-byte group of a strip (this lane's 4 columns of tile q of a 32 x 32 block): row 16 (q >> 1) + l16,
    // columns cbase + 16 (q & 1) + 4 lq ..
    auto strip_put = [&](unsigned char* strip, int cbase, int q, u32x2 v) {
        *(u32x2*)(strip + (16 * (q >> 1) + l16) * RS + (cbase + 16 * (q & 1) + 4 * lq) * 2) = v;
    };
    auto strip_get = [&](const unsigned char* strip, int cbase, int q) {
        return *(const u32x2*)(strip + (16 * (q >> 1) + l16) * RS + (cbase + 16 * (q & 1) + 4 * lq) * 2);
    };
    // Global accesses of the epilogue go through buffer resources whose base is this wave's corner of the tile and
    // whose extent ends with the matrix's last row: for an offset at or beyond the extent the hardware returns zero
    // to a load and drops a store.  A lane whose columns lie outside the matrix (or whose row is dropped) is given
    // such an offset.  The accesses are then unconditional instructions, so the count of those in flight is known
    // and the wait for the next fragment row's loads leaves this row's stores in flight (behind a branch per store
    // the wait would be for everything).  Offsets inside a wave's part stay below 2^30 (see gemm_mfma_supported).
    constexpr uint32_t kOutside = 0x80000000u;
    const int wrow0 = m0 + WM * wm; // first output row of this wave
    const int wrows = g.M - wrow0 < 0 ? 0 : (g.M - wrow0 > WM ? WM : g.M - wrow0); // its rows inside the matrix
    // the base is the same in all lanes; saying so keeps the resource in scalar registers
    auto uniform_rsrc = [](const uint16_t* base, uint32_t bytes) {
        const uint64_t a = (uint64_t)base;
        const uint64_t u = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32) |
                           (uint32_t)__builtin_amdgcn_readfirstlane((int)a);
        return __builtin_amdgcn_make_buffer_rsrc((void*)u, 0, (int)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
    };
    auto wave_rsrc = [&](const uint16_t* base, int64_t ld) {
        return uniform_rsrc(base + (int64_t)wrow0 * ld + wcol0, (uint32_t)(wrows * ld * 2));
    };
    // byte offset of chunk c of fragment row 0 (rows of leading dimension ld); fragment row i lies 64 i ld bytes on
    auto chunk_offset = [&](int c, int64_t ld) {
        const int row = c / CPR, cc = c % CPR;
        return (NCH % 64 == 0 || c < NCH) && wcol0 + cc * 8 < g.N ? (uint32_t)((row * ld + cc * 8) * 2) : kOutside;
    };
    // cache policy of an epilogue access: kStream marks data this kernel touches once (non-temporal), so that it
    // does not push the operand panels, which every tile of a row or column re-reads, out of the L2
    constexpr int kKeep = 0, kStream = 2;
    // strip -> global: rows of `out` (leading dimension ld)
    auto strip_store = [&](const unsigned char* strip, uint16_t* out, int64_t ld, int i, auto policy) {
        const __amdgpu_buffer_rsrc_t rs = wave_rsrc(out, ld);
#pragma unroll
        for (int it = 0; it < (NCH + 63) / 64; ++it) {
            const int c = NCH % 64 == 0 || it * 64 + lane < NCH ? it * 64 + lane : 0;
            const int row = c / CPR, cc = c % CPR;
            const u32x2 lo = *(const u32x2*)(strip + row * RS + cc * 16);
            const u32x2 hi = *(const u32x2*)(strip + row * RS + cc * 16 + 8);
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{lo[0], lo[1], hi[0], hi[1]}, rs,
                                                   chunk_offset(it * 64 + lane, ld) + (uint32_t)(64 * i * ld), 0, decltype(policy)::value);
        }
    };
    // the same with a row scatter (a negative entry drops the row): destination rows may lie anywhere, plain stores
    auto strip_store_scatter = [&](const unsigned char* strip, uint16_t* out, int64_t ld, const int32_t* scatter, int i) {
#pragma unroll
        for (int it = 0; it < (NCH + 63) / 64; ++it) {
            const int c = it * 64 + lane;
            if (NCH % 64 != 0 && c >= NCH) break;
            const int row = c / CPR, cc = c % CPR;
            const u32x2 lo = *(const u32x2*)(strip + row * RS + cc * 16);
            const u32x2 hi = *(const u32x2*)(strip + row * RS + cc * 16 + 8);
            const int m = wrow0 + 32 * i + row, n = wcol0 + cc * 8;
            if (m < g.M && n < g.N) {
                const int64_t orow = kHeads ? listed_row(scatter, g.heads, m) : scatter[m];
                if (orow >= 0) *(u32x4*)(out + orow * ld + n) = u32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        }
    };
    // global -> registers -> strip: the same chunk mapping, zero outside the matrix.  The two halves are
    // separate so that the loads of fragment row i + 1 fly while row i is computed and stored.
    constexpr int NLD = (NCH + 63) / 64;
    auto strip_fetch = [&](u32x4 (&v)[NLD], const uint16_t* in, int64_t ld, int i, auto policy) {
        const __amdgpu_buffer_rsrc_t rs = wave_rsrc(in, ld);
#pragma unroll
        for (int it = 0; it < NLD; ++it)
            v[it] = __builtin_amdgcn_raw_buffer_load_b128(rs, chunk_offset(it * 64 + lane, ld) + (uint32_t)(64 * i * ld), 0,
                                                           decltype(policy)::value);
    };
    auto strip_commit = [&](unsigned char* strip, const u32x4 (&v)[NLD]) {
#pragma unroll
        for (int it = 0; it < NLD; ++it) {
            const int c = it * 64 + lane;
            if (NCH % 64 != 0 && c >= NCH) break;
            const int row = c / CPR, cc = c % CPR;
            *(u32x2*)(strip + row * RS + cc * 16) = u32x2{v[it][0], v[it][1]};
            *(u32x2*)(strip + row * RS + cc * 16 + 8) = u32x2{v[it][2], v[it][3]};
        }
    };

    // neuron-major copies: output row of each of this wave's SW strip columns, relative to trow0.  Without an
    // index list it is the column itself; with one (backward masking) it is the column's rank among the listed
    // columns, or -1 for columns that are not listed.  The encoded ranks were fetched before the main loop.
    int32_t* ranktab = (int32_t*)(strip0 + Geo::NSTRIP * Geo::STRIP);
    int trow0 = 0; // output row of the first (listed) column of this wave
    if (EPI == EPI_SWIGLU_BWD && g.Ct) {
        const int first = __builtin_amdgcn_readfirstlane(crank_pre[0]);
        trow0 = first >= 0 ? first : -1 - first;
#pragma unroll
        for (int h = 0; h < (SW + 63) / 64; ++h)
            if (SW % 64 == 0 || 64 * h + lane < SW) ranktab[64 * h + lane] = crank_pre[h] >= 0 ? crank_pre[h] - trow0 : -1;
    }
    // strip -> neuron-major global: out[trow0 + ranktab[column]][token].  A transposing LDS read hands the lanes
    // of a 16-lane block, for 4 adjacent strip columns, 4 consecutive rows each; two of them give every lane
    // 8 consecutive tokens of one column, i.e. one 16-byte store, and 4 lanes cover the 32 tokens (64 bytes).
    auto strip_store_t = [&](const unsigned char* strip, uint16_t* out, int i) {
        const int gi = lane >> 4, li = lane & 15, q = li >> 2, cn = li & 3;
        const int src_row = 8 * (li & 3) + (li >> 2); // as source lane: rows 8 q' + e for the lanes that receive from it
        const bool m_in = 32 * i + 8 * q < wrows;
        const __amdgpu_buffer_rsrc_t rs = uniform_rsrc(out + (int64_t)trow0 * g.ldct + wrow0, kOutside);
#pragma unroll
        for (int it = 0; it < SW / 16; ++it) {
            const int c4 = 16 * it + 4 * gi;
            const unsigned char* p = strip + src_row * RS + c4 * 2;
            const s16x4 h0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p);
            const s16x4 h1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * RS));
            const int row = ranktab[c4 + cn];
            const uint32_t off = row >= 0 && m_in ? (uint32_t)((row * g.ldct + 32 * i + 8 * q) * 2) : kOutside;
            const u32x2 a = __builtin_bit_cast(u32x2, h0), b = __builtin_bit_cast(u32x2, h1);
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{a[0], a[1], b[0], b[1]}, rs, off, 0, kKeep); // read next, by the weight-gradient launch
        }
    };

    // residual of a single-problem store (the skip connection of a block): fetched one fragment row ahead like G, U
    constexpr bool kResidual = (EPI == EPI_STORE || EPI == EPI_DUAL_ACC) && !kBatched;
    u32x4 rpre[kResidual ? NLD : 1];
    const bool has_r = kResidual && g.R != nullptr;
    if constexpr (kResidual) {
        if (has_r) strip_fetch(rpre, g.R, g.ldr, 0, std::integral_constant<int, kKeep>{});
    }
    // The fragment rows, one after the other.  kT: SWIGLU_BWD with the neuron-major copies; the loop exists once
    // per case, so that between a row's loads and the next row's use of them the stores issued are the same on
    // every path and can be left in flight.
    auto rows = [&](auto with_t) __attribute__((always_inline)) {
        constexpr bool kT = decltype(with_t)::value;
        u32x4 gpre[NLD], upre[NLD]; // SWIGLU_BWD: G and U of the next fragment row, in flight
        if (EPI == EPI_SWIGLU_BWD) {
            strip_fetch(gpre, g.Gin, g.ldg, 0, std::integral_constant<int, kStream>{});
            strip_fetch(upre, g.Uin, g.ldg, 0, std::integral_constant<int, kStream>{});
        }
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            // keep the scheduler from pulling later fragment rows' work (and its registers) up here
            __builtin_amdgcn_sched_barrier(0);
            if (EPI == EPI_STORE || EPI == EPI_DUAL_ACC) {
                if constexpr (kResidual) {
                    if (has_r) {
                        // row chunks -> strip -> each lane's own accumulator positions; added in fp32
                        strip_commit(strip0, rpre);
                        if (i + 1 < FM) strip_fetch(rpre, g.R, g.ldr, i + 1, std::integral_constant<int, kKeep>{});
                        u32x2 rq[FN][4];
#pragma unroll
                        for (int j = 0; j < FN; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q) rq[j][q] = strip_get(strip0, 32 * j, q);
#pragma unroll
                        for (int j = 0; j < FN; ++j)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                acc[i][j][q][0] += lo_bf16(rq[j][q][0]);
                                acc[i][j][q][1] += hi_bf16(rq[j][q][0]);
                                acc[i][j][q][2] += lo_bf16(rq[j][q][1]);
                                acc[i][j][q][3] += hi_bf16(rq[j][q][1]);
                            }
                    }
                }
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        strip_put(strip0, 32 * j, q,
                                  pack4(acc[i][j][q][0], acc[i][j][q][1], acc[i][j][q][2], acc[i][j][q][3]));
                if (g.cs) strip_store_scatter(strip0, gC, g.ldc, g.cs, i); else strip_store(strip0, gC, g.ldc, i, std::integral_constant<int, kKeep>{});
            } else if (EPI == EPI_SWIGLU_FWD) {
                // fragments 2 jj (gate) and 2 jj + 1 (up) cover the same 32 neurons
#pragma unroll
                for (int which = 0; which < 3; ++which) {
#pragma unroll
                    for (int jj = 0; jj < FN / 2; ++jj)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            float v[4];
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const float gv = acc[i][2 * jj][q][r], uv = acc[i][2 * jj + 1][q][r];
                                v[r] = which == 0 ? gv : (which == 1 ? uv : swiglu_fwd<false>(gv, uv));
                            }
                            strip_put(strip0, 32 * jj, q, pack4(v[0], v[1], v[2], v[3]));
                        }
                    strip_store(strip0, which == 0 ? g.C : (which == 1 ? g.C2 : g.C3), which == 2 ? g.ldc3 : g.ldc, i, std::integral_constant<int, kKeep>{});
                }
            } else { // EPI_SWIGLU_BWD: three strips per wave (dG, dU, Act)
                unsigned char* strip1 = strip0 + Geo::STRIP;
                unsigned char* strip2 = strip1 + Geo::STRIP;
                strip_commit(strip0, gpre);
                strip_commit(strip1, upre);
                if (i + 1 < FM) {
                    strip_fetch(gpre, g.Gin, g.ldg, i + 1, std::integral_constant<int, kStream>{});
                    strip_fetch(upre, g.Uin, g.ldg, i + 1, std::integral_constant<int, kStream>{});
                }
                u32x2 gq[FN][4], uq[FN][4];
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        gq[j][q] = strip_get(strip0, 32 * j, q);
                        uq[j][q] = strip_get(strip1, 32 * j, q);
                    }
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float dg[4], du[4], act[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const uint32_t gw = gq[j][q][r >> 1], uw = uq[j][q][r >> 1];
                            const float gv = (r & 1) ? hi_bf16(gw) : lo_bf16(gw);
                            const float uv = (r & 1) ? hi_bf16(uw) : lo_bf16(uw);
                            swiglu_bwd<false>(acc[i][j][q][r], gv, uv, dg[r], du[r], act[r]);
                        }
                        strip_put(strip0, 32 * j, q, pack4(dg[0], dg[1], dg[2], dg[3]));
                        strip_put(strip1, 32 * j, q, pack4(du[0], du[1], du[2], du[3]));
                        strip_put(strip2, 32 * j, q, pack4(act[0], act[1], act[2], act[3]));
                    }
                strip_store(strip0, g.C, g.ldc, i, std::integral_constant<int, kStream>{});
                strip_store(strip1, g.C2, g.ldc, i, std::integral_constant<int, kStream>{});
                if (g.C3) strip_store(strip2, g.C3, g.ldc, i, std::integral_constant<int, kStream>{});
                if constexpr (kT) {
                    strip_store_t(strip0, g.Ct, i);
                    strip_store_t(strip1, g.Ct2, i);
                    strip_store_t(strip2, g.Ct3, i);
                }
            }
        }
    };
    if constexpr (EPI == EPI_SWIGLU_BWD) {
        if (g.Ct) rows(std::true_type{}); else rows(std::false_type{});
    } else {
        rows(std::false_type{});
    }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int OP, int KM>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, BM == 64 && BN == 64 ? 2 : 1) void sdp_gemm_kernel(Dev g, SideArg<OP> side) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    if constexpr (carries_side(OP)) {
        if ((int)blockIdx.x >= g.ntot) {
            constexpr int NW = WAVES_M * WAVES_N, HALVES = NW / 4;
            constexpr int N = side_tiles(NW * 64, Geometry<BM, BN, WAVES_M, WAVES_N, EPI, KM>::LDS);
            const int half = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8);
            side_transposes<N>(side, ((int)blockIdx.x - g.ntot) * HALVES + half, smem + half * N * kTransposeLds,
                               threadIdx.x & 255);
            return;
        }
    }
    gemm_tile<BM, BN, WAVES_M, WAVES_N, EPI, OP, KM>(g, (int)blockIdx.x, smem);
}

// A single problem with a depth-major right operand (dX) and a batched launch (the weight gradients) side by side, in tiles of
// BX x BX and BW x BW (128, eight waves; 64, four waves, for which a workgroup of eight has four that leave at once: barriers wait
// for the others alone).  The longer chains come first: x_first.
template <int BX, int BW>
constexpr int pair_threads() { return BX == 128 || BW == 128 ? 512 : 256; }
template <int B, int THREADS, int EPI, int OP, int KM>
__device__ __attribute__((always_inline)) inline void pair_tile(const Dev& g, int id, unsigned char* smem) {
    if constexpr (B == 128) {
        gemm_tile<128, 128, 4, 2, EPI, OP, KM>(g, id, smem);
    } else {
        if (THREADS > 256 && threadIdx.x >= 256) return;
        gemm_tile<64, 64, 2, 2, EPI, OP, KM>(g, id, smem);
    }
}
template <int BX, int BW, int EPIX, int KMX, int KMW>
__global__ __launch_bounds__((pair_threads<BX, BW>()), 1) void sdp_gemm_pair_kernel(Dev x, Dev w, int x_first) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int id = (int)blockIdx.x, ix = x_first ? id : id - w.ntot;
    if (ix >= 0 && ix < x.ntot) pair_tile<BX, pair_threads<BX, BW>(), EPIX, EPIX == EPI_DUAL_ACC ? OP_DX : OP_DOWN, KMX>(x, ix, smem);
    else pair_tile<BW, pair_threads<BX, BW>(), EPI_STORE, OP_DW, KMW>(w, x_first ? id - x.ntot : id, smem);
}

constexpr int kNumCU = 256;

// Overrides of the tile shape and order for tuning runs.  The library's behaviour is a pure function of its
// arguments: the environment is consulted only in a build with -DSDP_TUNING_SWITCHES (never the shipped one),
// once per process, and values outside the accepted sets are ignored.
struct Tuning {
    int force_tile = 0; // SDP_FORCE_TILE: 0 = choose; 1 + a Shape
    int group_m = 0;    // 0 = choose
    bool plain_order = false;
    int tail_parts = -1; // SDP_TAIL_PARTS: -1 = choose; 0 = no tail cut; n = cut into n ranges where a cut applies
};
const Tuning& tuning() {
    static const Tuning t = [] {
        Tuning v;
#ifdef SDP_TUNING_SWITCHES
        if (const char* e = getenv("SDP_FORCE_TILE")) {
            const int f = atoi(e);
            if (f >= 1 && f <= 6) v.force_tile = f;
        }
        if (const char* e = getenv("SDP_GROUP_M")) v.group_m = atoi(e) > 0 ? atoi(e) : 0;
        v.plain_order = getenv("SDP_PLAIN_ORDER") != nullptr;
        if (const char* e = getenv("SDP_TAIL_PARTS")) v.tail_parts = atoi(e) >= 0 && atoi(e) <= 8 ? atoi(e) : -1;
#endif
        return v;
    }();
    return t;
}

// Tile-rows per group of the workgroup -> tile order: the tiles resident on one XCD at a time (its
// share of the launch, at most one per CU) form a block of nbatch x group_m x columns; pick the
// group_m for which that block touches the fewest distinct operand rows (A rows weigh na operands,
// B rows nb), i.e. the least traffic into that XCD's L2.
int choose_group_m(int tiles_m, int tiles_n, int nbatch, int na, int nb, int bm, int bn) {
    const int64_t ntot = (int64_t)tiles_m * tiles_n * nbatch;
    const int per_xcd = kNumCU / NUM_XCD;
    int64_t c = (ntot + NUM_XCD - 1) / NUM_XCD;
    if (c > per_xcd) c = per_xcd;
    int best = 1;
    int64_t best_cost = -1;
    for (int gm = 1; gm <= tiles_m && gm <= per_xcd; ++gm) {
        const int64_t cols = (c + (int64_t)nbatch * gm - 1) / ((int64_t)nbatch * gm); // tile-columns the block needs
        const int64_t groups = (cols + tiles_n - 1) / tiles_n;
        const int64_t ncols = cols < tiles_n ? cols : tiles_n;
        const int64_t cost = (int64_t)na * gm * groups * bm + (int64_t)nb * ncols * bn;
        if (best_cost < 0 || cost < best_cost) best_cost = cost, best = gm;
    }
    return best;
}

// group_m of the stacked order (tile_of_shared): the one whose first round of resident tiles (each XCD's range,
// at most one tile per CU) touches the fewest operand bytes, counted by walking that very order.
int choose_group_shared(int tiles_m, int tiles_n, int np0, int nbatch, int ksplit, int bm, int bn) {
    // the walk costs a fraction of a millisecond of host time: remembered per shape
    static std::mutex mu;
    static std::map<std::array<int, 7>, int> known;
    const std::array<int, 7> key = {tiles_m, tiles_n, np0, nbatch, ksplit, bm, bn};
    {
        std::lock_guard<std::mutex> lk(mu);
        auto it = known.find(key);
        if (it != known.end()) return it->second;
    }
    const int ntot = tiles_m * tiles_n * nbatch * ksplit;
    const int per_xcd = kNumCU / NUM_XCD;
    const int max_rows = (np0 > nbatch - np0 ? np0 : nbatch - np0) * tiles_m;
    int best = 1;
    int64_t best_cost = -1;
    std::vector<char> seen_a((size_t)ksplit * nbatch * tiles_m), seen_b((size_t)ksplit * 2 * tiles_n);
    for (int gm = 1; gm <= max_rows && gm <= 2 * per_xcd; ++gm) {
        int64_t cost = 0;
        for (int x = 0; x < NUM_XCD; ++x) {
            const int base = ntot / NUM_XCD, rem = ntot % NUM_XCD;
            const int start = x * base + (x < rem ? x : rem);
            int count = base + (x < rem ? 1 : 0);
            count = count < per_xcd ? count : per_xcd;
            std::fill(seen_a.begin(), seen_a.end(), 0);
            std::fill(seen_b.begin(), seen_b.end(), 0);
            for (int lin = start; lin < start + count; ++lin) {
                int b, tm, tn;
                tile_of_shared(lin, tiles_m, tiles_n, np0, nbatch, ksplit, gm, b, tm, tn);
                const int range = b / nbatch, z = b % nbatch; // a depth range reads its own part of every row
                char& a = seen_a[(size_t)b * tiles_m + tm];
                char& bb = seen_b[((size_t)range * 2 + (z < np0 ? 0 : 1)) * tiles_n + tn];
                if (!a) a = 1, cost += bm;
                if (!bb) bb = 1, cost += bn;
            }
        }
        if (best_cost < 0 || cost < best_cost) best_cost = cost, best = gm;
    }
    std::lock_guard<std::mutex> lk(mu);
    known[key] = best;
    return best;
}

// OP_DW_TAIL, second kernel: the depth ranges' fp32 tiles of every tile of the last round, added in range order,
// rounded and stored (optional row scatter).  One thread per 8 columns of a tile row; the tile's place in its
// problem comes from the same mapping as in the contraction kernel.
struct TailReduceArgs {
    const float* partial;
    int parts, tail, ntiles, n_head;
    int tiles_m, tiles_n, np0, nbatch, group_m;
    int M, N;
    uint16_t* Cb[kMaxBatch];
    int64_t ldc;
    const int32_t* cs;
};
template <int BM, int BN>
__global__ __launch_bounds__(256) void tail_reduce_kernel(TailReduceArgs r) {
    constexpr int PER_TILE = BM * BN / 8 / 256; // workgroups per tile
    const int q = blockIdx.x / PER_TILE;
    const int e = (blockIdx.x % PER_TILE) * 256 + threadIdx.x;
    const int row = e / (BN / 8), col = (e % (BN / 8)) * 8;
    const int bid = tail_position(q, r.ntiles, r.n_head);
    int batch, tile_m, tile_n;
    if (r.np0 > 0) {
        tile_of_shared(bid, r.tiles_m, r.tiles_n, r.np0, r.nbatch, 1, r.group_m, batch, tile_m, tile_n);
    } else {
        const int per_group = r.group_m * r.tiles_n * r.nbatch;
        const int grp = bid / per_group;
        const int first_m = grp * r.group_m;
        const int gm = r.tiles_m - first_m < r.group_m ? r.tiles_m - first_m : r.group_m;
        int in = bid - grp * per_group;
        batch = in % r.nbatch;
        in /= r.nbatch;
        tile_m = first_m + in % gm;
        tile_n = in / gm;
    }
    const int m = tile_m * BM + row, n = tile_n * BN + col;
    if (m >= r.M || n >= r.N) return;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    for (int k = 0; k < r.parts; ++k) { // ranges in depth order
        const float* p = r.partial + ((int64_t)k * r.tail + q) * (BM * BN) + row * BN + col;
        a += *(const f32x4*)p;
        b += *(const f32x4*)(p + 4);
    }
    uint16_t* out = batch == 0 ? r.Cb[0] : (batch == 1 ? r.Cb[1] : (batch == 2 ? r.Cb[2] : r.Cb[3]));
    const int64_t orow = r.cs ? r.cs[m] : m;
    if (orow < 0) return; // dropped row
    *(u32x4*)(out + orow * r.ldc + n) = u32x4{pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3]), pack_bf16(b[0], b[1]), pack_bf16(b[2], b[3])};
}

template <int BM, int BN>
int tail_reduce(const Dev& g, const GemmDesc& d, hipStream_t s) {
    TailReduceArgs r{g.partial, g.ksplit, g.tail, g.ntot, g.n_head, g.tiles_m, g.tiles_n, g.np0, g.nbatch, g.group_m,
                     g.M, g.N, {}, g.ldc, g.cs};
    for (int z = 0; z < kMaxBatch; ++z) r.Cb[z] = g.Cb[z];
    ProfileScope ps(d.tail_name, s);
    tail_reduce_kernel<BM, BN><<<(unsigned)(g.tail * (BM * BN / 8 / 256)), 256, 0, s>>>(r);
    return launch_status();
}

// Whether a launch of `tiles` tiles, `round` us a round, carries `wgs` workgroups of transposes: when the CUs that its last
// round leaves idle get through them meanwhile.  A workgroup moves 8 to 16 tiles (side_tiles); several of them one after the
// other on a CU take about 5 us each and 5 more for the first.  T = 5000, d = 1600, p = 2664 (28 us of transposes a worker beside 420 and 220 tiles): step of two workers
// 1020 -> 980 us; beside the 512 tiles of T = 8192, p = 2048, two full rounds, W2's transpose cost 12 us more than on its own.
// W1's and W3's beside the weight gradients (144 tiles; dact has 256) at T = 1024, d = 768, p = 1024: step of two workers
// 113.7 -> 107.1 us; four at T = 8192, d = 1536, p = 2048 (192 tiles) 1786 -> 1754.
bool carry(int64_t tiles, double round, int64_t wgs) {
    const int64_t idle = tiles % kNumCU ? kNumCU - tiles % kNumCU : 0;
    return idle > 0 && (double)((wgs + idle - 1) / idle) * 5.0 + 5.0 <= 1.2 * round;
}

constexpr int kMaxLds = 160 * 1024;
inline int list_bytes(int K) { return (K + BK - 1) / BK * BK * 4; }

// kernel arguments of a descriptor, for tiles of BM x BN
template <int BM, int BN, int EPI, int OP>
int describe(const GemmDesc& d, Dev& g) {
    g.M = d.M, g.N = d.N, g.K = d.K;
    g.A = (const uint16_t*)d.A, g.A2 = (const uint16_t*)d.A2, g.B = (const uint16_t*)d.B, g.B2 = (const uint16_t*)d.B2;
    g.lda = d.lda, g.ldb = d.ldb, g.ag = d.a_gather, g.bg = d.b_gather, g.cs = d.c_scatter, g.heads = d.heads;
    g.C = (uint16_t*)d.C, g.C2 = (uint16_t*)d.C2, g.C3 = (uint16_t*)d.C3, g.ldc = d.ldc;
    g.ldc3 = d.ldc3 ? d.ldc3 : d.ldc;
    g.R = (const uint16_t*)d.R, g.ldr = d.ldr;
    g.Gin = (const uint16_t*)d.Gin, g.Uin = (const uint16_t*)d.Uin, g.ldg = d.ldg;
    g.Ct = (uint16_t*)d.Ct, g.Ct2 = (uint16_t*)d.Ct2, g.Ct3 = (uint16_t*)d.Ct3, g.ldct = d.ldct;
    g.crank = d.crank;
    g.tiles_m = (d.M + BM - 1) / BM;
    const int ncols = EPI == EPI_SWIGLU_FWD ? BN / 2 : BN;
    g.tiles_n = (d.N + ncols - 1) / ncols;
    const int64_t ntiles = (int64_t)g.tiles_m * g.tiles_n;
    constexpr bool kBatched = OP == OP_DW || OP == OP_DW_SPLIT || OP == OP_DW_TAIL;
    const int ksplit = OP == OP_DW_SPLIT ? d.ksplit : 1;
    const int nbatch = (kBatched ? d.nbatch : 1) * ksplit; // problems of the launch
    if (ntiles * nbatch > 0x7FFFFFFF) return SDP_ERR_SHAPE;
    g.ntot = (int)(ntiles * nbatch);
    g.nbatch = kBatched ? d.nbatch : 1;
    g.ksplit = OP == OP_DW_TAIL ? d.ksplit : ksplit;
    g.ksteps = ((d.K + BK - 1) / BK + g.ksplit - 1) / g.ksplit;
    g.partial = (float*)(OP == OP_DW_TAIL ? d.tail_ws : d.split_ws);
    g.n_head = g.ntot, g.tail = 0;
    int na = 1, nbo = 1; // distinct A / B operands among the problems of a batch
    for (int z = 0; z < kMaxBatch; ++z) {
        g.Ab[z] = (const uint16_t*)d.Ab[z], g.Bb[z] = (const uint16_t*)d.Bb[z], g.Cb[z] = (uint16_t*)d.Cb[z];
        g.ldab[z] = d.ldab[z] ? d.ldab[z] : d.lda;
    }
    if (kBatched) {
        na = nbo = 0;
        for (int z = 0; z < d.nbatch; ++z) {
            bool newa = true, newb = true;
            for (int y = 0; y < z; ++y) newa &= d.Ab[y] != d.Ab[z], newb &= d.Bb[y] != d.Bb[z];
            na += newa, nbo += newb;
        }
    }
    g.group_m = choose_group_m(g.tiles_m, g.tiles_n, nbatch, na * ksplit, nbo * ksplit, BM, BN);
    g.np0 = 0;
    if (kBatched && d.nbatch > 1 && nbo <= 2 && !tuning().plain_order) {
        // problems that share B must be neighbours: [0, np0) on Bb[0], the rest on one other operand (or none)
        int np0 = 1;
        while (np0 < d.nbatch && d.Bb[np0] == d.Bb[0]) ++np0;
        bool ok = true;
        for (int z = np0; z < d.nbatch; ++z) ok = ok && d.Bb[z] == d.Bb[np0] && d.Bb[z] != d.Bb[0];
        if (ok) {
            g.np0 = np0;
            g.group_m = choose_group_shared(g.tiles_m, g.tiles_n, np0, d.nbatch, ksplit, BM, BN);
        }
    }
    if (tuning().group_m > 0) g.group_m = tuning().group_m;
    profile_shape(d.name, BM, BN, g.group_m, g.np0 > 0 ? 1 : 0);
    return SDP_OK;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int OP, int KM>
int launch_cfg(const GemmDesc& d, double round, hipStream_t s) {
    using Geo = Geometry<BM, BN, WAVES_M, WAVES_N, EPI, KM>;
    constexpr int NTHREADS = WAVES_M * WAVES_N * 64;
    constexpr int LDS = Geo::LDS;
    constexpr bool kBList = (KM & 4) != 0;
    const int lds = LDS + (kBList ? list_bytes(d.K) : 0);
    if (lds > kMaxLds) return SDP_ERR_INVALID_ARG;
    // what this kernel would leave undone or misread
    if ((!carries_side(OP) && d.nside > 0) || (!takes_heads(OP) && d.heads.width > 0)) return SDP_ERR_INVALID_ARG;
    Dev g;
    const int drc = describe<BM, BN, EPI, OP>(d, g);
    if (drc != SDP_OK) return drc;
    int64_t grid = (int64_t)g.ntot;
    if (OP == OP_DW_TAIL) {
        g.n_head = g.ntot / kNumCU * kNumCU, g.tail = g.ntot - g.n_head;
        grid = (int64_t)g.n_head + (int64_t)g.tail * d.ksplit;
        if (g.tail < 1 || d.ksplit < 2 || !d.tail_ws || grid > 0x7FFFFFFF) return SDP_ERR_INVALID_ARG;
    }
    SideArg<OP> side{};
    if constexpr (carries_side(OP)) {
        if (d.nside > 0) {
            constexpr int PER_WG = side_tiles(NTHREADS, LDS) * (NTHREADS / 256);
            const int t = side_jobs(d.side, d.nside, &side);
            const int64_t wgs = ((int64_t)t + PER_WG - 1) / PER_WG;
            if (t > 0 && carry(g.ntot, round, wgs) && grid + wgs <= 0x7FFFFFFF) {
                grid += wgs;
            } else {
                const int rc = transpose_batch(d.side, d.nside, d.side_name, s);
                if (rc != SDP_OK) return rc;
            }
        }
    }
    auto kern = sdp_gemm_kernel<BM, BN, WAVES_M, WAVES_N, EPI, OP, KM>;
    // once per instantiation (initialisation of a function-local static is thread-safe)
    static const hipError_t attr =
        hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kBList ? kMaxLds : LDS);
    if (attr != hipSuccess) return SDP_ERR_HIP;
    // When this kernel is being timed, the launch itself carries the two events (their timestamps are the
    // kernel's own begin and end): events recorded around the launch would put a bubble of several
    // microseconds on either side of it.
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    if (profile_launch_events(d.name, &ev0, &ev1))
        hipExtLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NTHREADS), (uint32_t)lds, s, ev0, ev1, 0u, g, side);
    else
        kern<<<dim3((unsigned)grid), NTHREADS, lds, s>>>(g, side);
    const int rc = launch_status();
    if (OP == OP_DW_TAIL && rc == SDP_OK) return tail_reduce<BM, BN>(g, d, s);
    return rc;
}

// Tile shapes (rows x columns), and what each costs: a workgroup takes step0 us a depth step on an otherwise idle chip and
// step1 us with all CUs at work, plus an epilogue of e0 us and e1 us per 1024 outputs that depends on what it moves; the
// launch takes as many such rounds as its tiles need on 256 CUs.  The 256-row tiles and 64 x 64 are fitted to 75 contractions
// of 15 MLP and attention shapes (128 to 8192 rows, depths of 128 to 8192) with row-major operands, each timed at every shape;
// the 128-row tiles and the SwiGLU backward's epilogue, for their present loop and stores under forward masking, to the launches
// of seven of these shapes (depths of 512 to 8192), where the choice is the fastest or within 6 % of it.  What the model does
// not know: depth-major operands, whose steps cost the same here though both at once take a tenth longer (256 x 192, 8192
// deep: 162 us against 147); the neuron-major stores of the SwiGLU backward; and the cut of a last round (plan_tail), which it
// prices as a whole one: 128-row tiles in whole rounds may then win over 256-row tiles with a cut round that would be faster
// (3976 x 1984 x 3, 15488 deep under backward masking: 652 us as chosen, 554 with 256 x 256 and their reduction, when the tokens
// were copied first; 4096 x 1536 x 3, 8192 deep 298 and 281; but 3944 x 1504 x 3, 9120 deep 343 and 365).
// The smaller shapes buy idle CUs at more L2 -> LDS traffic per flop: 4096 x 1200
// outputs, depth 3200: 57, 47, 41, 35, 46, 60 us in the order below; 8192 x 1536, depth 2048: 46, 44, 54, 49, 53, 94;
// 1500 x 1024, depth 1536: 29, 24, 19, 15, 12, 15.
enum Shape { T256x256, T256x192, T128x256, T128x192, T128x128, T64x64, NUM_SHAPES };
struct ShapeInfo {
    int bm, bn;
    double step0, step1;
};
constexpr ShapeInfo kShapes[NUM_SHAPES] = {{256, 256, 1.02, 1.35}, {256, 192, 0.87, 1.20}, {128, 256, 0.74, 0.84},
                                           {128, 192, 0.58, 0.78}, {128, 128, 0.47, 0.60}, {64, 64, 0.23, 0.22}};
struct EpilogueCost {
    double e0, e1;
};
constexpr EpilogueCost epilogue_cost(int epi) {
    return epi == EPI_SWIGLU_FWD ? EpilogueCost{5.0, 0.055} : epi == EPI_SWIGLU_BWD ? EpilogueCost{2.4, 0.36} : EpilogueCost{2.8, 0.03};
}
// the SwiGLU-forward epilogue pairs gate and up columns inside a wave's columns and has no 192- or 64-wide variant
constexpr bool shape_exists(int epi, int shape) {
    return epi != EPI_SWIGLU_FWD || (shape != T256x192 && shape != T128x192 && shape != T64x64);
}

// nbatch problems, the depth of each cut into ksplit ranges that are problems of their own
template <int EPI>
int64_t shape_tiles(const GemmDesc& d, int nbatch, int ksplit, int shape) {
    const int ncols = EPI == EPI_SWIGLU_FWD ? 2 * d.N : d.N; // gate and up interleaved double the tile columns
    const ShapeInfo& h = kShapes[shape];
    return (int64_t)((d.M + h.bm - 1) / h.bm) * ((ncols + h.bn - 1) / h.bn) * nbatch * ksplit;
}
// one round of it, on a chip of which this share of the CUs works
template <int EPI>
double round_cost(const GemmDesc& d, int ksplit, int shape, double busy) {
    const double steps = ((d.K + BK - 1) / BK + ksplit - 1) / ksplit * (EPI == EPI_DUAL_ACC ? 2 : 1);
    const EpilogueCost e = epilogue_cost(EPI);
    const ShapeInfo& h = kShapes[shape];
    return steps * (h.step0 + (h.step1 - h.step0) * busy) + e.e0 + e.e1 * h.bm * h.bn / 1024;
}
template <int EPI>
Shape choose_shape(const GemmDesc& d, int nbatch, int ksplit, double* round = nullptr, double* whole = nullptr) {
    const int force = tuning().force_tile - 1;
    Shape best = T256x256;
    double best_cost = -1;
    for (int i = 0; i < NUM_SHAPES; ++i) {
        if (!shape_exists(EPI, i) || (force >= 0 && i != force && shape_exists(EPI, force))) continue;
        const int64_t tiles = shape_tiles<EPI>(d, nbatch, ksplit, i), rounds = (tiles + kNumCU - 1) / kNumCU;
        const double one = round_cost<EPI>(d, ksplit, i, tiles < kNumCU ? (double)tiles / kNumCU : 1.0), cost = (double)rounds * one;
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost, best = (Shape)i;
            if (round) *round = one;
            if (whole) *whole = cost;
        }
    }
    return best;
}

template <int EPI, int OP, int KM = 0>
int launch(const GemmDesc& d, hipStream_t s) {
    const int nbatch = OP == OP_DW || OP == OP_DW_TAIL || OP == OP_DW_SPLIT ? d.nbatch : 1;
    double round = 0;
    const Shape shape = choose_shape<EPI>(d, nbatch, OP == OP_DW_SPLIT ? d.ksplit : 1, &round);
    if (shape == T256x256) return launch_cfg<256, 256, 2, 4, EPI, OP, KM>(d, round, s);
    if (shape == T128x256) return launch_cfg<128, 256, 2, 4, EPI, OP, KM>(d, round, s);
    if (shape == T128x128) return launch_cfg<128, 128, 4, 2, EPI, OP, KM>(d, round, s);
    if constexpr (EPI != EPI_SWIGLU_FWD) {
        if (shape == T256x192) return launch_cfg<256, 192, 4, 2, EPI, OP, KM>(d, round, s);
        if (shape == T128x192) return launch_cfg<128, 192, 4, 2, EPI, OP, KM>(d, round, s);
        if (shape == T64x64) return launch_cfg<64, 64, 2, 2, EPI, OP, KM>(d, round, s);
    }
    return SDP_ERR_UNSUPPORTED; // not reached: choose_shape returns one of the above
}

// Single problems whose right operand is depth-major as it is stored (down, dX and the attention's out and dX with the weights
// themselves in the place of transposed copies): LDS of one, with the list of its depth rows; 0: not such a shape.
template <int EPI>
int stored_lds(const GemmDesc& d, Shape shape) {
    const int list = d.b_gather ? list_bytes(d.K) : 0;
    if (shape == T64x64) return Geometry<64, 64, 2, 2, EPI, 2>::LDS + list;
    return shape == T128x128 ? Geometry<128, 128, 4, 2, EPI, 2>::LDS + list : 0;
}
// The 128 bytes that a 64-wide tile takes of a stored row are one line where rows are whole lines, else two: worth it for short
// depths alone then.  Event times of down, dX and the launches that made or carried the copies, two workers at T = 304, p = 4000
// (4032): d = 600 89 us with copies, 91 without; d = 640 84, 81; whole steps: T = 2000, d = 400, p = 2400 189 -> 197, T = 1176,
// d = 456, F = 5472 308 -> 323, but T = 1504, d = 504, p = 1000 131 -> 124.  A launch of its own has only the copy to win, and
// down at T = 928, d = 376, p = 1832 (29 steps) lost by it, four workers 267 -> 271 us; 20 steps (T = 520, d = 1888, p = 1272,
// eight workers 766 -> 743) are taken.
template <int EPI>
bool stored_lines(const GemmDesc& d, int most = 40) {
    return d.ldb % 64 == 0 || (d.K + BK - 1) / BK * (EPI == EPI_DUAL_ACC ? 2 : 1) <= most;
}
// In a launch of its own: 64 x 64 tiles.  A transposing pair of reads costs what two row-major reads do, so that the larger tiles do
// better with the copies that other launches carry (block of 4 x 1024 tokens, d = 1200, F = 3200 and its masked neighbour 1068 -> 1098 us
// with every 128-row tile this way); the smallest launches do better without.  Two workers, with copies / as stored: T = 256, d = 768,
// p = 1024 104 / 99 us, T = 512, d = 1024, F = 5504 under backward masking 282 / 250, T = 1000, d = 2048, p = 4128 522 / 516;
// attention of 500 tokens, 28 heads of 64 113 / 104.
template <int EPI>
bool stored_shape(const GemmDesc& d) {
    return choose_shape<EPI>(d, 1, 1) == T64x64 && stored_lines<EPI>(d, EPI == EPI_DUAL_ACC ? 40 : 20) && stored_lds<EPI>(d, T64x64) <= kMaxLds;
}

// Whether the launch of `d` is one to give its transposes to.  Their workgroups take 16 tiles each beside 256 x 256 and 128 x 256,
// 14 to 16 beside 256 x 192, 12 to 16 beside 128 x 192, 10 beside 128 x 128 and 8 beside 64 x 64; 7 are counted, which asks for
// idle CUs to spare.  Counted exactly, ten shapes whose choice between dact and dw that changes took, geometric mean, 1 % longer:
// two workers at T = 1800, d = 888, p = 2856 (dw to dact) 356 -> 364 us, at T = 1064, d = 520, p = 1832 (the other way) 162 -> 169,
// at T = 1064, d = 1320, F = 1520, p = 1080 under backward masking (the other way) 221 -> 215.  The launch then decides by carry
// with its own count, and transposes that it does not take run before it.
template <int EPI>
bool would_carry(const GemmDesc& d, int nbatch) {
    double round = 0;
    const ShapeInfo& h = kShapes[choose_shape<EPI>(d, nbatch, 1, &round)];
    int64_t side = 0;
    for (int i = 0; i < d.nside; ++i) side += (int64_t)((d.side[i].R + 63) / 64) * ((d.side[i].C + 63) / 64);
    const int64_t tiles = (int64_t)((d.M + h.bm - 1) / h.bm) * ((d.N + h.bn - 1) / h.bn) * nbatch;
    return carry(tiles, round, (side + 6) / 7);
}

// Tail cut of a batched launch (OP_DW_TAIL).  With T tiles on 256 CUs the launch runs floor(T / 256) full rounds
// and a last round of T mod 256 tiles; when that round leaves many CUs idle, each of its tiles is cut into
// `parts` depth ranges that spread over all CUs (every range at least 32 steps deep), at the price of one fp32
// tile per range written and read back.  Returns the number of ranges (0: no cut) for the shape choose_shape
// picks; *tail_tiles and *tile_elems describe the scratch.
int plan_tail(const GemmDesc& d, int* tail_tiles, int* tile_elems) {
    if (d.nbatch < 1 || d.N % 8 || d.M < 1 || d.K < 1) return 0;
    const ShapeInfo& shape = kShapes[choose_shape<EPI_STORE>(d, d.nbatch, 1)];
    const int bm = shape.bm, bn = shape.bn;
    const int64_t tiles = (int64_t)((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn) * d.nbatch;
    if (tiles > 0x7FFFFFFF) return 0;
    const int head = (int)(tiles / kNumCU) * kNumCU, tail = (int)tiles - head;
    if (head == 0 || tail == 0) return 0; // less than a round: the uniform depth cut (gemm_choose_ksplit) covers that case
    const int nk = (d.K + BK - 1) / BK;
    int best = 0;
    double best_cost = 0.85; // a cut has to shorten the last round by at least 15 % (of a whole tile's time)
    for (int parts = 2; parts <= 6 && nk / parts >= 32; ++parts) {
        const int rounds = (tail * parts + kNumCU - 1) / kNumCU;
        const double cost = (double)rounds / parts + 0.04 * parts; // the second term: traffic of the partial tiles
        if (cost < best_cost) best_cost = cost, best = parts;
    }
    if (tuning().tail_parts >= 0) best = tuning().tail_parts >= 2 && nk / tuning().tail_parts >= 32 ? tuning().tail_parts : 0;
    if (best == 0) return 0;
    const int steps = (nk + best - 1) / best;
    best = (nk + steps - 1) / steps; // no empty range
    if (tail_tiles) *tail_tiles = tail;
    if (tile_elems) *tile_elems = bm * bn;
    return best;
}

// sum of the depth ranges' fp32 partial results -> bf16 rows of the problems' outputs (optional row scatter);
// one thread per 8 columns
struct ReduceArgs {
    const float* partial;
    int ksplit, nbatch, M, N;
    uint16_t* Cb[kMaxBatch];
    int64_t ldc;
    const int32_t* cs;
    HeadList heads;
};
__global__ __launch_bounds__(256) void splitk_reduce_kernel(ReduceArgs r) {
    const int64_t per = (int64_t)r.M * (r.N / 8);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= per * r.nbatch) return;
    const int z = (int)(i / per);
    const int64_t rem = i - z * per;
    const int m = (int)(rem / (r.N / 8)), n = (int)(rem % (r.N / 8)) * 8;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    for (int k = 0; k < r.ksplit; ++k) { // ranges in depth order
        const float* p = r.partial + (((int64_t)k * r.nbatch + z) * r.M + m) * r.N + n;
        a += *(const f32x4*)p;
        b += *(const f32x4*)(p + 4);
    }
    uint16_t* out = z == 0 ? r.Cb[0] : (z == 1 ? r.Cb[1] : (z == 2 ? r.Cb[2] : r.Cb[3]));
    const int64_t row = listed_row(r.cs, r.heads, m);
    if (row < 0) return; // dropped row
    *(u32x4*)(out + row * r.ldc + n) = u32x4{pack_bf16(a[0], a[1]), pack_bf16(a[2], a[3]), pack_bf16(b[0], b[1]), pack_bf16(b[2], b[3])};
}

} // namespace

// A batched launch with few tiles and a deep K leaves most CUs idle for the whole depth of a tile.  Cutting
// the depth into r ranges multiplies the workgroups by r at the price of writing and re-reading r fp32
// copies of the outputs: taken when the 256 x 192 tiling has at most half as many tiles as there are CUs,
// r = as many as fit in one round (at most 4), every range at least 16 steps deep.
int gemm_choose_ksplit(int M, int N, int K, int nbatch) {
    if (nbatch < 1 || N % 8) return 1;
    const int64_t tiles = (int64_t)((M + 255) / 256) * ((N + 191) / 192) * nbatch;
    const int nk = (K + BK - 1) / BK;
    if (tiles * 2 > kNumCU) return 1;
    int r = (int)(kNumCU / tiles);
    r = r > 4 ? 4 : r;
    while (r > 1 && nk / r < 16) --r;
    if (r < 2) return 1;
    const int steps = (nk + r - 1) / r;
    return (nk + steps - 1) / steps; // no empty range
}

size_t gemm_split_ws_bytes(int M, int N, int K, int nbatch) {
    const int r = gemm_choose_ksplit(M, N, K, nbatch);
    return r > 1 ? (size_t)r * nbatch * M * N * sizeof(float) : 0;
}

size_t gemm_tail_ws_bytes(int M, int N, int K, int nbatch) {
    GemmDesc d;
    d.M = M, d.N = N, d.K = K, d.nbatch = nbatch;
    int tail = 0, elems = 0;
    const int parts = plan_tail(d, &tail, &elems);
    return parts > 1 ? (size_t)parts * tail * elems * sizeof(float) : 0;
}

bool gemm_mfma_supported(const GemmDesc& d) {
    if (d.M < 1 || d.N < 1 || d.K < 1) return false;
    // 16-byte global chunks (a depth that is no multiple of 64 ends in a step whose missing chunks are zeros: any
    // multiple of 8 will do.  T = 5000, d = 1600, p = 2664, whose depths p and T are odd multiples of 8: a step of two
    // workers takes 0.98 ms here, 12.0 ms with those depths on the plain kernel), 32-bit byte offsets inside each operand
    if ((d.K % 8 && !(d.a_km && d.b_km)) || d.lda % 8 || d.ldb % 8 || d.N % 8 || d.ldc % 8) return false;
    // depth-major operands: batched launches, B or both, columns in whole chunks; single ones, B
    if (d.b_km && d.nbatch == 0) {
        if (d.a_km || d.a_gather || !gemm_depth_major_ld(d.ldb) || !gemm_depth_major_ld(d.lda)) return false;
        if (d.b_gather && (d.b_rows <= 0 || d.K > (1 << 20) || d.b_rows * d.ldb * 2 >= ((int64_t)1 << 32))) return false;
        if (d.epilogue != EPI_STORE && d.epilogue != EPI_DUAL_ACC) return false;
    } else if (d.a_km || d.b_km) {
        if (d.nbatch == 0 || !d.b_km || d.b_gather || (d.a_km && (d.M % 8 || (d.a_gather && !d.a_gather_chunks)))) return false;
        if (!gemm_depth_major_ld(d.ldb) || (d.a_km && !gemm_depth_major_ld(d.lda))) return false;
        for (int z = 0; z < d.nbatch; ++z)
            if (z < kMaxBatch && (d.ldab[z] % 8 || !gemm_depth_major_ld(d.ldab[z]))) return false;
    } else if (d.nbatch > 0) {
        return false;
    }
    // the epilogue addresses a wave's part of the tile (at most 128 rows) with 32-bit byte offsets below 2^31
    constexpr int64_t kMaxLd = (int64_t)1 << 22;
    if (d.ldc >= kMaxLd || d.ldc3 >= kMaxLd || d.ldc3 % 8 || (d.R && d.ldr >= kMaxLd)) return false;
    if (d.epilogue == EPI_SWIGLU_BWD && (d.ldg >= kMaxLd || (d.Ct && d.ldct >= kMaxLd))) return false;
    if (!d.a_km && (d.a_rows > 0 ? d.a_rows : (int64_t)d.M) * d.lda * 2 >= ((int64_t)1 << 32)) return false;
    if (d.a_gather && (d.a_rows <= 0 || d.epilogue == EPI_DUAL_ACC)) return false;
    if (!d.b_km && (d.b_rows > 0 ? d.b_rows : (int64_t)d.N) * d.ldb * 2 >= ((int64_t)1 << 32)) return false;
    if (d.b_gather && d.b_rows <= 0) return false;
    if (d.R) {
        if (d.nbatch > 0 || (d.epilogue != EPI_STORE && d.epilogue != EPI_DUAL_ACC)) return false;
        if (!aligned16(d.R) || d.ldr % 8 || d.c_scatter) return false;
    }
    if (d.nbatch > 0) {
        if (d.nbatch > kMaxBatch || d.epilogue != EPI_STORE) return false;
        for (int z = 0; z < d.nbatch; ++z)
            if (!d.Ab[z] || !d.Bb[z] || !d.Cb[z] || !aligned16(d.Ab[z]) || !aligned16(d.Bb[z]) || !aligned16(d.Cb[z]))
                return false;
    } else {
        for (const void* p : {d.A, d.B, (const void*)d.C})
            if (!p || !aligned16(p)) return false;
    }
    if (d.epilogue == EPI_DUAL_ACC || d.epilogue == EPI_SWIGLU_FWD)
        if (!d.B2 || !aligned16(d.B2)) return false;
    if (d.epilogue == EPI_DUAL_ACC && (!d.A2 || !aligned16(d.A2))) return false;
    if (d.epilogue == EPI_SWIGLU_FWD) {
        if (!d.C2 || !d.C3 || !aligned16(d.C2) || !aligned16(d.C3)) return false;
    }
    if (d.epilogue == EPI_SWIGLU_BWD) {
        if (!d.C2 || !aligned16(d.C2) || (d.C3 && !aligned16(d.C3))) return false; // Act row-major is optional
        if (!d.Gin || !d.Uin || !aligned16(d.Gin) || !aligned16(d.Uin) || d.ldg % 8) return false;
        if (d.Cc || d.Cc2 || d.Cc3) return false; // row-major compact copies: plain kernel only
        if (d.Ct) {
            if (!d.Ct2 || !d.Ct3 || !aligned16(d.Ct) || !aligned16(d.Ct2) || !aligned16(d.Ct3)) return false;
            if (d.ldct % 8 || d.M % 8 || d.ldct < d.M) return false;
            if (d.cidx && !d.crank) return false;
        }
    }
    return true;
}

// depth ranges of a batched launch (both operands depth-major: the only kind whose callers bring the scratch)
static int uniform_cut(const GemmDesc& d) {
    return d.split_ws && d.a_km ? gemm_choose_ksplit(d.M, d.N, d.K, d.nbatch) : 1;
}

bool gemm_reads_as_stored(const GemmDesc& d) {
    if (!d.b_km || d.nbatch > 0 || !gemm_mfma_supported(d)) return false;
    return d.epilogue == EPI_STORE ? stored_shape<EPI_STORE>(d) : stored_shape<EPI_DUAL_ACC>(d);
}

namespace {

template <int BX, int BW, int EPIX, int KMX, int KMW>
int launch_pair(const GemmDesc& dx, const GemmDesc& dw, bool x_first, const char* name, hipStream_t s) {
    Dev x, w;
    int rc = describe<BX, BX, EPIX, EPIX == EPI_DUAL_ACC ? OP_DX : OP_DOWN>(dx, x);
    if (rc == SDP_OK) rc = describe<BW, BW, EPI_STORE, OP_DW>(dw, w);
    if (rc != SDP_OK) return rc;
    const int lx = stored_lds<EPIX>(dx, BX == 64 ? T64x64 : T128x128);
    constexpr int LW = BW == 64 ? Geometry<64, 64, 2, 2, EPI_STORE, KMW>::LDS : Geometry<128, 128, 4, 2, EPI_STORE, KMW>::LDS;
    const int lds = lx > LW ? lx : LW;
    if (lds > kMaxLds || dw.nside > 0) return SDP_ERR_INVALID_ARG;
    auto kern = sdp_gemm_pair_kernel<BX, BW, EPIX, KMX, KMW>;
    static const hipError_t attr = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (attr != hipSuccess) return SDP_ERR_HIP;
    ProfileScope ps(name, s);
    kern<<<dim3((unsigned)(x.ntot + w.ntot)), pair_threads<BX, BW>(), lds, s>>>(x, w, x_first ? 1 : 0);
    return launch_status();
}

struct PairPlan {
    Shape x, w;
    bool x_first;
};
// Side by side in the tiles that each would take alone, a workgroup per CU: worth it when the two, the longer tiles first, are
// modelled to end in 85 % of the time of one launch after the other (kGap: what a launch costs between two kernels).  Whole steps,
// one after the other / side by side: two workers at T = 2048, d = 768, p = 1024 160 / 129 us, T = 128, d = 256, p = 256 66 / 57,
// T = 1504, d = 504, p = 1000 131 / 124; attention of 1500 tokens, 4 of 8 heads of 128 116 / 105, 2 x 256 tokens, 6 heads of 64 53 / 49.
bool plan_pair(const GemmDesc& x, const GemmDesc& w, PairPlan& plan) {
    constexpr double kGap = 2.5;
    if (uniform_cut(w) > 1 || (w.tail_ws && plan_tail(w, nullptr, nullptr) > 1)) return false;
    const bool dual = x.epilogue == EPI_DUAL_ACC;
    double cx = 0, cw = 0;
    const Shape tw = choose_shape<EPI_STORE>(w, w.nbatch, 1, nullptr, &cw);
    const Shape tx = dual ? choose_shape<EPI_DUAL_ACC>(x, 1, 1, nullptr, &cx) : choose_shape<EPI_STORE>(x, 1, 1, nullptr, &cx);
    if ((tw != T128x128 && tw != T64x64) || (tx != T128x128 && tx != T64x64) || (tx == T128x128 && tw == T64x64)) return false;
    if (dual ? !stored_lines<EPI_DUAL_ACC>(x) || stored_lds<EPI_DUAL_ACC>(x, tx) > kMaxLds
             : !stored_lines<EPI_STORE>(x) || stored_lds<EPI_STORE>(x, tx) > kMaxLds)
        return false;
    const int64_t nx = shape_tiles<EPI_STORE>(x, 1, 1, tx), nw = shape_tiles<EPI_STORE>(w, w.nbatch, 1, tw);
    const double busy = nx + nw < kNumCU ? (double)(nx + nw) / kNumCU : 1.0;
    const double rx = dual ? round_cost<EPI_DUAL_ACC>(x, 1, tx, busy) : round_cost<EPI_STORE>(x, 1, tx, busy);
    const double rw = round_cost<EPI_STORE>(w, 1, tw, busy);
    plan = {tx, tw, rx > rw};
    const int64_t n1 = plan.x_first ? nx : nw, n2 = plan.x_first ? nw : nx, beside = kNumCU - n1; // long tiles, short ones
    const double r1 = plan.x_first ? rx : rw, r2 = plan.x_first ? rw : rx;
    if (beside <= 0) return false;
    // the short tiles all beside the long ones, or a round of them there and the others behind both
    const double all_beside = (double)((n2 + beside - 1) / beside) * r2, behind = n2 - beside <= kNumCU ? r1 + r2 : 1e30;
    const double end = all_beside < behind ? all_beside : behind;
    return (end > r1 ? end : r1) < 0.85 * (cx + cw + kGap);
}

} // namespace

bool gemm_pairs(const GemmDesc& x, const GemmDesc& w) {
    PairPlan plan;
    if (!x.b_km || x.nbatch > 0 || w.nbatch < 1 || w.nside > 0 || !w.b_km) return false;
    if (x.epilogue == EPI_STORE ? !w.a_km : x.b_gather && !w.a_km) return false; // not among the kernels of gemm_mfma_pair
    return gemm_mfma_supported(x) && gemm_mfma_supported(w) && plan_pair(x, w, plan);
}

int gemm_mfma_pair(const GemmDesc& x, const GemmDesc& w, const char* name, hipStream_t s) {
    PairPlan plan;
    if (!gemm_pairs(x, w) || !plan_pair(x, w, plan)) return SDP_ERR_UNSUPPORTED;
    auto go = [&](auto epi, auto kmx, auto kmw) {
        constexpr int EPI = decltype(epi)::value, KMX = decltype(kmx)::value, KMW = decltype(kmw)::value;
        if (plan.x == T128x128) return launch_pair<128, 128, EPI, KMX, KMW>(x, w, plan.x_first, name, s);
        if (plan.w == T128x128) return launch_pair<64, 128, EPI, KMX, KMW>(x, w, plan.x_first, name, s);
        return launch_pair<64, 64, EPI, KMX, KMW>(x, w, plan.x_first, name, s);
    };
    using std::integral_constant;
    constexpr integral_constant<int, EPI_DUAL_ACC> dual{};
    constexpr integral_constant<int, EPI_STORE> store{};
    constexpr integral_constant<int, 2> right{};
    constexpr integral_constant<int, 3> both{};
    constexpr integral_constant<int, 6> listed{};
    if (x.epilogue == EPI_STORE) return x.b_gather ? go(store, listed, both) : go(store, right, both);
    if (!w.a_km) return go(dual, right, right); // backward masking
    return x.b_gather ? go(dual, listed, both) : go(dual, right, both);
}

bool gemm_carries(const GemmDesc& d) {
    if (!gemm_mfma_supported(d)) return false;
    if (d.epilogue == EPI_SWIGLU_BWD) return would_carry<EPI_SWIGLU_BWD>(d, 1);
    if (d.nbatch == 0 || uniform_cut(d) > 1) return false;
    if (d.tail_ws && plan_tail(d, nullptr, nullptr) > 1) return false;
    return would_carry<EPI_STORE>(d, d.nbatch);
}

int gemm_mfma_bf16(const GemmDesc& d, hipStream_t s) {
    if (!gemm_mfma_supported(d)) return SDP_ERR_UNSUPPORTED;
    // OP only gives every call site its own kernel symbol, so that profiles name the step
    if (d.epilogue == EPI_STORE && d.nbatch > 0) {
        const int r = uniform_cut(d);
        if (r < 2 && d.tail_ws) {
            const int parts = plan_tail(d, nullptr, nullptr);
            if (parts > 1) {
                GemmDesc dt = d;
                dt.ksplit = parts;
                return d.a_km ? launch<EPI_STORE, OP_DW_TAIL, 3>(dt, s) : launch<EPI_STORE, OP_DW_TAIL, 2>(dt, s); // followed by its reduction
            }
        }
        if (r < 2) return d.a_km ? launch<EPI_STORE, OP_DW, 3>(d, s) : launch<EPI_STORE, OP_DW, 2>(d, s);
        GemmDesc ds = d;
        ds.ksplit = r;
        int rc = launch<EPI_STORE, OP_DW_SPLIT, 3>(ds, s);
        if (rc != SDP_OK) return rc;
        ReduceArgs ra{(const float*)d.split_ws, r, d.nbatch, d.M, d.N, {}, d.ldc, d.c_scatter, d.heads};
        for (int z = 0; z < kMaxBatch; ++z) ra.Cb[z] = (uint16_t*)d.Cb[z];
        const int64_t threads = (int64_t)d.nbatch * d.M * (d.N / 8);
        ProfileScope ps("splitk_reduce", s);
        splitk_reduce_kernel<<<(unsigned)((threads + 255) / 256), 256, 0, s>>>(ra);
        return launch_status();
    }
    if (d.b_km && d.nbatch == 0) {
        if (!gemm_reads_as_stored(d)) return SDP_ERR_UNSUPPORTED;
        if (d.epilogue == EPI_STORE) return d.b_gather ? launch_cfg<64, 64, 2, 2, EPI_STORE, OP_DOWN, 6>(d, 0, s) : launch_cfg<64, 64, 2, 2, EPI_STORE, OP_DOWN, 2>(d, 0, s);
        return d.b_gather ? launch_cfg<64, 64, 2, 2, EPI_DUAL_ACC, OP_DX, 6>(d, 0, s) : launch_cfg<64, 64, 2, 2, EPI_DUAL_ACC, OP_DX, 2>(d, 0, s);
    }
    if (d.epilogue == EPI_STORE && d.nbatch == 0) return launch<EPI_STORE, OP_DOWN>(d, s);
    if (d.epilogue == EPI_DUAL_ACC) return launch<EPI_DUAL_ACC, OP_DX>(d, s);
    if (d.epilogue == EPI_SWIGLU_FWD) return launch<EPI_SWIGLU_FWD, OP_GATE_UP>(d, s);
    if (d.epilogue == EPI_SWIGLU_BWD) return launch<EPI_SWIGLU_BWD, OP_DACT>(d, s);
    return SDP_ERR_UNSUPPORTED;
}

} // namespace sdp
